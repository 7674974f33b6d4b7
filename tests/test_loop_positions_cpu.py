"""Where the main loops of the built library begin within the 32-byte pieces that instructions are fetched in: the speed of the
MFMA kernels hangs on it, and a position left to itself changes with any line in front of the loop.  CPU only (a listing of this
package's own kernels)."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2602_05885_amd import build as pgbuild

OBJDUMP = next((p for p in (shutil.which("llvm-objdump"), "/opt/rocm/llvm/bin/llvm-objdump") if p and os.path.exists(p)), None)
STAGE_MFMAS = (32, 48, 64)      # of one stage of a main loop, per wavefront


def _loops(listing):
    """(kernel, MFMA instructions, first byte) of every innermost loop that has MFMA instructions."""
    for kernel in re.split(r"\n(?=[0-9a-f]{16} <)", listing):
        name = re.match(r"[0-9a-f]{16} <(\S+)>:", kernel)
        if not name or "v_mfma" not in kernel:
            continue
        code = [(int(m.group(1), 16), line) for line in kernel.split("\n") for m in [re.search(r"// ([0-9A-F]{12}):", line)] if m]
        mfma = [at for at, line in code if "v_mfma" in line]
        for at, line in code:
            jump = re.match(r"\s*s_c?branch\S* (\d+)", line)
            if jump:
                offset = int(jump.group(1))
                to = at + 4 + 4 * (offset - 65536 if offset >= 32768 else offset)
                inside = sum(to <= a <= at for a in mfma)
                if to < at and at - to < 2048 and inside in STAGE_MFMAS:
                    yield name.group(1), inside, to


@pytest.mark.skipif(OBJDUMP is None, reason="needs llvm-objdump")
def test_main_loops_begin_where_they_run_well(tmp_path):
    so = tmp_path / "lib.so"
    shutil.copy(pgbuild.LIB, so)
    subprocess.run([OBJDUMP, "--offloading", str(so)], check=True, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, timeout=120)
    found = []
    for f in sorted(tmp_path.glob("lib.so.*amdgcn*")):
        listing = subprocess.run([OBJDUMP, "-d", "--mcpu=gfx950", str(f)], check=True, stdout=subprocess.PIPE, text=True, timeout=120).stdout
        found += list(_loops(listing))
    count = {k: sum(k in name for name, _, _ in found) for k in ("lmhead_fwd_kernel", "lmhead_dlogits_kernel", "gemm_store_kernel")}
    assert count == {"lmhead_fwd_kernel": 3, "lmhead_dlogits_kernel": 2, "gemm_store_kernel": 6}, found
    for name, mfmas, at in found:
        assert at % 32 >= (16 if "lmhead_fwd" in name else 8), (name, mfmas, at % 32)
