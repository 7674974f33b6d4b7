"""The native marshalling module only shortens the host time of four calls: without it the library builds and loads, and those
calls go the general way.  CPU only."""
import os
import shutil
import subprocess
import sys

import pytest

from paper_2602_05885_amd import build as pgbuild

SCRIPT = """
import warnings
import torch
from paper_2602_05885_amd import binding as B
with warnings.catch_warnings():
    warnings.simplefilter("error")          # calls that have nothing to do with it say nothing
    assert B.pg_workspace_bytes(256, 128, 512, 1, B.Params(), B.CALL_LOSS_FWD_BWD) > 0
f, u = torch.rand(4), torch.ones(4, dtype=torch.uint8)
with warnings.catch_warnings(record=True) as said:
    warnings.simplefilter("always")
    for call in (lambda: B.turn_reward(u, f[:-1], f), lambda: B.prs_retain(f, u[:-1], 1)):
        try:
            call()
        except AssertionError:              # the general path looks at the arguments
            continue
        raise SystemExit("the general path was not taken")
assert len(said) == 1 and "_stage_calls.so does not load" in str(said[0].message), said
print("fine")
"""


@pytest.mark.parametrize("module", [None, b"no shared object"])
def test_library_loads_without_the_module(tmp_path, module):
    pkg = tmp_path / "paper_2602_05885_amd"
    pkg.mkdir()
    for f in ("__init__.py", "binding.py", "libpg_head.so"):
        shutil.copy(os.path.join(pgbuild.PKG, f), pkg / f)
    if module is not None:
        (pkg / "_stage_calls.so").write_bytes(module)
    r = subprocess.run([sys.executable, "-c", SCRIPT], cwd=tmp_path, env=dict(os.environ, PYTHONPATH=str(tmp_path)), stdout=subprocess.PIPE, stderr=subprocess.STDOUT,
                       text=True, timeout=300)
    assert r.returncode == 0 and "fine" in r.stdout, r.stdout[-2000:]


def test_library_is_linked_where_the_module_does_not_build(tmp_path, monkeypatch):
    cc = tmp_path / "cc"                    # stands in for hipcc: writes what it is told to write
    cc.write_text('#!/bin/sh\nwhile [ $# -gt 0 ]; do if [ "$1" = -o ]; then echo built > "$2"; fi; shift; done\n')
    cc.chmod(0o755)
    monkeypatch.setattr(pgbuild, "PKG", str(tmp_path))
    monkeypatch.setattr(pgbuild, "LIB", str(tmp_path / "libpg_head.so"))
    monkeypatch.setattr(pgbuild, "STAGE_CALLS", str(tmp_path / "_stage_calls.so"))
    monkeypatch.setattr(pgbuild, "hipcc", lambda: str(cc))
    monkeypatch.setattr(pgbuild, "stage_calls_command", lambda: ["false"])
    (tmp_path / "_stage_calls.so").write_text("of an earlier build")
    with pytest.warns(UserWarning, match="did not build"):
        assert pgbuild.build(verbose=False) == str(tmp_path / "libpg_head.so")
    assert (tmp_path / "libpg_head.so").read_text() == "built\n"
    assert not (tmp_path / "_stage_calls.so").exists()
