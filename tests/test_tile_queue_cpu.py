"""Host-side sweep of the persistent kernels' tile orders and queue shares (tests/tile_queue_driver.hip):
the integer functions the kernels use on the device are compiled for the host as well and checked to hand out
every tile exactly once, for both orders and several thousand tile counts.  CPU only."""
import os
import random
import shutil
import subprocess

import pytest

from paper_2602_05885_amd import build as pgbuild
from tests._cases import dh_form

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


pytestmark = pytest.mark.skipif(shutil.which("hipcc") is None and not os.path.exists("/opt/rocm/bin/hipcc"), reason="needs hipcc")


@pytest.fixture(scope="module")
def driver(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("tile_queue") / "tile_queue_driver")
    flags = [f for f in pgbuild.FLAGS if f not in ("-fPIC",)]
    subprocess.run([pgbuild.hipcc(), *flags, os.path.join(ROOT, "tests", "tile_queue_driver.hip"), "-o", exe],
                   check=True, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True, timeout=300)
    return exe


def test_every_tile_is_handed_out_exactly_once(driver):
    r = subprocess.run([driver], stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True, timeout=120)
    assert r.returncode == 0 and "(0 failures)" in r.stdout, r.stdout[-2000:]


def test_the_restated_dh_rule_is_the_library_s(driver):
    rng = random.Random(5)
    cases = []
    for _ in range(3000):
        n_pad = 256 * int(2 ** rng.uniform(0, 8))
        acc_rows = rng.choice([n_pad, max(n_pad, 32768), int(n_pad * 2 ** rng.uniform(0, 6.5))])
        cases.append((n_pad, acc_rows, 64 * int(2 ** rng.uniform(0, 7)), int(2 ** rng.uniform(0, 13)), rng.randrange(2), rng.randrange(2)))
    r = subprocess.run([driver, "forms"], input="".join("%d %d %d %d %d %d\n" % c for c in cases), capture_output=True, text=True, timeout=120)
    got = [tuple(int(x) for x in line.split()) for line in r.stdout.splitlines()]
    assert len(got) == len(cases)
    for c, f in zip(cases, got):
        assert f == tuple(int(x) for x in dh_form(*c)), c
