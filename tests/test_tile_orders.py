"""Which tile runs where (no GPU): the small-size kernels' tile order
(dmpt_tiles.h, small_split) and the general products' job lists (build_prod_list,
dmpt_lists.h), compiled into a host program (tests/csrc/tile_orders_check.cpp) and
run over every padded size up to 4608 (1536 - 9216 for the lists), both tile
edges, several observables, kinds and numbers of CUs.  Every tile runs once, every
entry of the partial sums is written once and lies in its area."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2409_17033_amd", "csrc")


@pytest.fixture(scope="module")
def checker(tmp_path_factory):
    hipcc = os.environ.get("HIPCC") or shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(hipcc) and not shutil.which(hipcc):
        pytest.skip("hipcc not found")
    exe = str(tmp_path_factory.mktemp("orders") / "tile_orders_check")
    r = subprocess.run([hipcc, "--offload-arch=gfx950", "-O2", "-std=c++17", "-I", CSRC,
                        os.path.join(ROOT, "tests", "csrc", "tile_orders_check.cpp"), "-o", exe],
                       capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stderr[-2000:]
    return exe


def test_every_tile_runs_once(checker):
    r = subprocess.run([checker], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stdout[-2000:] + r.stderr[-2000:]


def test_checker_sees_a_missing_tile(checker):
    r = subprocess.run([checker, "drop"], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stdout[-500:] + r.stderr[-2000:]
    assert r.stdout.count("FAIL") > 1000
