"""Work items of the pair kernels (tests/pair_items_check.cpp): a job that may not take
the shared form has a workgroup for each residual direction, as many in all as the
grids are sized for, each (tile, split, direction, quadrant) once."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_items_cover_every_direction_once(tmp_path):
    from paper_2403_03772_amd import build as b
    hipcc = b.HIPCC if os.path.exists(b.HIPCC) else shutil.which("hipcc")
    if not hipcc:
        pytest.skip("hipcc not found")
    exe = str(tmp_path / "pair_items_check")
    r = subprocess.run([hipcc, "-std=c++17", "-O2", "-I", b.INCLUDE, "-I", b.CSRC,
                        os.path.join(ROOT, "tests", "pair_items_check.cpp"), "-o", exe],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-3000:]
    r = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0 and r.stdout.strip() == "ok", r.stdout
