"""Order of the FP64 pair kernel's work items over the XCDs
(tests/pair64_order_check.cpp): no XCD gets more than 1.1 of the mean of the samples,
whether or not the jobs of a batch are of one length."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_every_xcd_gets_its_share(tmp_path):
    from paper_2403_03772_amd import build as b
    hipcc = b.HIPCC if os.path.exists(b.HIPCC) else shutil.which("hipcc")
    if not hipcc:
        pytest.skip("hipcc not found")
    exe = str(tmp_path / "pair64_order_check")
    r = subprocess.run([hipcc, "-std=c++17", "-O2", "-I", b.INCLUDE, "-I", b.CSRC,
                        os.path.join(ROOT, "tests", "pair64_order_check.cpp"), "-o", exe],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-3000:]
    r = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0 and r.stdout.strip() == "ok", r.stdout
