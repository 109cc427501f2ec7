"""The pair kernels' registers and LDS against the residency that their bounded grids
are sized for (pair_waves_per_cu), and no spilled registers: their loops are bound by
instruction issue, and a spill doubles their time without a wrong result."""
import os
import re
import shutil
import subprocess

import pytest

CU_LDS, SIMD_VGPRS, SIMDS = 160 * 1024, 512, 4


@pytest.fixture(scope="module")
def hipcc():
    from paper_2403_03772_amd import build as b
    h = b.HIPCC if os.path.exists(b.HIPCC) else shutil.which("hipcc")
    if not h:
        pytest.skip("hipcc not found")
    return h, b


@pytest.fixture(scope="module")
def kernels(hipcc, tmp_path_factory):
    """name -> (waves a workgroup, registers, spilled registers, LDS bytes)"""
    h, b = hipcc
    d = tmp_path_factory.mktemp("asm")
    runs = []
    for src in ("lingam_kernels.hip", "lingam_learned.hip"):
        out = str(d / (src + ".s"))
        runs.append((out, subprocess.Popen(
            [h, *[f for f in b.COMMON if f != "-fPIC"], "-S", "--cuda-device-only", "-o", out,
             os.path.join(b.CSRC, src)], stdout=subprocess.PIPE, stderr=subprocess.PIPE)))
    found = {}
    for out, p in runs:
        assert p.wait(timeout=300) == 0, p.stderr.read().decode()[-2000:]
        for block in re.split(r"\n  - (?=\.a)", open(out).read().split("amdhsa.kernels:")[1]):
            name = re.search(r"\.name: +(\S+)", block)
            if name and re.search(r"\dk_pair(_loop|_cand|_susp|_ext)?ILi", name.group(1)):
                v = [int(re.search(rf"\.{k}: +(\d+)", block).group(1)) for k in (
                    "max_flat_workgroup_size", "vgpr_count", "vgpr_spill_count",
                    "group_segment_fixed_size")]
                found[name.group(1)] = (v[0] // 64, *v[1:])
    assert len(found) == 30, sorted(found)  # five kernels of 1, 2 and 4 waves, two forms
    return found


def test_no_register_is_spilled(kernels):
    assert {n: k[2] for n, k in kernels.items() if k[2]} == {}


def test_bounded_grids_match_the_residency(hipcc, kernels, tmp_path):
    h, b = hipcc
    src, exe = tmp_path / "waves.cpp", tmp_path / "waves"
    src.write_text('#include <cstdio>\n#include "lingam_internal.h"\n'
                   'int main() { std::printf("%d %d", lg::pair_waves_per_cu(false),'
                   ' lg::pair_waves_per_cu(true)); }\n')
    subprocess.run([h, "-std=c++17", "-I", b.INCLUDE, "-I", b.CSRC, str(src), "-o", str(exe)],
                   check=True, capture_output=True)
    planned = subprocess.run([str(exe)], capture_output=True, text=True).stdout.split()
    for name, (waves, vgprs, _, lds) in kernels.items():
        resident = SIMDS * (SIMD_VGPRS // (-(-vgprs // 8) * 8)) // waves
        want = int(planned["Lb1E" in name])  # kShared
        assert min(resident, CU_LDS // lds) * waves == want, name
