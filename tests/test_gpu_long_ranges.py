"""Sample ranges longer than the pair kernels' shared form counts exponents for (4096
blocks of 64 samples a wave): two ranges of 4097 blocks, measured in the separate form
and made those of the shared form.  The halves of the data have different means, so
that either range's signed sum is far from 0: left in, it would move E log cosh by a
quarter.  Against fp32_ties, which measures the same sums and adds nothing; what may
differ is the sums' scale, rounded to FP32 (6e-8 of sums below n / 2), within the
tolerance of gpu_helpers."""
import numpy as np
import pytest

from gpu_helpers import FLOOR, REL

pytestmark = pytest.mark.gpu


def test_ranges_past_the_shared_form(lib):
    import torch
    d, n = 256, 2 * 64 * 4097  # 528 tiles, 1056 items: two splits at 8 items of 256 CUs
    g = torch.Generator(device="cuda").manual_seed(12)
    X = torch.rand((n, d), generator=g, device="cuda") ** 2
    X[: n // 2] += 0.5 * torch.rand(d, generator=g, device="cuda")
    for k in range(1, d):
        X[:, k] += 0.6 * X[:, k - 1]
    print(f"case d={d} n={n}", flush=True)
    a = lib.causal_order(X, with_measures=True)["measures"][0].cpu().numpy()
    b = lib.causal_order(X, with_measures=True, fp32_ties=True)["measures"][0].cpu().numpy()
    assert np.isfinite(a).all()
    off = np.abs(a - b) / np.maximum(np.abs(b), FLOOR * np.abs(b).max())
    assert off.max() <= REL, off.max()
