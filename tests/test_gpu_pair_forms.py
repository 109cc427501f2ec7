"""The pair kernels' two forms of the sample loop (both directions with shared
exponentials; one direction at a time) and the rule between them.

Against the FP64 oracle: ordinary data at the edges of tiles and sample blocks,
and samples far out on one side of the 4 x 4 sub-blocks (tolerance of
gpu_helpers).  Against the separate form alone, which fp32_ties selects: samples
far out on both sides, and samples whose product of 1 + e^{-2u} overflows (the
wave then measures its pairs again).  With samples that far out the FP32 copies
alone move small measures by up to 6e-4 in either form, so that comparison is
for the faults the rule could have: a range measured in the other form without
its share of the signed sum moves E log cosh by u / n (0.02 at n = 2500), R by
its whole size; the tolerance is 1e-2 of a measure or of 1e-3 of the step's
largest.  Also a workspace without the shared form's region."""
import ctypes

import numpy as np
import pytest

import oracle
from paper_2403_03772_amd import lib as binding
from paper_2403_03772_amd import synth
from gpu_helpers import FLOOR, check_step

pytestmark = pytest.mark.gpu


def _data(d, n, far, seed):
    """Gene-family SEM with single samples moved far out in some variables."""
    X = synth.er_sem(d, n, indeg=2.0, noise_family=("uniform", "laplace", "exp"), seed=seed).X
    sd = X.std(axis=0)
    if far == "one side":      # every other sub-block of four variables
        cols = [v for v in range(d) if (v // 4) % 2 == 0]
        X[n // 3, cols] = 20.0 * sd[cols]
    elif far == "both":        # all variables, in different samples: |z| past 13 everywhere
        for v in range(d):
            X[(7 * v) % n, v] = (-1.0) ** v * 18.0 * sd[v]
    elif far == "overflow":    # u past 44 (2^(2 u log2 e) > 2^127) in one variable of sixteen
        for v in range(0, d, 16):
            X[(11 * v) % n, v] = -1e4 * sd[v]
    return np.ascontiguousarray(X, dtype=np.float32)


def _check_oracle(X, order, mg):
    _, mr, _ = oracle.causal_order(X, forced=order, mode="table", with_measures=True)
    for t in range(X.shape[1] - 1):
        bad, ok = check_step(mg[t], mr[t], order[t])
        assert bad == 0, f"step {t}: {bad} measures outside tolerance"
        assert ok, f"step {t}: chose {order[t]} outside a near-tie"


@pytest.mark.parametrize("d,n,far", [
    (66, 640, "none"), (73, 2049, "none"), (80, 64 * 33, "one side"), (97, 3000, "one side")])
def test_forms_match_oracle(lib, d, n, far):
    import torch
    X = _data(d, n, far, 900 + d)
    print(f"pair forms d={d} n={n} far={far}", flush=True)
    out = lib.causal_order(torch.as_tensor(X).cuda(), with_measures=True)
    _check_oracle(X, out["order"].cpu().numpy(), out["measures"].cpu().numpy())


@pytest.mark.parametrize("d,n,far", [
    (72, 2500, "both"), (65, 500, "both"), (81, 2500, "overflow"), (100, 9001, "overflow"),
    (97, 3000, "one side"), (130, 300, "none")])
def test_forms_match_each_other(lib, d, n, far):
    import torch
    X = torch.as_tensor(_data(d, n, far, 900 + d)).cuda()
    print(f"pair forms d={d} n={n} far={far}", flush=True)
    order = lib.causal_order(X)
    a = lib.causal_order(X, forced=order, with_measures=True)["measures"].cpu().numpy()
    b = lib.causal_order(X, forced=order, with_measures=True, fp32_ties=True)
    b = b["measures"].cpu().numpy()
    for t in range(d - 1):
        on = np.isfinite(b[t])
        assert np.array_equal(on, np.isfinite(a[t]))
        off = np.abs(a[t][on] - b[t][on]) / np.maximum(np.abs(b[t][on]), FLOOR * -b[t][on].min())
        assert off.max() <= 1e-2, f"step {t}: {off.max():.2e}"


@pytest.mark.parametrize("d,n", [(70, 1000), (130, 777)])
def test_small_workspace_takes_the_separate_form(lib, d, n):
    """A workspace that lacks only the shared form's region (4 (d + 1) n_pad
    bytes, the last one) is accepted, and measures within the tolerance."""
    import torch
    X = _data(d, n, "none", 950 + d)
    Xd = torch.as_tensor(X).cuda()
    L = lib.load()
    need = lib.workspace_size(n, d)
    region = -(-(4 * (d + 1) * (-(-n // 64) * 64)) // 256) * 256
    order = torch.empty(d, dtype=torch.int32, device="cuda")
    meas = torch.empty((d - 1, d), dtype=torch.float64, device="cuda")
    opts, _, _ = binding._new_opts(L)
    opts.step_measures = meas.data_ptr()
    for size, ok in ((need - region, True), (need - region - 256, False)):
        ws = torch.empty(size, dtype=torch.uint8, device="cuda")
        print(f"workspace d={d} n={n} bytes={size}", flush=True)
        code = L.lingam_causal_order(binding._ptr(Xd), n, d, d, binding._ptr(order),
                                     ctypes.byref(opts), binding._ptr(ws), size, None)
        torch.cuda.synchronize()
        assert code == (binding.OK if ok else binding.E_WORKSPACE)
        if ok:
            o = order.cpu().numpy()
            _check_oracle(X, o, meas.cpu().numpy())
            assert np.array_equal(o, lib.causal_order(Xd).cpu().numpy())
