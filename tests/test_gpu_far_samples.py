"""Heavy tails: variables with samples past the pair kernels' shared form.

Sub-blocks with such variables on both sides take the separate form over all
samples, with sums that leave nothing out, as every sub-block does under fp32_ties:
where all variables are far out, a step's measures are those of fp32_ties bit for bit.
Where some are, the candidate, suspect and extension rows of the learned form and the
all-pairs kernel group the variables differently, so their forms differ; a measure
whose sums were taken for the other form's would be off by the signed sum of its
residuals (E log cosh by u / n, R by its whole size), and the forms' own rounding on
samples that far out is 6e-4 of a measure: tolerance 1e-2 of a measure or of 1e-3 of
the step's largest.  The orders are equal: near-ties are decided in FP64."""
import numpy as np
import pytest

from paper_2403_03772_amd import synth
from gpu_helpers import FLOOR

pytestmark = pytest.mark.gpu


def _data(d, n, every, seed):
    """Gene-family SEM; every `every`-th variable gets a sample past 13 deviations (a
    sample of its own, so that no pair becomes collinear)."""
    import torch
    X = synth.er_sem(d, n, indeg=2.0, noise_family=("uniform", "laplace", "exp"), seed=seed).X
    sd = X.std(axis=0)
    for v in range(0, d, every):
        X[(7 * v) % n, v] = (-1.0) ** v * 20.0 * sd[v]
    return torch.as_tensor(np.ascontiguousarray(X, dtype=np.float32)).cuda()


@pytest.mark.parametrize("d,n", [(65, 4000), (72, 2500), (131, 1800), (200, 700)])
def test_far_on_both_sides_equals_the_separate_form(lib, d, n):
    X = _data(d, n, 1, 40 + d)
    print(f"far both d={d} n={n}", flush=True)
    a = lib.causal_order(X, with_measures=True)["measures"][0].cpu().numpy()
    b = lib.causal_order(X, with_measures=True, fp32_ties=True)["measures"][0].cpu().numpy()
    assert np.isfinite(a).all() and np.array_equal(a, b)


def _close(a, b):
    on = np.isfinite(a) & np.isfinite(b)
    if not on.any():
        return
    off = np.abs(a[on] - b[on]) / np.maximum(np.abs(b[on]), FLOOR * -np.nanmin(b))
    assert off.max() <= 1e-2, off.max()


@pytest.mark.parametrize("every", [1, 3, 7])
def test_sub_blocks_of_either_kind(lib, every):
    import torch
    d, n = 150, 2200
    X = _data(d, n, every, 3 + every)
    print(f"far every {every} of d={d} n={n}", flush=True)
    order = lib.causal_order(X)
    a = lib.causal_order(X, forced=order, with_measures=True)["measures"].cpu().numpy()
    b = lib.causal_order(X, forced=order, with_measures=True, fp32_ties=True)
    b = b["measures"].cpu().numpy()
    for t in range(d - 1):
        assert np.array_equal(np.isfinite(a[t]), np.isfinite(b[t]))
        _close(a[t], b[t])


@pytest.mark.parametrize("every,extension", [(1, 0), (3, 0), (1, 64), (3, 64), (5, 64)])
def test_learned_rows(lib, every, extension):
    import torch
    from paper_2403_03772_amd import train_proposer
    d, n = 300, 1600
    X = _data(d, n, every, 90 + every)
    raw = train_proposer.default_proposer().clone()
    raw[32:] = torch.as_tensor(train_proposer.init_weights(1), device="cuda")
    plain = lib.causal_order(X, with_measures=True)
    m = plain["measures"].cpu().numpy()
    for P in (train_proposer.default_proposer(), raw):
        print(f"learned far every {every} extension={extension}", flush=True)
        out = lib.causal_order(X, with_measures=True,
                               learned=lib.Learned(P, topk=32, extension=extension))
        assert out["learned_stats"].learned_steps > 0
        assert torch.equal(out["order"], plain["order"])
        rows = out["measures"].cpu().numpy()
        for t in range(d - 1):
            _close(rows[t], m[t])
