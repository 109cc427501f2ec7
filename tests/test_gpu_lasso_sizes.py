"""Pruned adjacency at the edges of its lasso kernel: active sets at the sizes of
a wave, of its rows of sixteen and of the cap, predecessors at the sizes of a
workgroup, and the path state on either side of its LDS limit (1024
predecessors).  Sampled rows against the oracle, FP64 on both sides: the kept
predictors exactly, their coefficients to 1e-8 of the largest.
"""
import numpy as np
import pytest

from oracle import lasso as LA
from paper_2403_03772_amd import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d,n,indeg,cap", [(18, 400, 17.0, 64), (66, 900, 40.0, 64),
                                           (66, 900, 40.0, 63), (66, 900, 40.0, 17),
                                           (258, 1200, 3.0, 64), (1025, 2500, 2.0, 64),
                                           (1026, 2500, 2.0, 64)])
def test_sampled_rows_match_oracle(lib, d, n, indeg, cap):
    import torch
    print(f"case d={d} n={n} indeg={indeg} cap={cap}", flush=True)
    s = synth.er_sem(d, n, indeg=indeg, noise_family=("uniform", "laplace", "exp"), seed=d + cap)
    X32 = np.ascontiguousarray(s.X, dtype=np.float32)
    B = lib.adjacency_pruned(torch.as_tensor(X32).cuda(), s.order, max_active=cap).cpu().numpy()
    pos = [q for q in (1, 15, 16, 17, 63, 64, 65, 255, 256, 257, 1023, 1024, 1025) if q < d]
    ref = LA.adaptive_lasso_adjacency(X32.astype(np.float64), s.order, max_active=cap,
                                      positions=pos)
    for q in pos:
        y = s.order[q]
        assert np.array_equal(B[y] != 0, ref[y] != 0), q
        assert np.max(np.abs(B[y] - ref[y])) <= 1e-8 * max(1.0, np.max(np.abs(ref[y]))), q
