"""Pruned adjacency by the lasso kernel that holds rows of the correlation matrix in
registers (up to 256 predecessors, a thread each): its largest size, positions at the
edges of all four waves, and paths on which predictors leave again before the kept
breakpoint, so that the rows move down.  Sampled rows against the oracle, FP64 on both
sides: the kept predictors exactly, their coefficients to 1e-8 of the largest."""
import numpy as np
import pytest

from oracle import lasso as LA
from paper_2403_03772_amd import synth

pytestmark = pytest.mark.gpu


def _leaves(X, order, q, cap):
    """Predictors that leave the path of position q before its kept breakpoint."""
    Z = (X - X.mean(axis=0)) / X.std(axis=0)
    A, y = Z[:, order[:q]], Z[:, order[q]]
    b = np.linalg.solve(A.T @ A, A.T @ y)
    A = A * np.abs(b)
    G, c = A.T @ A, A.T @ y
    path = LA.lars_lasso_path(G, c, cap)
    kept = LA.bic_select(G, c, len(Z), len(Z) - b @ (Z[:, order[:q]].T @ y), path)
    return sum(bool(np.any((path[i - 1] != 0) & (path[i] == 0))) for i in range(1, kept + 1))


@pytest.mark.parametrize("d,n,indeg,seed,leave", [
    (257, 1200, 3.0, 321, False), (200, 500, 20.0, 1, True), (200, 400, 30.0, 2, True),
    (256, 700, 30.0, 5, True)])
def test_rows_in_registers_match_oracle(lib, d, n, indeg, seed, leave):
    import torch
    s = synth.er_sem(d, n, indeg=indeg, noise_family=("uniform", "laplace", "exp"), seed=seed)
    X32 = np.ascontiguousarray(s.X, dtype=np.float32)
    X = X32.astype(np.float64)
    pos = [q for q in (64, 127, 128, 129, 170, 191, 192, 193, 199, 255, 256) if q < d]
    print(f"case d={d} n={n} indeg={indeg}", flush=True)
    B = lib.adjacency_pruned(torch.as_tensor(X32).cuda(), s.order).cpu().numpy()
    ref = LA.adaptive_lasso_adjacency(X, s.order, max_active=64, positions=pos)
    left = [_leaves(X, s.order, q, 64) for q in pos if q > 128]
    assert not leave or min(left[-3:]) > 0, left
    for q in pos:
        y = s.order[q]
        assert np.array_equal(B[y] != 0, ref[y] != 0), q
        assert np.max(np.abs(B[y] - ref[y])) <= 1e-8 * max(1.0, np.max(np.abs(ref[y]))), q
