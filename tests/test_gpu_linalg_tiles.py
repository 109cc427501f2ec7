"""FP64 linear algebra by 32-wide blocks at the edges of its blocks: the blocked
Cholesky factor with its inverse (adjacency along a given order), the inverse of
a unit lower-triangular matrix merged level by level (total effects), and
covariances whose samples are split over workgroups, against numpy in FP64.

Both sides see the same data and differ in the order of FP64 roundings only:
p eps times the condition number (below 1e4 here) is under 1e-9 of the largest
coefficient; the bound is 1e-8, as for the other adjacency tests.
"""
import numpy as np
import pytest

import oracle
from gpu_helpers import measure_close

pytestmark = pytest.mark.gpu


def _data(p, n, seed):
    """Noise mixed by a sparse lower-triangular map along a random order."""
    rng = np.random.default_rng(seed)
    L = np.tril(rng.uniform(-0.5, 0.5, (p, p)), -1)
    L *= rng.random((p, p)) < min(1.0, 3.0 / p)
    order = rng.permutation(p)
    X = np.empty((n, p))
    X[:, order] = rng.laplace(size=(n, p)) @ np.linalg.inv(np.eye(p) - L).T
    return X.astype(np.float32), order.astype(np.int32)


def _reference(X32, order):
    """B by ordinary least squares along the order, through the factor of the covariance."""
    X = X32.astype(np.float64)[:, order]
    X -= X.mean(axis=0)
    L = np.linalg.cholesky(X.T @ X)
    Li = np.linalg.inv(L)
    P = -np.tril(np.diag(L)[:, None] * Li, -1)
    B = np.zeros_like(P)
    B[np.ix_(order, order)] = P
    return B


# p: one block less one, exact, plus one; each level of merged pairs full, cut
# in its second half and without one.  n: fewer than 256 samples (no split), a
# remainder in the last chunk, a last range that is short or empty.
@pytest.mark.parametrize("p,n", [(1, 40), (31, 255), (32, 256), (33, 257), (63, 2049), (64, 1000),
                                 (65, 5121), (95, 300), (96, 777), (97, 2000), (128, 513),
                                 (129, 4000), (191, 700), (225, 1031), (257, 900)])
def test_block_edges(lib, p, n):
    import torch
    print(f"case p={p} n={n}", flush=True)
    X32, order = _data(p, n, seed=p + n)
    B = lib.adjacency(torch.as_tensor(X32).cuda(), order)
    ref = _reference(X32, order)
    tol = 1e-8 * max(1.0, np.abs(ref).max())
    assert np.abs(B.cpu().numpy() - ref).max() <= tol
    T = lib.total_effects(B, order).cpu().numpy()
    full = np.linalg.inv(np.eye(p) - ref)
    assert np.abs(T - full).max() <= 1e-8 * np.abs(full).max()


@pytest.mark.parametrize("d,n", [(2, 255), (3, 257), (10, 2049), (32, 999), (33, 3000),
                                 (64, 640), (97, 1300)])
def test_split_correlations_of_a_job(lib, d, n):
    """A job's correlation matrix, added up from ranges of samples: every
    measure of its first step within the tolerance of the other parity tests (a
    lost or doubled range moves them by more than its samples' share, 1/12 here)."""
    import torch
    print(f"case d={d} n={n}", flush=True)
    X32, _ = _data(d, n, seed=7 * d + n)
    out = lib.causal_order(torch.as_tensor(X32).cuda(), with_measures=True)
    first = int(out["order"][0])
    _, ref, _ = oracle.causal_order(X32.astype(np.float64), forced=[first], mode="table",
                                    with_measures=True)
    assert measure_close(out["measures"][0].cpu().numpy(), ref[0]).all()


@pytest.mark.parametrize("p,n", [(5, 3000), (40, 1111)])
def test_workspace_without_partial_tiles(lib, p, n):
    """A workspace a byte short of the query holds all but the partial covariance
    tiles: accepted, one range of samples, the same coefficients."""
    import torch
    from paper_2403_03772_amd import lib as binding
    L = binding.load()
    print(f"case p={p} n={n}", flush=True)
    X32, order = _data(p, n, seed=3 * p + n)
    X, o = torch.as_tensor(X32).cuda(), torch.as_tensor(order).cuda()
    need = int(L.lingam_adjacency_workspace_size(n, p))
    ws = torch.empty(need, dtype=torch.uint8, device="cuda")
    B = torch.empty((p, p), dtype=torch.float64, device="cuda")
    code = L.lingam_adjacency(binding._ptr(X), n, p, None, n, p, binding._ptr(o), binding._ptr(B),
                              binding._ptr(ws), need - 1, binding._stream_ptr(torch, X.device))
    assert code == 0
    ref = _reference(X32, order)
    assert np.abs(B.cpu().numpy() - ref).max() <= 1e-8 * max(1.0, np.abs(ref).max())
