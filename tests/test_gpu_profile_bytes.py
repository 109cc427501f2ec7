"""lingam_profile.resid_bytes: what the residual kernel moves, with and without the
exponentials of the pair kernels' shared form."""
import ctypes

import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("least,bytes_each", [(False, 32), (True, 28)])
def test_bytes_of_the_residual_update(lib, least, bytes_each):
    import torch
    from paper_2403_03772_amd import lib as binding
    L, (n, d) = binding.load(), (500, 70)
    X = torch.rand((n, d), device="cuda") ** 3
    opts, prof, _ = binding._new_opts(L, profile=True)
    query = lambda o: L.lingam_workspace_size(n, d, o)
    size = int(binding._least(query, opts) if least else query(ctypes.byref(opts)))
    ws = torch.empty(size, dtype=torch.uint8, device="cuda")
    order = torch.empty(d, dtype=torch.int32, device="cuda")
    print(f"case n={n} d={d} bytes={size}", flush=True)
    assert L.lingam_causal_order(binding._ptr(X), n, d, d, binding._ptr(order),
                                 ctypes.byref(opts), binding._ptr(ws), size, None) == 0
    steps = sum(m - 1 for m in range(3, d + 1))
    assert prof.resid_bytes == bytes_each * n * steps
