"""A batch in the smallest workspace it accepts: the sizes below are those that the
query gave before the pair kernels' shared form and the second schedule had their
regions (256 CUs), so callers that kept them are still served.  Data of at most 64
variables take the FP64 steps alone, whose results do not depend on the regions: the
orders and measures are those of the full workspace bit for bit; larger ones are
compared by their orders."""
import ctypes

import numpy as np
import pytest

from paper_2403_03772_amd import synth

pytestmark = pytest.mark.gpu

CASES = [([(1000, 10)], 142848, 192768),
         ([(1000, 10), (500, 70)], 860672, 1107200),
         ([(300, 66), (700, 12), (450, 5)], 596736, 776448),
         ([(64, 3)] * 17, 118784, 274944),
         ([(200 + 7 * k, 4 + k) for k in range(40)], 5534976, 6353664),
         ([(90 + k, 2 + k % 9) for k in range(65)], 1154048, 1756160),
         ([(100, 4)] * 200, 2363904, 3887360)]


def _run(lib, jobs, size, learned=None):
    """Status of the batch in a workspace of exactly `size` bytes, its outputs."""
    import torch
    from paper_2403_03772_amd import lib as binding
    L = binding.load()
    arr = (binding._Job * len(jobs))()
    orders, meas, keep = [], [], []
    for a, X in zip(arr, jobs):
        n, d = X.shape
        orders.append(torch.empty(d, dtype=torch.int32, device="cuda"))
        meas.append(torch.full((d - 1, d), float("nan"), dtype=torch.float64, device="cuda"))
        a.X, a.n_rows, a.ldx, a.n, a.d = X.data_ptr(), n, d, n, d
        a.order, a.step_measures = orders[-1].data_ptr(), meas[-1].data_ptr()
    opts, _, _ = binding._new_opts(L, learned=learned, keep=keep)
    if size is None:
        size = int(L.lingam_batch_workspace_size(arr, len(jobs), ctypes.byref(opts)))
    ws = torch.empty(size, dtype=torch.uint8, device="cuda")
    code = L.lingam_batch_causal_order(arr, len(jobs), None, ctypes.byref(opts),
                                       binding._ptr(ws), size, None)
    torch.cuda.synchronize()
    return code, orders, meas


@pytest.mark.parametrize("with_proposer", [False, True])
@pytest.mark.parametrize("sizes,plain,learned", CASES)
def test_previous_size_is_accepted(lib, sizes, plain, learned, with_proposer):
    import torch
    from paper_2403_03772_amd import train_proposer
    jobs = [torch.as_tensor(synth.er_sem(d, n, indeg=min(2.0, (d - 1) / 2), seed=17 + k).X
                            .astype(np.float32)).cuda() for k, (n, d) in enumerate(sizes)]
    cfg = lib.Learned(train_proposer.default_proposer()) if with_proposer else None
    size = learned if with_proposer else plain
    print(f"batch of {len(jobs)} in {size} bytes, proposer={with_proposer}", flush=True)
    code, orders, meas = _run(lib, jobs, size, cfg)
    assert code == 0
    full, want, wanted = _run(lib, jobs, None, cfg)
    assert full == 0
    for o, w, m, v in zip(orders, want, meas, wanted):
        assert torch.equal(o, w)
        if len(o) <= 64:
            assert torch.equal(torch.nan_to_num(m), torch.nan_to_num(v))
    assert _run(lib, jobs, size - 256, cfg)[0] == -4
