"""lingam_bootstrap_regress returns when its counts are complete: the stream has
nothing left to do (orders, rows and workspace may be reused from any stream), and
a call with refused resamples gives the first one's code and counts nothing."""
import pytest

pytestmark = pytest.mark.gpu


def _call(lib, X, rows, orders, counts, stream):
    import torch
    from paper_2403_03772_amd import lib as binding
    L = binding.load()
    (count, n), d = rows.shape, X.shape[1]
    need = int(L.lingam_bootstrap_regress_workspace_size(n, d, count))
    ws = torch.empty(need, dtype=torch.uint8, device="cuda")
    torch.cuda.synchronize()
    return L.lingam_bootstrap_regress(
        binding._ptr(X), X.shape[0], d, binding._ptr(rows), n, d, binding._ptr(orders), count,
        0.0, binding._ptr(counts[0]), binding._ptr(counts[1]), None, binding._ptr(ws), need,
        stream.cuda_stream)


def _inputs(d, n, count):
    import torch
    g = torch.Generator(device="cuda").manual_seed(d)
    X = torch.randn((2 * n, d), generator=g, device="cuda")
    rows = torch.randint(0, 2 * n, (count, n), generator=g, dtype=torch.int32, device="cuda")
    orders = torch.arange(d, dtype=torch.int32, device="cuda").repeat(count, 1)
    counts = [torch.zeros((d, d), dtype=torch.int32, device="cuda") for _ in range(2)]
    return X, rows, orders, counts


def test_nothing_is_left_on_the_stream(lib):
    import torch
    d, count = 48, 400
    X, rows, orders, counts = _inputs(d, 200, count)
    stream = torch.cuda.Stream()
    print(f"case d={d} count={count}", flush=True)
    assert _call(lib, X, rows, orders, counts, stream) == 0
    assert stream.query()
    with torch.cuda.stream(torch.cuda.Stream()):
        below = torch.tril(torch.ones((d, d), dtype=torch.int32, device="cuda"), -1)
        assert torch.equal(counts[0], count * below)


@pytest.mark.parametrize("refused,flat,code", [(517, 300, -2), (255, 256, -1), (599, None, -1),
                                               (None, 0, -2)])
def test_first_refused_resample(lib, refused, flat, code):
    import torch
    X, rows, orders, counts = _inputs(2, 20, 600)
    if refused is not None:
        rows[refused, 3] = X.shape[0]  # a row that is not there: invalid
    if flat is not None:
        rows[flat] = 7                 # one row only: degenerate
    print(f"case refused={refused} flat={flat}", flush=True)
    assert _call(lib, X, rows, orders, counts, torch.cuda.current_stream()) == code
    torch.cuda.synchronize()
    assert int(counts[0].abs().sum()) == 0 and int(counts[1].abs().sum()) == 0
