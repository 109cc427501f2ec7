"""Gradient of the proposer at the edges of the backward pass's groups of 16 rows
and of its partial gradients (one for every 64 rows, at most 512, eight at a
time in the reduction): against the oracle's FP64 backward pass at the same
BF16-rounded weights and inputs.

The kernel rounds dh2, dh1 and the first layer to BF16 where the oracle keeps
them: three relative errors of at most 2^-9 a product, 6e-3 of a gradient's
norm; the bound is 1e-2.
"""
import numpy as np
import pytest

from oracle import proposer as OP

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("rows,lists", [(2, 1), (15, 2), (16, 1), (17, 3), (64, 5), (65, 2),
                                        (1023, 9), (8193, 40), (32785, 70)])
def test_grad_row_edges(lib, rows, lists):
    import torch
    print(f"case rows={rows} lists={lists}", flush=True)
    rng = np.random.default_rng(rows)
    norm = np.concatenate([rng.normal(scale=0.3, size=16), rng.uniform(0.5, 2.0, 16)])
    prop = np.concatenate([norm, OP.init_params(rows)])
    cuts = np.sort(rng.choice(np.arange(1, rows), lists - 1, replace=False))
    offs = np.concatenate([[0], cuts, [rows]]).astype(np.int64)
    tg = np.array([rng.integers(a, b) for a, b in zip(offs[:-1], offs[1:])], dtype=np.int64)
    F = rng.normal(size=(rows, 16)).astype(np.float32)

    def t(a, dtype=np.float32):
        return torch.as_tensor(np.ascontiguousarray(a, dtype=dtype)).cuda()

    loss, grad, _, _ = lib.proposer_grad(t(prop), t(F), t(offs, np.int64), t(tg, np.int64))
    g = grad.cpu().numpy().astype(np.float64)
    p = OP.unpack(prop[32:].copy())
    for k in ("W1", "W2", "w3"):
        p[k] = OP.bf16(p[k])
    flat = OP.pack(p)
    s, cache = OP.forward(flat, OP.bf16(OP.normalize(F, prop[:32])), emulate_bf16=True)
    ref_loss, ds = OP.listwise_ce(s.astype(np.float32).astype(np.float64), offs, tg)
    ref = OP.backward(flat, cache, ds)
    assert abs(float(loss.item()) - ref_loss) <= 1e-4 * max(1.0, abs(ref_loss))
    o = 0
    for name, shape in OP.SHAPES:
        k = int(np.prod(shape))
        a, b = g[o:o + k], ref[o:o + k]
        o += k
        if name == "b3":
            assert abs(a[0]) <= 1e-6  # softmax minus a distribution sums to 0
        else:
            assert np.linalg.norm(a - b) <= 1e-2 * max(np.linalg.norm(b), 1e-12), name
