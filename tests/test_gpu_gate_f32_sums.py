"""The order in which the fp32 gate adds its products, which its distance from 64-bit sums hangs on: pieces of 32 k-values (8 beyond 64
experts) dealt to the waves of a block in turn, a wave's products one after the other, then the waves in order.  Logits of +-1e-3 that are sums of
terms of size 64 are read back from the softmax weights and compared with the same sums made on the host."""
import numpy as np
import pytest
import torch

import paper_2511_16947_amd as fm

pytestmark = pytest.mark.gpu


def in_order(x, w, piece, waves):
    T, d = x.shape
    total = None
    for wave in range(waves):
        acc = np.zeros(T, np.float32)
        for k0 in range(wave * piece, d, waves * piece):
            for j in range(piece // 8):
                for q in range(4):
                    for k in (k0 + 8 * j + q, k0 + 8 * j + 4 + q):      # an MFMA's two
                        if k < d:      # (a product of floats is exact in 64 bits: one rounding, as of an fma)
                            acc = (acc + x[:, k].astype(np.float64) * np.float64(w[k])).astype(np.float32)
        total = acc if total is None else total + acc
    return total.astype(np.float64)


@pytest.mark.parametrize("d,E", [(d, E) for E in (2, 32) for d in (31, 128, 800, 1024, 1025, 1152, 1280, 1536, 1825, 2048, 2175, 3000)]
                         + [(1152, 40), (1152, 100), (1152, 200)])
def test_sums_of_the_f32_gate_in_their_order(d, E):
    T = 40
    rng = np.random.default_rng(d)
    w = rng.standard_normal(d).astype(np.float32)
    x = 64.0 * rng.standard_normal((T, d))
    x = (x - np.outer(x @ w / (w.astype(np.float64) @ w), w)).astype(np.float32)
    w_router, bias = torch.zeros(d, E), torch.full((E,), -100.0)
    w_router[:, 1] = torch.from_numpy(w)
    bias[:2] = 0.0
    shape = fm.Shape(T, d, 64, E, 2, 1, fm.FINE_F32)
    idx = torch.empty(T, 2, dtype=torch.int32, device="cuda")
    out = torch.empty(T, 2, device="cuda")
    fm.fine_topk(shape, torch.from_numpy(x).cuda(), w_router.cuda(), bias.cuda(), idx, out)
    idx, out = idx.cpu().numpy(), out.cpu().numpy().astype(np.float64)
    assert (np.sort(idx, 1) == [0, 1]).all()
    logit = np.log(out[:, 0] / out[:, 1]) * np.where(idx[:, 0] == 1, 1, -1)
    want = in_order(x, w, *((32, 8) if E <= 64 else (8, 4)))
    # the weights' own roundings: exponential, sum and quotient of two weights, 2^-24 to 2^-23 each
    assert np.abs(logit - want).max() <= 1e-6
    if d >= 800:      # the terms' roundings are far above that, so that another order would be seen
        assert np.abs(want - x.astype(np.float64) @ w).max() > 1e-4
