"""The gate where fewer than K logits are ordinary numbers: experts masked with -inf or the lowest float, NaN and +inf
logits, ties.  The K picks of a token are distinct, in descending order of the logits (equal ones: lower index first;
NaN below everything), whichever kernel takes the call."""
import numpy as np
import pytest
import torch

import paper_2511_16947_amd as fm
from oracle import router

pytestmark = pytest.mark.gpu

CASES = [
    # T, d, E, K, dtype
    (70, 64, 5, 3, "bf16"), (33, 128, 8, 8, "bf16"), (65, 64, 20, 6, "bf16"), (40, 64, 64, 32, "bf16"),
    (70, 64, 96, 8, "bf16"), (40, 128, 255, 32, "bf16"),
    (40, 4608, 163, 8, "bf16"), (40, 4608, 256, 32, "bf16"),      # with the workspace: blocks share a token tile
    (48, 64, 300, 8, "bf16"), (48, 64, 1024, 32, "bf16"),
    (70, 31, 5, 3, "f32"), (33, 64, 33, 8, "f32"), (40, 50, 70, 32, "f32"), (65, 40, 200, 8, "f32"), (36, 40, 300, 32, "f32"),
]


def _biases(E, K, rng):
    keep = max(1, min(K, E) // 2)
    for mask in (-np.inf, np.finfo(np.float32).min):
        b = np.full(E, mask, np.float32)
        b[rng.choice(E, keep, replace=False)] = 0.0
        yield b
        yield np.full(E, mask, np.float32)
    b = np.zeros(E, np.float32)
    b[rng.random(E) < 0.5] = np.nan
    yield b
    b = np.full(E, -np.inf, np.float32)
    b[rng.choice(E, keep, replace=False)] = np.nan
    b[rng.integers(E)] = np.inf
    yield b
    yield np.zeros(E, np.float32)                                  # ties only


@pytest.mark.parametrize("case", CASES, ids=lambda c: "T%d_d%d_E%d_K%d_%s" % c)
def test_masked_logits(case):
    T, d, E, K, dtype = case
    rng = np.random.default_rng(E + K)
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32
    shape = fm.Shape(T, d, 64, E, K, 1, fm.FINE_BF16 if dtype == "bf16" else fm.FINE_F32)
    # one non-zero per token and small whole weights: every logit is exact in any order of summation, and many are equal
    x = np.zeros((T, d), np.float32)
    x[np.arange(T), rng.integers(0, d, T)] = 1.0
    w = rng.integers(-5, 6, (d, E)).astype(np.float32)
    x_d, w_d = torch.from_numpy(x).to("cuda", dt), torch.from_numpy(w).to("cuda", dt)
    for n, bias in enumerate(_biases(E, K, rng)):
        logits = ((x @ w) + bias[None, :]).astype(np.float32)
        with np.errstate(invalid="ignore"):
            want_idx, want_w = router.topk_from_logits_fast(logits, K)
        for ws in (None, fm.alloc_workspace(shape, fm.WS_TOPK, "cuda")):
            idx = torch.full((T, K), -1, dtype=torch.int32, device="cuda")
            tw = torch.full((T, K), -1.0, dtype=torch.float32, device="cuda")
            fm.fine_topk(shape, x_d, w_d, torch.from_numpy(bias).cuda(), idx, tw, ws)
            got = idx.cpu().numpy()
            assert (np.diff(np.sort(got, axis=1), axis=1) > 0).all(), (n, "an expert picked twice")
            assert np.array_equal(got, want_idx), n
            # weights: NaN where the definition gives NaN (all logits -inf, a NaN or +inf among the picks), else a
            # softmax of at most 32 terms in fp32: a few ulps of exp, sum and quotient
            assert np.allclose(tw.cpu().numpy(), want_w, rtol=1e-5, atol=1e-7, equal_nan=True), n
