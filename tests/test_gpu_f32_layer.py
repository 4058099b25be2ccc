"""fp32 layers on the fp32 matrix cores: every element of y_perm and act_save against the fp64 oracle at the
edges of the kernels' tiles (64 rows, 64 or 128 columns; small launches 32 rows, 32 columns; 32 k-values, which small
launches deal to four waves; 16-byte and 4-byte operand loads)."""
import numpy as np
import pytest
import torch

import paper_2511_16947_amd as fm
import workloads as wl
from gpu_common import GpuLayer, max_rel_err, to64

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d,f", [(128, 256), (4, 4), (1, 1), (33, 65), (63, 31), (132, 68), (133, 858), (256, 132)])
@pytest.mark.parametrize("T,E,K,G", [(64, 4, 2, 2), (130, 3, 3, 1), (260, 8, 2, 4), (2200, 3, 3, 1), (40, 40, 1, 4)])
def test_f32_ffn_every_element(d, f, T, E, K, G):
    cfg = wl.scaled(wl.CONFIGS["cfg1_tiny_f32"], T=T, d=d, f=f, E=E, K=K, G=G, seed=11)
    inp = wl.make_inputs(cfg, "cuda:0")
    layer = GpuLayer(cfg, inp)
    layer.act_save = torch.full((layer.shape.P, 2 * f), float("nan"), device="cuda")
    for per_rank in (True, False):
        layer.y_perm.fill_(float("nan"))
        layer.forward(per_rank=per_rank)
        idx = layer.topk_idx.cpu().numpy()
        pair_of_row = layer.sb.pair_of_row.cpu().numpy()
        x, y, act = to64(inp.x), to64(layer.y_perm), to64(layer.act_save)
        want, want_act = np.empty_like(y), np.empty_like(act)
        for e in range(E):
            rows = np.nonzero(idx.reshape(-1)[pair_of_row] == e)[0]
            X = x[pair_of_row[rows] // K]
            A, B = X @ to64(inp.w_gate[e]), X @ to64(inp.w_up[e])
            want_act[rows] = np.concatenate([A, B], 1)
            want[rows] = (A / (1 + np.exp(-A)) * B) @ to64(inp.w_down[e])
        # 1e-5: the library's bound for fp32 outputs (sums of up to 858 products: eps sqrt(858) = 1.7e-6)
        assert max_rel_err(act, want_act) <= 1e-5
        assert max_rel_err(y, want) <= 1e-5


@pytest.mark.parametrize("rows", [[5, 0, 40], [8000, 0, 6500]])      # launches of 32-row and of 64-row tiles
@pytest.mark.parametrize("d,f", [(1, 33), (33, 63), (63, 1), (65, 133), (4, 132), (36, 4)])
def test_f32_ffn_reads_no_weights_of_others(d, f, rows):
    """k-ranges that end inside a 32-value step: what follows an expert's weights (an expert without rows, and behind the
    last expert the rest of the buffer) is NaN, which no factor of zero would hide."""
    E, P = len(rows), sum(rows)
    shape = fm.Shape(P, d, f, E, 1, 1, fm.FINE_F32)
    gen = torch.Generator(device="cuda").manual_seed(d * f)
    x = torch.randn(P, d, generator=gen, device="cuda")
    weights = []
    for n, m in ((d, f), (d, f), (f, d)):
        buf = torch.full(((E + 40) * n * m + 64,), float("nan"), device="cuda")
        w = buf[:E * n * m].view(E, n, m)
        for e in range(E):
            if rows[e]:
                w[e] = torch.randn(n, m, generator=gen, device="cuda") * n ** -0.5
        weights.append(w)
    seg_off = torch.tensor([0] + rows, device="cuda").cumsum(0).int()[None].contiguous()
    y = torch.full((P, d), float("nan"), device="cuda")
    fm.fine_grouped_ffn(shape, -1, x, *weights, seg_off, y, None, fm.alloc_workspace(shape, fm.WS_FFN))
    r = 0
    for e, n in enumerate(rows):
        xe, (wg, wu, wd) = x[r:r + n].double(), [w[e].double() for w in weights]
        want = (torch.nn.functional.silu(xe @ wg) * (xe @ wu)) @ wd
        if n:      # 1e-5: as above
            assert max_rel_err(to64(y[r:r + n]), to64(want)) <= 1e-5
        r += n


def test_fewer_rows_take_no_longer():
    """Rows that are no multiple of 16 bytes: 900 rows on 3 experts (205 64-row tiles) against 1000 (224).  Measured 1.00 times as
    long; 1.38 times where the smaller launch takes the tiles of small launches."""
    d, f, E = 700, 777, 3
    gen = torch.Generator(device="cuda").manual_seed(1)
    w = [torch.randn(E, n, m, generator=gen, device="cuda") * n ** -0.5 for n, m in ((d, f), (d, f), (f, d))]

    def us(P):
        shape = fm.Shape(P, d, f, E, 1, 1, fm.FINE_F32)
        x, y = torch.randn(P, d, generator=gen, device="cuda"), torch.empty(P, d, device="cuda")
        seg_off = torch.tensor([[0, P // 3, 2 * P // 3, P]], dtype=torch.int32, device="cuda")
        ws, t = fm.alloc_workspace(shape, fm.WS_FFN), []
        for _ in range(9):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            for _ in range(10):
                fm.fine_grouped_ffn(shape, 0, x, *w, seg_off, y, None, ws)
            b.record()
            b.synchronize()
            t.append(a.elapsed_time(b) * 100)
        return float(np.median(t))

    us(1000)      # (clocks)
    assert us(900) < 1.12 * us(1000)


@pytest.mark.parametrize("P,d,f,E,G", [(2048, 768, 768, 16, 8), (1300, 333, 777, 13, 5)])
def test_rank_calls_against_the_call_for_all_ranks(P, d, f, E, G):
    """Ranks of few tiles take the kernel that adds k in four ranges, the call for all of them the one that adds it in one chain:
    equal up to fp32 summation order."""
    shape = fm.Shape(P, d, f, E, 1, G, fm.FINE_F32)
    gen = torch.Generator(device="cuda").manual_seed(P)
    x = torch.randn(P, d, generator=gen, device="cuda")
    w = [torch.randn(E, n, m, generator=gen, device="cuda") * n ** -0.5 for n, m in ((d, f), (d, f), (f, d))]
    start = torch.linspace(0, P, E + 1, device="cuda").int()
    seg_off = torch.stack([start.clamp(P // G * g, P // G * (g + 1)) for g in range(G)]).contiguous()
    ws, ys, acts = fm.alloc_workspace(shape, fm.WS_FFN), [], []
    for ranks in ((-1,), range(G)):
        ys.append(torch.full((P, d), float("nan"), device="cuda"))
        acts.append(torch.full((P, 2 * f), float("nan"), device="cuda"))
        for rank in ranks:
            fm.fine_grouped_ffn(shape, rank, x, *w, seg_off, ys[-1], acts[-1], ws)
    # sums of n products in two orders: 2 eps sqrt(n) of their norm = 3.3e-6 for n = 768 (measured 1.3e-6)
    assert max_rel_err(to64(acts[1]), to64(acts[0])) <= 3.3e-6
    # and what the difference of H makes in y adds to that (measured 1.4e-6)
    assert max_rel_err(to64(ys[1]), to64(ys[0])) <= 1e-5
