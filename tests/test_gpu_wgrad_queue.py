"""Weight gradients of experts of very different rows: more tiles than two rounds of the 256 blocks (handed out as blocks become
free), experts without rows among them, and contractions on both sides of the limit from which on they are stored through the caches."""
import pytest
import torch

import paper_2511_16947_amd as fm

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("ranks", ["all", "each"])
@pytest.mark.parametrize("d,f", [(256, 256), (320, 448)])
def test_weight_gradients_handed_out(d, f, ranks):
    rows0 = [1, 0, 384, 385, 0, 448, 64, 65, 2, 700] + [3, 0, 17] * 60
    rows1 = [0, 0, 1, 0, 5, 60, 0, 31, 900, 2] + [0, 0, 40] * 60
    E, G, P0, P = len(rows0), 2, sum(rows0), sum(rows0) + sum(rows1)
    tiles = -(-d // 256) * -(-f // 256) * 3 * E
    assert tiles > 512, tiles
    pad = P % 2                                      # every rank has as many tokens
    rows1[-1] += pad
    P += pad
    gen = torch.Generator(device=DEV).manual_seed(d)

    def normal(*s, std=1.0):
        return (torch.randn(*s, generator=gen, device=DEV) * std).bfloat16()

    x, y, d_out, act = normal(P, d), normal(P, d), normal(P, d), normal(P, 2 * f)
    wg, wu, wd = normal(E, d, f, std=d ** -0.5), normal(E, d, f, std=d ** -0.5), normal(E, f, d, std=f ** -0.5)
    pairs = torch.arange(P, dtype=torch.int32, device=DEV)
    seg_off = torch.stack([torch.tensor([0] + rows0).cumsum(0), P0 + torch.tensor([0] + rows1).cumsum(0)]).int().to(DEV).contiguous()
    w = torch.rand(P, 1, generator=gen, device=DEV)
    shape = fm.Shape(P, d, f, E, 1, G, flags=fm.FLAG_LOCALITY)
    d_x, d_w = torch.empty(P, d, dtype=torch.bfloat16, device=DEV), torch.empty(P, 1, device=DEV)
    grads = [torch.full((E, *m), 7.0, device=DEV) for m in ((d, f), (d, f), (f, d))]
    ws = fm.alloc_workspace(shape, fm.WS_BACKWARD)

    def run(rank, accumulate):
        fm.fine_backward(shape, rank, d_out, x, y, act, wg, wu, wd, pairs, pairs, seg_off, w, d_x, d_w, *grads, accumulate, ws)

    if ranks == "all":
        run(-1, False)
        once = [g.clone() for g in grads]
        run(-1, True)
    else:
        run(0, False)
        run(1, True)
        once = [g.clone() for g in grads]
        run(0, True)
        run(1, True)
    assert sum(rows0[e] + rows1[e] == 0 for e in range(E)) > 60
    for e in range(E):
        r = torch.cat([torch.arange(int(seg_off[g, e]), int(seg_off[g, e + 1])) for g in range(G)]).to(DEV)
        dy = (w[r] * d_out[r].float()).bfloat16().double()
        dh = dy @ wd[e].double().T
        a, b = act[r, :f].double(), act[r, f:].double()
        s = torch.sigmoid(a)
        da, db = dh * b * s * (1 + a * (1 - s)), dh * a * s
        for g1, g2, m in zip(once, grads, (x[r].double().T @ da, x[r].double().T @ db, (a * s * b).T @ dy)):
            # dH, dA | dB and H are rounded to bf16 (2^-9 each) before the sum over the rows
            tol = 2e-2 * max(1.0, float(m.abs().max()))
            assert (g1[e].double() - m).abs().max() <= tol, e
            assert (g2[e].double() - 2 * m).abs().max() <= 2 * tol, e
