"""Data gradients on 128-row tiles of 4 waves (those of matrices past the 8-wave kernels' offsets) and on 128-row and 256-row tiles of 8:
edges of the tiles, contractions of one to a few steps, runs of one tile.  Every element against 64-bit sums,
and all three bit for bit (a row's sums do not depend on the tile it lies in)."""
import pytest
import torch

import paper_2511_16947_amd as fm

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("d,f,rows", [
    (64, 64, [1, 64, 65, 127, 128, 129, 255, 256, 257, 300]),      # dH: 1 step of 64, dXp: 2
    (128, 64, [1, 0, 128, 40]),                                    # 2, 2
    (192, 128, [128, 129, 0, 33, 260]),                            # 3, 4
    (320, 448, [1, 31, 128, 384, 511]),                            # 5, 14; two column tiles, the second ragged
    (64, 832, [128] * 40),                                         # 1, 26: whole tiles only
])
def test_data_gradients_on_tiles_of_both_heights(d, f, rows):
    E, P = len(rows), sum(rows)
    gen = torch.Generator(device=DEV).manual_seed(P + d)

    def normal(*s, std=1.0):
        return (torch.randn(*s, generator=gen, device=DEV) * std).bfloat16()

    x, y, d_out, act = normal(P, d), normal(P, d), normal(P, d), normal(P, 2 * f)
    wg, wu, wd = normal(E, d, f, std=d ** -0.5), normal(E, d, f, std=d ** -0.5), normal(E, f, d, std=f ** -0.5)
    pairs = torch.arange(P, dtype=torch.int32, device=DEV)
    seg_off = torch.tensor([0] + rows, device=DEV).cumsum(0).int()[None].contiguous()
    w = torch.rand(P, 1, generator=gen, device=DEV)
    got = []
    for tile in (1, 2, 3):
        shape = fm.Shape(P, d, f, E, 1, 1, flags=fm.FLAG_LOCALITY | (tile << fm.FLAG_TILE_SHIFT))
        d_x, d_w = torch.full((P, d), 7.0, dtype=torch.bfloat16, device=DEV), torch.full((P, 1), 7.0, device=DEV)
        grads = [torch.full((E, *m), 7.0, device=DEV) for m in ((d, f), (d, f), (f, d))]
        fm.fine_backward(shape, -1, d_out, x, y, act, wg, wu, wd, pairs, pairs, seg_off, w, d_x, d_w, *grads, False,
                         fm.alloc_workspace(shape, fm.WS_BACKWARD))
        got.append([d_x] + grads)
    assert all(torch.equal(a, b) and torch.equal(a, c) for a, b, c in zip(*got))
    r = 0
    for e, n in enumerate(rows):
        if n == 0:
            continue
        dy = (w[r:r + n] * d_out[r:r + n].float()).bfloat16().double()
        dh = dy @ wd[e].double().T
        a, b = act[r:r + n, :f].double(), act[r:r + n, f:].double()
        s = torch.sigmoid(a)
        da, db = dh * b * s * (1 + a * (1 - s)), dh * a * s
        want = da @ wg[e].double().T + db @ wu[e].double().T
        # dH, dA | dB and d_x are rounded to bf16 (2^-9 each); d_x is a sum of 2 f such terms of either sign
        err = (got[0][0][r:r + n].double() - want).abs().max()
        assert err <= 2e-2 * max(1.0, float(want.abs().max())), (e, n, float(err))
        for g, m in zip(got[0][1:], (x[r:r + n].double().T @ da, x[r:r + n].double().T @ db, (a * s * b).T @ dy)):
            assert (g[e].double() - m).abs().max() <= 2e-2 * max(1.0, float(m.abs().max())), (e, n)
        r += n
