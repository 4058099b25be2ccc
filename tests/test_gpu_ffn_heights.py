"""Expert FFN on lists of 256-row and of 128-row tiles: runs that end in short tiles, and a last round of few tiles, which are
cut into parts of unequal length.  Every element against 64-bit sums."""
import pytest
import torch

import paper_2511_16947_amd as fm

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("tile,d,f,rows", [
    (3, 128, 192, [1, 128, 129, 255, 256, 257, 384, 385, 640]),
    (0, 128, 192, [1, 128, 129, 255, 256, 257, 384, 385, 640]),
    (3, 2112, 2816, [1100, 1290, 200]),      # GEMM 1: 12 x 22 = 264 tiles of 33 k-steps
    (2, 2112, 2816, [600, 650, 100]),        # the same from tiles of 128 rows
    (3, 192, 2112, [256] * 33),              # GEMM 1: 33 x 17 = 561 tiles; GEMM 2: 33 tiles of 33 k-steps
    (3, 1024, 8192, [256] * 3),              # GEMM 1: 192 tiles of 16 k-steps, too many for two parts each; GEMM 2: 12 of 128
    (2, 1024, 5632, [128] * 3),              # the same from tiles of 128 rows: 132 tiles; 12 of 88
])
def test_tiles_of_both_heights(tile, d, f, rows):
    E, P = len(rows), sum(rows)
    shape = fm.Shape(P, d, f, E, 1, 1, flags=fm.FLAG_LOCALITY | (tile << fm.FLAG_TILE_SHIFT))
    gen = torch.Generator(device=DEV).manual_seed(P)

    def normal(*s, std=1.0):
        return (torch.randn(*s, generator=gen, device=DEV) * std).bfloat16()

    x, wg, wu, wd = normal(P, d), normal(E, d, f, std=d ** -0.5), normal(E, d, f, std=d ** -0.5), normal(E, f, d, std=f ** -0.5)
    seg_off = torch.tensor([0] + rows, device=DEV).cumsum(0).int()[None].contiguous()
    y, ws = torch.full((P, d), 7.0, dtype=torch.bfloat16, device=DEV), fm.alloc_workspace(shape, fm.WS_FFN)
    got = []
    for _ in range(2):
        fm.fine_grouped_ffn(shape, -1, x, wg, wu, wd, seg_off, y, None, ws)
        got.append(y.clone())
    assert torch.equal(got[0], got[1])
    r = 0
    for e, n in enumerate(rows):
        xe = x[r:r + n].double()
        h = (torch.nn.functional.silu(xe @ wg[e].double()) * (xe @ wu[e].double())).bfloat16().double()
        want = h @ wd[e].double()
        # H and y are rounded to bf16 (2^-9 each); an H on the other side of a rounding boundary moves y by 2^-8 of one
        # of its f terms.  y has unit scale here.
        assert (y[r:r + n].double() - want).abs().max() <= 2e-2 * max(1.0, float(want.abs().max())), (e, n)
        r += n


@pytest.mark.parametrize("E,G", [(1024, 14), (1024, 15), (200, 9)])
def test_work_list_of_many_segments(E, G):
    """One call over all ranks (segment table in LDS up to 60 KB, 14 x 1025 entries) against one call per rank."""
    gen = torch.Generator().manual_seed(E + G)
    n = torch.randint(0, 4, (G, E), generator=gen) * (torch.rand(G, E, generator=gen) < 0.3)
    n[1:, E // 2] += 70                      # a run of one expert over ranks only where nothing lies between
    n[3] = 0                                 # a rank without rows
    n[3, 5] = 200
    n[4] = 0
    n[4, 5] = 90
    off = torch.zeros(G, E + 1, dtype=torch.int64)
    off[:, 1:] = n.cumsum(1)
    off += (n.sum(1).cumsum(0) - n.sum(1))[:, None]
    P = int(n.sum())
    shape = fm.Shape(P * G, 64, 64, E, 1, G)
    x = torch.randn(P, 64, generator=gen).bfloat16().to(DEV)
    wg, wu, wd = [(torch.randn(E, 64, 64, generator=gen) / 8).bfloat16().to(DEV) for _ in range(3)]
    seg_off, ws = off.int().to(DEV), fm.alloc_workspace(shape, fm.WS_FFN)
    ys = [torch.full((P, 64), 7.0, dtype=torch.bfloat16, device=DEV) for _ in range(2)]
    fm.fine_grouped_ffn(shape, -1, x, wg, wu, wd, seg_off, ys[0], None, ws)
    for rank in range(G):
        fm.fine_grouped_ffn(shape, rank, x, wg, wu, wd, seg_off, ys[1], None, ws)
    assert torch.isfinite(ys[0]).all()
    assert torch.equal(ys[0], ys[1])         # a row's sums do not depend on the tile it lies in
