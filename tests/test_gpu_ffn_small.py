"""Expert FFN of small launches (k split over the waves of a block) and the work list of runs of segments: every
element against 64-bit sums, at the edges of row tiles, column tiles and k ranges."""
import pytest
import torch

import paper_2511_16947_amd as fm

DEV = "cuda:0"
pytestmark = pytest.mark.gpu


def _reference(x, wg, wu, wd):
    h = (torch.nn.functional.silu(x.double() @ wg.double()) * (x.double() @ wu.double())).bfloat16().double()
    return h, h @ wd.double()


# segments: rows of (rank, expert); the last expert of a rank and the first non-empty one of the next form one run
@pytest.mark.parametrize("tile", [0, 1, 2, 3])
@pytest.mark.parametrize("d,f,seg", [
    (64, 64, [[1, 0, 31], [0, 0, 2]]),                     # one k-step: three of the four waves have none
    (128, 192, [[32, 33, 0], [0, 63, 64]]),                # half a column tile at the end; tiles of 32 and 33 rows
    (192, 320, [[65, 0, 1], [0, 0, 127], [0, 0, 64]]),     # a run over three ranks: 192 rows of expert 2
    (64, 64, [[1] * 190 + [0] * 65 + [70], [2] * 256]),    # 256 experts: the most whose work list a wave keeps in registers
    (64, 64, [[1] * 190 + [0] * 66 + [70], [2] * 257]),
    (576, 832, [[0, 130, 0], [5, 0, 0], [0, 0, 0]]),       # odd numbers of k-steps; empty ranks
], ids=lambda v: None if isinstance(v, int) else "%dx%d" % (len(v), len(v[0])))
def test_small_launch_every_element(d, f, seg, tile):
    G, E = len(seg), len(seg[0])
    P = sum(map(sum, seg))
    shape = fm.Shape(P * G, d, f, E, 1, G, flags=fm.FLAG_LOCALITY | (tile << fm.FLAG_TILE_SHIFT))
    off, r = [], 0
    for row in seg:
        for n in row:
            off.append(r)
            r += n
        off.append(r)
    gen = torch.Generator().manual_seed(d + f)

    def normal(*s, std=1.0):
        return (torch.randn(*s, generator=gen) * std).bfloat16().to(DEV)

    x, wg, wu, wd = normal(P, d), normal(E, d, f, std=d ** -0.5), normal(E, d, f, std=d ** -0.5), normal(E, f, d, std=f ** -0.5)
    seg_off = torch.tensor(off, dtype=torch.int32, device=DEV)
    ws = fm.alloc_workspace(shape, fm.WS_FFN)
    act = torch.full((P, 2 * f), 7.0, dtype=torch.bfloat16, device=DEV)
    for ranks in ([-1], range(G)):
        y = torch.full((P, d), 7.0, dtype=torch.bfloat16, device=DEV)
        for rank in ranks:
            fm.fine_grouped_ffn(shape, rank, x, wg, wu, wd, seg_off, y, act, ws)
        r = 0
        for row in seg:
            for e, n in enumerate(row):
                _, want = _reference(x[r:r + n], wg[e], wu[e], wd[e])
                if n:
                    # H and y are rounded to bf16 (2^-9 each); an H that falls on the other side of a rounding
                    # boundary moves y by 2^-8 of one of its f terms.  y has unit scale here.
                    assert (y[r:r + n].double() - want).abs().max() <= 2e-2 * max(1.0, float(want.abs().max())), (r, e, n)
                    a = x[r:r + n].double() @ wg[e].double()
                    assert (act[r:r + n, :f].double() - a).abs().max() <= 2 ** -8 * float(a.abs().max())
                r += n


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("tile", [0, 1, 2, 3])
@pytest.mark.parametrize("d,f,seg,start", [
    (64, 128, [[70, 3], [40, 0], [0, 65]], [300, 3, 100]),                # gaps, ranks in another order
    (128, 64, [[0, 130, 1], [64, 0, 5], [0, 0, 33], [0, 0, 31]], [270, 0, 200, 233]),      # ranks 2 and 3: one run
    (64, 64, [[1] * 600, [2] * 599 + [0]], [1300, 10]),                     # 1200 segments: several per thread
], ids=lambda v: None if isinstance(v, int) else str(len(v)))
def test_ranks_rows_in_any_order(d, f, seg, start, tile, dtype):
    """The rows of the ranks lie anywhere in the buffers, with rows between them that belong to nobody."""
    if dtype == "f32" and tile != 0:
        pytest.skip("tile variants are for the bf16 kernels")
    dt = torch.float32 if dtype == "f32" else torch.bfloat16
    G, E = len(seg), len(seg[0])
    off, where = [], []
    for row, r in zip(seg, start):
        for e, n in enumerate(row):
            off.append(r)
            where.append((r, e, n))
            r += n
        off.append(r)
    P = max(off) + 7
    shape = fm.Shape(P * G, d, f, E, 1, G, fm.FINE_F32 if dtype == "f32" else fm.FINE_BF16,
                     fm.FLAG_LOCALITY | (tile << fm.FLAG_TILE_SHIFT))
    gen = torch.Generator().manual_seed(d + f)

    def normal(*s, std=1.0):
        return (torch.randn(*s, generator=gen) * std).to(DEV, dt)

    x, wg, wu, wd = normal(P, d), normal(E, d, f, std=d ** -0.5), normal(E, d, f, std=d ** -0.5), normal(E, f, d, std=f ** -0.5)
    seg_off = torch.tensor(off, dtype=torch.int32, device=DEV)
    ws = fm.alloc_workspace(shape, fm.WS_FFN)
    for ranks in ([-1], range(G)):
        y = torch.full((P, d), 7.0, dtype=dt, device=DEV)
        for rank in ranks:
            fm.fine_grouped_ffn(shape, rank, x, wg, wu, wd, seg_off, y, None, ws)
        left = torch.ones(P, dtype=torch.bool, device=DEV)
        for r, e, n in where:
            if n:
                _, want = _reference(x[r:r + n], wg[e], wu[e], wd[e])      # (H rounded to bf16: see above for the bound)
                assert (y[r:r + n].double() - want).abs().max() <= 2e-2 * max(1.0, float(want.abs().max())), (r, e, n)
                left[r:r + n] = False
        assert (y[left] == 7.0).all()
