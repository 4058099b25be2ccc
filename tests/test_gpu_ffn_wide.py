"""Expert FFN at the widths where byte offsets outgrow 32 bits: a whole weight matrix of 4 GiB, the widest rows that each
kernel takes, and one step beyond the widest (which goes to the kernel with 64-bit addresses)."""
import pytest
import torch

import paper_2511_16947_amd as fm

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _normal(seed, *shape, std=1.0):
    gen = torch.Generator(device=DEV).manual_seed(seed)
    t = torch.empty(shape, dtype=torch.bfloat16, device=DEV)
    return t.normal_(0.0, std, generator=gen)


def _setup(T, d, f, tile=0):
    shape = fm.Shape(T, d, f, 1, 1, 1, flags=fm.FLAG_LOCALITY | (tile << fm.FLAG_TILE_SHIFT))
    w = _normal(1, 1, d, f, std=d ** -0.5), _normal(2, 1, d, f, std=d ** -0.5), _normal(3, 1, f, d, std=f ** -0.5)
    return shape, _normal(4, T, d), w, torch.tensor([0, T], dtype=torch.int32, device=DEV)


def _forward(shape, x, w, seg):
    y = torch.full((shape.T, shape.d), 7.0, dtype=torch.bfloat16, device=DEV)
    fm.fine_grouped_ffn(shape, -1, x, *w, seg, y, None, fm.alloc_workspace(shape, fm.WS_FFN))
    return y


def _close(got, want):
    # sums of unit scale with terms rounded to bf16 (2^-9 each): a few 1e-3 of the scale; a part that was left out or
    # read from elsewhere changes values by their own size
    assert (got.float() - want).abs().max() <= 3e-2 * float(want.abs().max())
    assert (got.float() - want).norm() <= 1e-2 * want.norm()


@pytest.mark.parametrize("T,d,f,tile", [
    (40, 1 << 16, 1 << 15, 0), (768, 1 << 16, 1 << 15, 0), (100, 1 << 15, 1 << 16, 3),       # d f = 2^31
    (256, 1 << 22, 448, 3), (255, 448, 1 << 22, 3), (100, 1 << 22, 448, 2),                   # widest on 8 waves
    (70, 1 << 24, 64, 0), (60, 64, 1 << 24, 0),                                               # widest with k split over waves
    (3, (1 << 24) + 64, 64, 0),
])
def test_wide_forward(T, d, f, tile):
    shape, x, w, seg = _setup(T, d, f, tile)
    print("wide forward", T, d, f, tile, flush=True)
    y = _forward(shape, x, w, seg)
    a, b = x.float() @ w[0][0].float(), x.float() @ w[1][0].float()
    h = (torch.nn.functional.silu(a) * b).bfloat16().float()
    del a, b
    _close(y, h @ w[2][0].float())


def test_wide_backward():
    T, d, f = 768, 1 << 16, 1 << 15
    shape, x, w, seg = _setup(T, d, f)
    y = _forward(shape, x, w, seg)
    rows = torch.arange(T, dtype=torch.int32, device=DEV)
    d_out, one = _normal(5, T, d), torch.ones(T, 1, device=DEV)
    d_x, d_tw = torch.empty_like(x), torch.empty(T, 1, device=DEV)
    d_w = [torch.empty(m.shape, device=DEV) for m in w]
    fm.fine_backward(shape, -1, d_out, x, y, None, *w, rows, rows, seg, one, d_x, d_tw, *d_w, False,
                     fm.alloc_workspace(shape, fm.WS_BACKWARD))
    a, b = x.float() @ w[0][0].float(), x.float() @ w[1][0].float()
    dh = d_out.float() @ w[2][0].float().T
    s = torch.sigmoid(a)
    da, db, h = dh * b * s * (1 + a * (1 - s)), dh * a * s, a * s * b
    del dh, s, a, b
    _close(d_x, da @ w[0][0].float().T + db @ w[1][0].float().T)
    for got, rows_in, cols in ((d_w[0][0], x, da), (d_w[1][0], x, db), (d_w[2][0], h, d_out)):
        for part in (slice(0, 4096), slice(-4096, None)):
            _close(got[part], rows_in.float().T[part] @ cols.float())
