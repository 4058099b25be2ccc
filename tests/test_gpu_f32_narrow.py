"""Small fp32 launches on 32 x 16 tiles, and those just past them on 32 x 32: edges of the 16 columns, of 32 rows and of the 32-value
k pieces dealt to four waves, 16-byte and 4-byte operand loads.  Every element against 64-bit sums."""
import pytest
import torch

import paper_2511_16947_amd as fm

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d,f,rows,narrow", [
    (4, 4, [1], True), (1, 17, [16, 0, 33], True), (15, 16, [17], True), (16, 15, [31, 1], True), (36, 28, [32, 15, 65], True),
    (128, 256, [128], True), (129, 257, [40, 1, 0, 24], True), (1024, 1024, [64], True), (140, 852, [16, 47], True),
    (256, 512, [200, 28, 156], False), (128, 256, [500, 33, 235], False), (300, 301, [300, 156], False),
])
def test_small_f32_launches_every_element(d, f, rows, narrow):
    E, P = len(rows), sum(rows)
    tiles32 = (P / 32 + E) * (-(-d // 32) + -(-f // 32)) / 2      # the dispatch's expectation, and its limit
    assert (tiles32 < 160) == narrow, tiles32
    shape = fm.Shape(P, d, f, E, 1, 1, fm.FINE_F32)
    gen = torch.Generator(device="cuda").manual_seed(d + f)
    x = torch.randn(P, d, generator=gen, device="cuda")
    wg, wu, wd = (torch.randn(E, n, m, generator=gen, device="cuda") * n ** -0.5 for n, m in ((d, f), (d, f), (f, d)))
    seg_off = torch.tensor([0] + rows, device="cuda").cumsum(0).int()[None].contiguous()
    y, act = torch.full((P, d), float("nan"), device="cuda"), torch.full((P, 2 * f), float("nan"), device="cuda")
    fm.fine_grouped_ffn(shape, 0, x, wg, wu, wd, seg_off, y, act, fm.alloc_workspace(shape, fm.WS_FFN))
    r = 0
    for e, n in enumerate(rows):
        if n == 0:
            continue
        xe = x[r:r + n].double()
        a, b = xe @ wg[e].double(), xe @ wu[e].double()
        want = (torch.nn.functional.silu(a) * b) @ wd[e].double()
        # 1e-5 of the largest: the library's bound for fp32 outputs (sums of up to 1024 products: eps sqrt(1024) = 1.9e-6)
        for got, m in ((act[r:r + n, :f], a), (act[r:r + n, f:], b), (y[r:r + n], want)):
            assert (got.double() - m).abs().max() <= 1e-5 * max(1.0, float(m.abs().max())), (e, n)
        r += n
