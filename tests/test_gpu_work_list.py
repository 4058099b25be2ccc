"""The work list that a call leaves in its workspace: every tile, and which of them are the only ones that read their expert's weights
(those alone are fetched past the caches where the weights would stay in them)."""
import random

import pytest
import torch

import paper_2511_16947_amd as fm

pytestmark = pytest.mark.gpu


def up(n):
    return -(-n // 256) * 256


def few(BM):
    return [[40, 0, 30, 300, BM, 0, 0, 0, 20],      # [rank][expert]
            [7, 0, 0, 10, 0, 50, 0, 1, 0],
            [0, 25, 0, 300, 0, 0, 0, 0, 9],
            [3, 25, 0, 5, 1, 0, BM + 1, 2, 0]]


def many(G, E):
    rng = random.Random(E)
    return lambda BM: [[rng.choice([0] * 20 + [1, 3, BM, BM + 1]) for _ in range(E)] for _ in range(G)]


@pytest.mark.parametrize("tile,BM", [(2, 128), (3, 256)])
@pytest.mark.parametrize("order,rows", [([0, 1, 2, 3], few), ([2, 0, 3, 1], few), (list(range(9)), many(9, 300)),
                                        (list(range(16))[::-1], many(16, 1000))])      # (more segments than LDS holds)
def test_sole_readers(tile, BM, order, rows):
    rows, d, f = rows(BM), 64, 64
    G, E = len(rows), len(rows[0])
    P = sum(map(sum, rows))
    rows[1][5] += -P % G                           # (as many tokens on every rank)
    P += -P % G
    at, seg, runs = 0, [None] * G, []              # runs: expert, first row, end
    for g in order:                                # ranks' rows lie in any order
        seg[g] = [at]
        for n in rows[g]:
            at += n
            seg[g].append(at)
    for g in range(G):
        for e in range(E):
            lo, hi = seg[g][e], seg[g][e + 1]
            if hi == lo:
                continue
            if runs and runs[-1][0] == e and runs[-1][2] == lo:      # goes on where the last rank's last expert ended
                runs[-1][2] = hi
            else:
                runs.append([e, lo, hi])
    want = []
    for e, lo, hi in runs:
        alone = 0 if hi - lo > BM else 2 if sum(r[0] == e for r in runs) == 1 else 1
        want += [(e, r, min(BM, hi - r), alone) for r in range(lo, hi, BM)]
    assert {0, 1, 2} == {w[3] for w in want}
    shape = fm.Shape(P, d, f, E, 1, G, flags=fm.FLAG_LOCALITY | (tile << fm.FLAG_TILE_SHIFT))
    gen = torch.Generator(device="cuda").manual_seed(1)
    x, wg, wu, wd = (torch.randn(*s, generator=gen, device="cuda").bfloat16() for s in ((P, d), (E, d, f), (E, d, f), (E, f, d)))
    ws = fm.alloc_workspace(shape, fm.WS_FFN)
    fm.fine_grouped_ffn(shape, -1, x, wg, wu, wd, torch.tensor(seg, dtype=torch.int32, device="cuda"), torch.empty_like(x), None, ws)
    tiles = up(P * f * 2)                          # behind H: at most P / 32 tiles and one per segment; then the count
    count = tiles + up((P // 32 + E * G + 1) * 16)
    assert int(ws[count:count + 4].view(torch.int32)) == len(want)
    got = ws[tiles:tiles + 16 * len(want)].view(torch.int32).reshape(-1, 4).tolist()
    assert [tuple(t) for t in got] == want
