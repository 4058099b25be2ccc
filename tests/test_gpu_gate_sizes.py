"""The gate at expert counts that are no multiple of 8 (pieces of the router matrix that reach past a row's end
and, in its last rows, past the matrix's), and for fp32 layers at the edges of their k pieces."""
import numpy as np
import pytest
import torch

import paper_2511_16947_amd as fm
import workloads as wl
from gpu_common import check_router, to64

pytestmark = pytest.mark.gpu

BF16 = [(37, 64, 1, 1), (64, 128, 3, 2), (33, 192, 7, 7), (100, 1088, 9, 3), (1305, 1088, 20, 3), (65, 320, 33, 4),
        (50, 256, 63, 8), (8225, 128, 31, 2), (8200, 128, 61, 3), (64, 64, 65, 8), (129, 704, 97, 4), (40, 4608, 163, 8),
        (70, 128, 255, 6), (48, 192, 300, 8)]
F32 = [(1, 1, 1, 1), (33, 31, 5, 2), (64, 32, 8, 2), (100, 133, 14, 8), (31, 257, 33, 3), (70, 300, 65, 4), (40, 50, 200, 8),
       (256, 1024, 16, 2), (36, 40, 300, 8)]


@pytest.mark.parametrize("case", [c + ("bf16",) for c in BF16] + [c + ("f32",) for c in F32],
                         ids=lambda c: "T%d_d%d_E%d_K%d_%s" % c)
def test_gate_sizes(case):
    T, d, E, K, dtype = case
    cfg = wl.LayerConfig("gate_size", T, d, 64, E, K, 1, dtype, 13, "scaled_z", 0.5)
    inp = wl.make_inputs(cfg, "cuda:0", with_weights=False)
    shape = fm.shape_of(cfg)
    idx = torch.full((T, K), -1, dtype=torch.int32, device="cuda:0")
    w = torch.full((T, K), -1.0, dtype=torch.float32, device="cuda:0")
    for ws in (None, fm.alloc_workspace(shape, fm.WS_TOPK, "cuda:0")):
        idx.fill_(-1)
        w.fill_(-1.0)
        fm.fine_topk(shape, inp.x, inp.w_router, inp.bias, idx, w, ws)
        torch.cuda.synchronize()
        check_router(cfg, inp, idx, w)
        got = idx.cpu().numpy()
        assert got.min() >= 0 and got.max() < E
        assert np.allclose(to64(w).sum(axis=1), 1.0, atol=1e-5)
