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
