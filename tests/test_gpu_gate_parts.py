"""The gate's logits in two to eight parts of the sum over d, which the selection adds four at a time."""
import pytest
import torch

import paper_2511_16947_amd as fm
import workloads as wl
from gpu_common import check_router

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("E,K", [(66, 1), (128, 17), (250, 8)])
@pytest.mark.parametrize("parts", [2, 3, 4, 5, 7, 8])
def test_selection_adds_every_part(E, K, parts):
    T, d = 45, 512 * parts
    cfg = wl.LayerConfig("gate_parts", T, d, 64, E, K, 1, "bf16", parts, "scaled_z", 0.5)
    inp = wl.make_inputs(cfg, "cuda:0", with_weights=False)
    shape = fm.shape_of(cfg)
    assert fm.fine_workspace_bytes(shape, fm.WS_TOPK) == parts * 64 * (128 if E <= 128 else 256) * 4
    idx = torch.full((T, K), -1, dtype=torch.int32, device="cuda:0")
    w = torch.full((T, K), -1.0, dtype=torch.float32, device="cuda:0")
    fm.fine_topk(shape, inp.x, inp.w_router, inp.bias, idx, w, fm.alloc_workspace(shape, fm.WS_TOPK, "cuda:0"))
    check_router(cfg, inp, idx, w)
    assert (w.double().sum(1) - 1).abs().max() <= 1e-5
