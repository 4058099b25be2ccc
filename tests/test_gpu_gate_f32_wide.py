"""The gate of fp32 layers with pieces of 128 k-values: widths around multiples of the eight waves' pieces, ragged tails."""
import pytest
import torch

import paper_2511_16947_amd as fm
import workloads as wl
from gpu_common import check_router

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T,E,K", [(1, 1, 1), (33, 8, 2), (70, 32, 5)])
@pytest.mark.parametrize("d", [1023, 1024, 1025, 1151, 1153, 2048, 2175])
def test_wide_f32_gate(T, d, E, K):
    cfg = wl.LayerConfig("gate_f32_wide", T, d, 64, E, K, 1, "f32", d, "scaled_z", 0.5)
    inp = wl.make_inputs(cfg, "cuda:0", with_weights=False)
    idx = torch.full((T, K), -1, dtype=torch.int32, device="cuda:0")
    w = torch.full((T, K), -1.0, dtype=torch.float32, device="cuda:0")
    fm.fine_topk(fm.shape_of(cfg), inp.x, inp.w_router, inp.bias, idx, w, None)
    check_router(cfg, inp, idx, w)
    assert (w.double().sum(1) - 1).abs().max() <= 1e-5
