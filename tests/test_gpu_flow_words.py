"""The replica-load solver keeps sets of experts in words of 64: list lengths around one, two and four words and beyond,
sets of ranks in 32 and in 64 bits, cold and from garbage."""
import numpy as np
import pytest
import torch

import paper_2511_16947_amd as fm
import workloads as wl
from gpu_common import check_schedule_against_oracle

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("E,G,T", [(64, 8, 256), (65, 8, 256), (128, 5, 250), (129, 32, 320), (257, 4, 400), (300, 33, 330)])
def test_lists_of_all_lengths(E, G, T):
    rng = np.random.default_rng(E)
    idx = wl.random_topk(T, E, 2, seed=E, skew=0.7)
    place = np.zeros((E, G), np.uint8)
    for e in range(E):                      # two or three replicas each: every expert is on the list
        place[e, rng.choice(G, rng.integers(2, 4), replace=False)] = 1
    shape = fm.Shape(T, 64, 64, E, 2, G)
    sb = fm.SchedBuffers(shape, "cuda")
    for warm in (False, True):
        sb.x_eg.copy_(torch.from_numpy(rng.integers(-2**31, 2**31 - 1, (E, G)).astype(np.int32)))
        sb.run(shape, torch.from_numpy(idx).cuda(), torch.from_numpy(place).cuda(), warm=warm)
        torch.cuda.synchronize()
        check_schedule_against_oracle(sb, idx, E, G, place, True)
