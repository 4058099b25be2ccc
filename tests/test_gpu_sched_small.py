"""The scheduler in one block (small problems) against the oracle, bit for bit, on both sides of the lines where it
stops: 2048 pairs (4096 with at most 32 experts, each on every rank), 128 experts, 2048 (expert, rank) entries, 64 KB of
tables; every expert on every rank and restricted placements."""
import numpy as np
import pytest
import torch

import paper_2511_16947_amd as fm
import workloads as wl
from gpu_common import check_schedule_against_oracle

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T,E,K,G", [
    (1, 1, 1, 1), (64, 8, 2, 64), (63, 5, 3, 7), (2048, 20, 1, 8), (2049, 20, 1, 3), (512, 128, 4, 4), (513, 128, 4, 3),
    (256, 64, 8, 8), (64, 64, 8, 8), (64, 65, 2, 8), (64, 512, 2, 1), (48, 16, 2, 16), (32, 8, 1, 32),
    (128, 128, 8, 16), (250, 129, 8, 5), (256, 128, 8, 8), (2048, 128, 1, 16), (272, 128, 4, 17),
    (2048, 32, 2, 8), (1025, 20, 4, 5), (1023, 32, 4, 3), (4096, 5, 1, 16), (3073, 8, 1, 7), (1030, 33, 3, 5),
])
@pytest.mark.parametrize("locality", [True, False])
def test_schedule_of_a_small_batch(T, E, K, G, locality):
    shape = fm.Shape(T, 64, 64, E, K, G, fm.FINE_BF16, fm.FLAG_LOCALITY if locality else 0)
    rng = np.random.default_rng(T + E)
    place = np.zeros((E, G), dtype=np.uint8)
    for e in range(E):
        place[e, rng.choice(G, size=int(rng.integers(1, min(G, 3) + 1)), replace=False)] = 1
    idx = wl.random_topk(T, E, K, seed=T + K, skew=1.2)
    idx_d = torch.from_numpy(idx).cuda()
    sb = fm.SchedBuffers(shape, "cuda")
    for p in (None, place):
        for _ in range(2):      # the second run finds the first one's tables
            sb.run(shape, idx_d, None if p is None else torch.from_numpy(p).cuda())
            torch.cuda.synchronize()
            check_schedule_against_oracle(sb, idx, E, G, p, locality)
