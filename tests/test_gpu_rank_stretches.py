"""The ordered pass of a rank compaction, in which every wavefront walks a stretch of its head: lengths
around the edges of a round, of four rounds and of a stretch, ties across the stretches, heads that lose
nothing or all, up to 1024 heads and above, rows that are kept in LDS and rows that are not."""
import numpy as np
import pytest
import torch

from oracle import kvc_oracle as O
from helpers import oracle_state
from test_gpu_sliced_moves import compare
from test_gpu_window_paths import make

pytestmark = pytest.mark.gpu
LENGTHS = [1, 64, 1023, 1024, 1025, 63, 4095, 4097, 65, 9000, 0, 2048]


@pytest.mark.parametrize("ties", [True, False])
@pytest.mark.parametrize("Lyr,Hk,b,room", [(2, 3, 16, 0), (2, 3, 2, 0), (2, 3, 16, 17000), (41, 25, 16, 0), (41, 25, 16, 17000)])
def test_rank_rounds(Lyr, Hk, b, room, ties):
    from paper_2410_00161_amd.session import KvcSession
    S, G = (2, 12) if Lyr == 2 else (1, 1025)
    lengths = LENGTHS if G == 12 else [LENGTHS[g % 12] if g % 41 < 12 else g % 50 for g in range(G)]
    shape, cache, _ = make(S, Lyr, Hk, 1, 8, b, lengths, "bf16", room)
    if ties:
        cache.metric = torch.randint(0, 3, cache.metric.shape, generator=torch.Generator().manual_seed(5)).float()
    st = oracle_state(cache)
    sess = KvcSession(cache)
    for frac in (0.3, 0.8):
        nb = (-(-st.lens() // b)).reshape(S, -1).sum(1)
        budget = (nb * frac).astype(np.int64)
        _, masks, _ = O.rank_schedule(st, budget, None, 1)
        sess.evict_rank_select(torch.from_numpy(budget).int(), protect_tail_blocks=1)
        compare(sess, st, sess.compact_rank(), O.compact_slots(st, masks))
