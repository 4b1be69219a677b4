"""Thresholds of the rank schedule picked by the launches that use them (up to 1024 heads) and, in a pool
too small for the histograms that takes, by launches of their own: several segments, empty ones, budgets
of nothing, of more than there is and below zero."""
import numpy as np
import pytest
import torch

from oracle import kvc_oracle as O
from paper_2410_00161_amd import binding as B
from helpers import oracle_state
from test_gpu_sliced_moves import compare
from test_gpu_window_paths import make

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("Lyr,Hk,b,longest,room", [(1, 2, 1, 30, 0), (1, 2, 4, 900, 0), (1, 2, 16, 900, 17000), (32, 5, 4, 60, 0)])
@pytest.mark.parametrize("ties", [False, True])
def test_segments(Lyr, Hk, b, longest, room, ties):
    from paper_2410_00161_amd.session import KvcSession
    S, off = 6, [0, 0, 1, 4, 4, 6]
    G = S * Lyr * Hk
    lengths = [int(x) for x in torch.randint(0, longest, (G,), generator=torch.Generator().manual_seed(3))]
    lengths[1] = 0
    shape, cache, _ = make(S, Lyr, Hk, 1, 8, b, lengths, "bf16", room)
    small = shape.num_blocks * b < 3 * 256 * 5
    assert G <= 1024 and small == (longest == 30)
    if ties:
        cache.metric = torch.randint(0, 3, cache.metric.shape, generator=torch.Generator().manual_seed(5)).float()
    st = oracle_state(cache)
    sess = KvcSession(cache)
    seg = torch.tensor(off, dtype=torch.int32)
    for share in ((0.0, 0.4, 0.0, 0.0, 0.7), (0.0, 9.0, 0.5, 0.0, 0.0)):
        nb = (-(-st.lens() // b)).reshape(S, -1).sum(1)
        budget = np.array([int(nb[a:e].sum() * f) for a, e, f in zip(off, off[1:], share)], dtype=np.int64)
        rows, masks, sel = O.rank_schedule(st, budget, np.array(off), 1)
        wrong = torch.from_numpy(budget).int()
        wrong[3] = -1   # of an empty segment
        with pytest.raises(B.KvcError):
            sess.evict_rank_select(wrong, seg, protect_tail_blocks=1)
        got = sess.evict_rank_select(torch.from_numpy(budget).int(), seg, protect_tail_blocks=1)
        np.testing.assert_array_equal(got[0].cpu().numpy().reshape(-1), np.asarray(rows).reshape(-1))
        np.testing.assert_array_equal(got[1].cpu().numpy(), sel)
        compare(sess, st, sess.compact_rank(), O.compact_slots(st, masks))
