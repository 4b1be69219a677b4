"""The rank schedule over few heads looks a head's rows below the threshold and at it up where the last
pass left them for every digit: against the oracle, by a wavefront or a workgroup per head, with ties (all at
one digit, metrics of zero), heads with nothing to lose, and a threshold whose last digit is 0 or 255."""
import numpy as np
import pytest
import torch

from oracle import kvc_oracle as O
from helpers import oracle_state
from test_gpu_sliced_moves import compare
from test_gpu_window_paths import make

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("b,room,protect", [(16, 0, 1), (1, 0, 0), (4, 0, 2), (16, 20000, 0), (32, 9000, 1)])
@pytest.mark.parametrize("values", ["spread", "ties", "zeros", "edges"])
def test_rows_by_digit(b, room, protect, values):
    from paper_2410_00161_amd.session import KvcSession
    S, Lyr, Hk, r = 3, 2, 2, 4
    G = S * Lyr * Hk
    g0 = torch.Generator().manual_seed(3)
    lengths = [int(x) for x in torch.randint(1200, 2000, (G,), generator=g0)]
    lengths[1], lengths[4], lengths[7] = 0, b, 2 * b + 1
    shape, cache, _ = make(S, Lyr, Hk, r, 8, b, lengths, "bf16", room)
    assert 3 * 256 * S + 512 * G <= shape.num_blocks * b * r   # the rows have room
    if values == "ties":
        cache.metric = torch.randint(0, 3, cache.metric.shape, generator=g0).float()
    elif values == "zeros":
        cache.metric = torch.zeros_like(cache.metric)
        cache.metric[::3, 0] = -0.0
    elif values == "edges":   # bit patterns that differ in the last digit alone, 0 and 255 among them
        bits = 0x3F800000 + torch.tensor([0, 255, 1, 254], dtype=torch.int32)[torch.randint(0, 4, cache.metric.shape, generator=g0)]
        cache.metric = bits.view(torch.float32)
    st = oracle_state(cache)
    sess = KvcSession(cache)
    for share in (0.37, 0.0, 0.6):
        nb = (-(-st.lens() // b)).reshape(S, -1).sum(1)
        budget = (nb * share).astype(np.int64)
        budget[1] = 10 * nb[1] if share else 0
        rows, masks, sel = O.rank_schedule(st, budget, None, protect)
        got = sess.evict_rank_select(torch.from_numpy(budget).int(), protect_tail_blocks=protect)
        np.testing.assert_array_equal(got[0].cpu().numpy().reshape(-1), np.asarray(rows).reshape(-1))
        np.testing.assert_array_equal(got[1].cpu().numpy(), sel)
        compare(sess, st, sess.compact_rank(), O.compact_slots(st, masks))
