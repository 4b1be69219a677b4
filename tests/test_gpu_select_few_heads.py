"""Keys, digit histograms, ties and flag prefixes of a block schedule with few heads, whose rows several
wavefronts share: blocks around the edges of one load and of four, heads with no candidate, keys that tie,
one sequence per segment and several, a key that is no number in the last share."""
import numpy as np
import pytest
import torch

from oracle import kvc_oracle as O
from paper_2410_00161_amd import binding as B
from helpers import oracle_state
from test_gpu_sliced_moves import compare
from test_gpu_window_paths import make

pytestmark = pytest.mark.gpu
BLOCKS = [63, 64, 65, 1, 255, 256, 257, 0, 1025, 320, 1023, 2, 511, 512, 513, 129]


@pytest.mark.parametrize("S,Lyr,Hk", [(2, 1, 1), (4, 2, 3), (4, 16, 16), (5, 41, 5)])   # 2, 24, 1024 and 1025 heads
@pytest.mark.parametrize("ties", [False, True])
def test_shared_rows(S, Lyr, Hk, ties):
    from paper_2410_00161_amd.session import KvcSession
    G = S * Lyr * Hk
    blocks = (BLOCKS * (G // len(BLOCKS) + 1))[:G] if G <= 64 else [BLOCKS[g % 16] if g % 37 < 9 else g % 5 for g in range(G)]
    lengths = [2 * n - (g % 2 if n else 0) for g, n in enumerate(blocks)]
    shape, cache, _ = make(S, Lyr, Hk, 1, 8, 2, lengths, "bf16", 2200)
    if ties:
        cache.metric = torch.randint(0, 3, cache.metric.shape, generator=torch.Generator().manual_seed(5)).float()
    st = oracle_state(cache)
    sess = KvcSession(cache)
    for off in ([0, 1, S], [0, S]):
        seg = torch.tensor(off, dtype=torch.int32)
        nb = (-(-st.lens() // 2)).reshape(S, -1).sum(1)
        budget = np.array([int(nb[a:b].sum() * 0.4) for a, b in zip(off, off[1:])], dtype=np.int64)
        sess.metric_reduce()
        key, _ = O.block_keys(st)
        flag, count, sel = O.evict_select(st, key, budget, seg_offsets=np.array(off), protect_tail_blocks=1)
        held = -(-st.lens() // 2)
        g = int(np.argmax(held))
        bad = sess.block_key.clone()
        bad.view(shape.G, -1)[g, int(held[g]) - 2] = float("nan")
        with pytest.raises(B.KvcError):
            sess.evict_select(torch.from_numpy(budget).int(), seg, block_key=bad)
        got = sess.evict_select(torch.from_numpy(budget).int(), seg)
        np.testing.assert_array_equal(got[0].cpu().numpy().reshape(flag.shape), flag)
        np.testing.assert_array_equal(got[1].cpu().numpy().reshape(-1), count)
        np.testing.assert_array_equal(got[2].cpu().numpy(), sel)
        compare(sess, st, sess.compact(), O.compact(st, flag, count))


@pytest.mark.parametrize("ties", [False, True])
@pytest.mark.parametrize("longest,Lyr", [(900, 1), (12, 1), (60, 80)])   # 12 heads, in a pool too small for the histograms too, and 960
def test_empty_segments(longest, Lyr, ties):
    from paper_2410_00161_amd.session import KvcSession
    S, off = 6, [0, 0, 1, 4, 4, 6]
    lengths = [int(x) for x in torch.randint(0, longest, (S * Lyr * 2,), generator=torch.Generator().manual_seed(3))]
    shape, cache, _ = make(S, Lyr, 2, 1, 8, 2, lengths, "bf16", 0)
    assert (shape.num_blocks * 2 < 3 * 256 * 5) == (longest == 12)
    if ties:
        cache.metric = torch.randint(0, 3, cache.metric.shape, generator=torch.Generator().manual_seed(5)).float()
    st = oracle_state(cache)
    sess = KvcSession(cache)
    seg = torch.tensor(off, dtype=torch.int32)
    for share in ((0.0, 0.4, 0.0, 0.0, 0.7), (0.0, 9.0, 0.5, 0.0, 0.0)):
        nb = (-(-st.lens() // 2)).reshape(S, -1).sum(1)
        budget = np.array([int(nb[a:e].sum() * f) for a, e, f in zip(off, off[1:], share)], dtype=np.int64)
        sess.metric_reduce()
        flag, count, sel = O.evict_select(st, O.block_keys(st)[0], budget, seg_offsets=np.array(off), protect_tail_blocks=1)
        wrong = torch.from_numpy(budget).int()
        wrong[3] = -1   # of an empty segment
        with pytest.raises(B.KvcError):
            sess.evict_select(wrong, seg)
        got = sess.evict_select(torch.from_numpy(budget).int(), seg)
        np.testing.assert_array_equal(got[0].cpu().numpy().reshape(flag.shape), flag)
        np.testing.assert_array_equal(got[1].cpu().numpy().reshape(-1), count)
        np.testing.assert_array_equal(got[2].cpu().numpy(), sel)
        compare(sess, st, sess.compact(), O.compact(st, flag, count))
