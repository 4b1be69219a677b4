"""One workspace under two configs, as a draft and a target model of one program may have it: what a call leaves there
for the calls after it (the meeting words of decodes without a list among it) is where no other config writes."""
import numpy as np
import pytest
import torch

from oracle import kvc_oracle as O
from paper_2410_00161_amd import binding as B
from paper_2410_00161_amd import workloads as W
from helpers import oracle_state

pytestmark = pytest.mark.gpu


def _model(S, Lyr, Hk, r, most, seed, dtype="bf16", d=128):
    g0 = torch.Generator().manual_seed(seed)
    ctx = (1 + most * torch.rand(S * Lyr * Hk, generator=g0)).to(torch.int32)
    shape = W.Shape(S, Lyr, Hk, r, d, 16, W.pool_size(ctx, 16, 1.2, 3), -(-(most + 40) // 16), dtype)
    cache = W.make_cache(shape, ctx, seed, init_metric="prefill")
    return shape, cache


@pytest.mark.parametrize("reset_under", ["draft", "target"])
@pytest.mark.parametrize("layers", [3, 32])
def test_two_configs_take_turns_on_one_workspace(reset_under, layers):
    from paper_2410_00161_amd.session import KvcSession
    draft_shape, draft_cache = _model(16, 1, 8, 4, 700, 3)
    shape, cache = _model(2, layers, 4, 4, 1500, 5)
    draft, target = KvcSession(draft_cache), KvcSession(cache.clone())
    ws = torch.empty(max(draft.ws.numel(), target.ws.numel()), dtype=torch.uint8, device=target.device)
    ws.fill_(0x5a)   # (what an allocator hands out)
    draft.ws = target.ws = ws
    B.kvc_workspace_reset((draft if reset_under == "draft" else target).cfg, ws)
    st = oracle_state(cache)
    q = W.make_query(shape, 5)
    qd = W.make_query(draft_shape, 3).to(draft.device)
    budget = torch.full((draft_shape.num_seqs,), 20, dtype=torch.int32)
    k_new, v_new = W.make_new_kv(draft_shape, 3)
    for turn in range(2):
        # the draft's turn: work lists, counts and prefix sums in the bytes behind its one layer's block
        draft.append(k_new.to(draft.device), v_new.to(draft.device))
        draft.paged_decode(qd)
        draft.metric_reduce()
        draft.evict_select(budget)
        draft.compact()
        # the target's: decodes without a list, layer by layer, of heads of several chunks
        want = O.paged_decode(st, q.double().numpy())
        out = torch.full_like(target.out, 7.0)
        for layer in range(layers):
            target.paged_decode(q.to(target.device), layer_begin=layer, layer_end=layer + 1, out=out)
        assert B.kvc_poll_status(target.cfg, ws) == B.KVC_OK
        got = out.cpu().numpy()
        # f32 sums over a 16-bit cache (2e-6 elsewhere in these tests)
        assert np.linalg.norm(got - want.reshape(got.shape)) <= 2e-6 * np.linalg.norm(want)
        live = st.free_map == 0
        np.testing.assert_allclose(target.cache.metric.cpu().numpy()[live], st.metric[live], rtol=0, atol=(turn + 1) * 4 * 2.0 ** -15)


def test_words_that_nobody_else_writes_hold_every_head():
    """64 heads of many chunks meet at words of two blocks: each at its own, back at zero after every call."""
    from paper_2410_00161_amd.session import KvcSession
    ctx = torch.tensor([400 + 37 * i for i in range(64)], dtype=torch.int32)
    shape = W.Shape(8, 1, 8, 1, 64, 16, W.pool_size(ctx, 16, 1.1, 3), 180, "fp8")
    cache = W.make_cache(shape, ctx, 9)
    st = oracle_state(cache)
    q = W.make_query(shape, 9)
    want = O.paged_decode(st, q.double().numpy())
    sess = KvcSession(cache)
    first = None
    for turn in range(3):
        out = sess.paged_decode(q.to(sess.device), accumulate_metric=False, out=torch.full_like(sess.out, 7.0)).cpu().numpy()
        assert np.linalg.norm(out - want.reshape(out.shape)) <= 2e-6 * np.linalg.norm(want)
        first = out if first is None else first
        np.testing.assert_array_equal(out, first)
    assert B.kvc_poll_status(sess.cfg, sess.ws) == B.KVC_OK
