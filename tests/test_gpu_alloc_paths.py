"""The allocator's launches at the sizes where they can go wrong, against the CPU oracle, bit
for bit: rows longer than a wavefront, head counts that no workgroup divides, requests that run
across tiles of the free map."""
import numpy as np
import pytest
import torch

from oracle import kvc_oracle as O
from paper_2410_00161_amd import binding as B
from paper_2410_00161_amd import workloads as W
from helpers import check_allocator_invariants, oracle_state

pytestmark = pytest.mark.gpu


def assert_tables_equal(sess, st):
    torch.cuda.synchronize()
    c = sess.cache
    np.testing.assert_array_equal(c.block_table.cpu().numpy().astype(np.int64), st.block_table)
    np.testing.assert_array_equal(c.ctx_len.cpu().numpy().astype(np.int64), st.ctx_len)
    np.testing.assert_array_equal(c.free_map.cpu().numpy(), st.free_map)


@pytest.mark.parametrize("S,Lyr,Hk,b,tokens", [
    (3, 3, 1, 16, [1023, 1, 16 * 64]),         # rows of 63, 1 and 64 blocks
    (4, 5, 2, 4, [0, 1300, 257, 4]),           # 5 full wavefronts of a row and a remainder; one sequence left out
    (17, 1, 1, 1, list(range(60, 77))),        # one block per token, more heads than a workgroup takes
])
def test_prompts_admitted_and_preempted(S, Lyr, Hk, b, tokens):
    from paper_2410_00161_amd.session import KvcSession
    G, L = S * Lyr * Hk, max(tokens)
    N = 2 * Lyr * Hk * sum(-(-t // b) for t in tokens) + 2100
    shape = W.Shape(S, Lyr, Hk, 2, 64, b, N, -(-L // b) + 1, "bf16")
    cache = W.make_cache(shape, torch.full((G,), 3 * b, dtype=torch.int32) if L > 4 * b else torch.zeros(G, dtype=torch.int32),
                         5, placement="fragmented")
    st = oracle_state(cache)
    sess = KvcSession(cache)
    dev = sess.device
    rng = np.random.RandomState(5)
    for turn in range(3):
        mask = torch.from_numpy((rng.rand(S) < 0.6).astype(np.uint8))
        freed = O.preempt(st, mask.numpy())
        assert B.kvc_preempt(sess.cfg, sess.st, mask.to(dev), sess.ws) == freed
        assert_tables_equal(sess, st)
        t = torch.tensor(tokens, dtype=torch.int32)
        t[mask == 0] = 0
        O.prefill_alloc(st, t.numpy())
        B.kvc_prefill_alloc(sess.cfg, sess.st, t.to(dev), sess.ws)
        assert_tables_equal(sess, st)
        check_allocator_invariants(st)
    # one request too many anywhere leaves everything as it was
    t = torch.zeros(S, dtype=torch.int32)
    t[S - 1] = (shape.max_blocks_per_head + 1) * b
    with pytest.raises(B.KvcError):
        B.kvc_prefill_alloc(sess.cfg, sess.st, t.to(dev), sess.ws)
    assert_tables_equal(sess, st)


@pytest.mark.parametrize("S,Lyr,Hk,b,slack_blocks,layers,odd_map", [
    (1, 1, 1, 1, 3, None, False),          # one head, one workgroup; then out of blocks
    (4, 2, 16, 2, 700, None, True),        # 128 heads: a workgroup of rows after the reservation; a map at an odd address
    (2, 2, 32, 2, 900, (1, 2), False),     # 64 heads of one layer: appended by the reservation's launch
    (5, 2, 13, 2, 900, (1, 2), False),     # 65 heads: rows written by a launch of their own
    (41, 5, 5, 1, 20000, None, False),     # 1025 heads: two workgroups of heads, two of the map
    (2, 4, 3, 1, 1200000, (0, 3), False),  # more of the map than 64 workgroups' first rounds
])
def test_append_takes_the_lowest_free_blocks(S, Lyr, Hk, b, slack_blocks, layers, odd_map):
    from paper_2410_00161_amd.session import KvcSession
    G = S * Lyr * Hk
    g0 = torch.Generator().manual_seed(3)
    ctx = torch.randint(0, 3 * b + 2, (G,), generator=g0, dtype=torch.int32)
    held = int(W.blocks_needed(ctx, b).sum())
    shape = W.Shape(S, Lyr, Hk, 1, 8, b, held + slack_blocks, 8, "bf16")
    cache = W.make_cache(shape, ctx, 7, placement="fragmented")
    if odd_map:
        buf = torch.empty(shape.num_blocks + 1, dtype=torch.uint8, device="cuda:0")
        cache = cache.to("cuda:0")
        buf[1:] = cache.free_map
        cache.free_map = buf[1:]
    st = oracle_state(cache)
    sess = KvcSession(cache)
    l0, l1 = layers or (0, Lyr)
    for step in range(2 * b + 2):
        k, v = W.make_new_kv(shape, 11, step)
        try:
            O.append(st, k.double().numpy(), v.double().numpy(), layer_begin=l0, layer_end=l1)
            failed = False
        except O.OracleError:   # raised with the state untouched
            failed = True
        if failed:
            with pytest.raises(B.KvcError):
                sess.append(k.to(sess.device), v.to(sess.device), None, l0, l1)
        else:
            sess.append(k.to(sess.device), v.to(sess.device), None, l0, l1)
        assert_tables_equal(sess, st)
    kc, vc = sess.cache.k_cache.float().cpu().numpy(), sess.cache.v_cache.float().cpu().numpy()
    metric, pos = sess.cache.metric.cpu().numpy(), sess.cache.pos.cpu().numpy()
    for g in range(0, G, max(1, G // 50)):
        n, o = O.slots_of(st, g)
        np.testing.assert_array_equal(kc[n, o], st.k_cache[n, o])
        np.testing.assert_array_equal(vc[n, o], st.v_cache[n, o])
        np.testing.assert_array_equal(pos[n, o], st.pos[n, o])
        np.testing.assert_array_equal(metric[n, o].astype(np.float64), st.metric[n, o])
