"""Prefill-end metrics at the edges of the kernels' row and chunk sizes, against the CPU oracle:
row counts around 32, 64, 128 and 256 (a kernel variant each), blocks of queries that are worked
off in several passes, tables with far more room than the heads hold, long rows without a work list,
logits that outgrow the first ones by far."""
import numpy as np
import pytest
import torch

from oracle import kvc_oracle as O
from paper_2410_00161_amd import binding as B
from paper_2410_00161_amd import workloads as W
from helpers import oracle_state

pytestmark = pytest.mark.gpu


def make(S, Lyr, Hk, r, d, b, lengths, dtype, room, seed=17):
    ctx = torch.tensor(lengths, dtype=torch.int32)
    maxb = -(-max(max(lengths), room) // b) + 1
    shape = W.Shape(S, Lyr, Hk, r, d, b, W.pool_size(ctx, b, 1.2, 5), maxb, dtype)
    cache = W.make_cache(shape, ctx, seed, placement="fragmented", init_metric="prefill")
    st = oracle_state(cache)
    real = torch.zeros_like(cache.metric, dtype=torch.bool)
    for g in range(st.G):
        n, o = O.slots_of(st, g)
        real[torch.from_numpy(n), torch.from_numpy(o)] = True
    if dtype == "fp8":
        cache.k_cache.view(torch.uint8)[~real] = 0x7F
    else:
        cache.k_cache[~real] = float("nan")     # slots that hold no KV must never leak in
    return shape, cache, real.numpy()


def queries(shape, w, seed=5):
    g = torch.Generator().manual_seed(seed)
    q = torch.randn((shape.num_seqs, shape.num_layers, shape.num_q_heads, w, shape.head_dim), generator=g)
    return q.to(torch.bfloat16)


def check(sess, st, real, before):
    torch.cuda.synchronize()
    m = sess.cache.metric.cpu().numpy().astype(np.float64)
    np.testing.assert_allclose(m[real], st.metric[real], rtol=0, atol=2e-3)
    grown = real & (np.abs(st.metric - before) > 1e-3)
    np.testing.assert_allclose((m - before)[grown], (st.metric - before)[grown], rtol=2e-2, atol=1e-6)
    np.testing.assert_array_equal(m[~real], before[~real])


@pytest.mark.parametrize("r,w,d,b,dtype,room", [
    (1, 32, 128, 16, "bf16", 0), (3, 11, 64, 16, "bf16", 0), (2, 32, 128, 16, "fp8", 0), (5, 13, 128, 8, "bf16", 0),
    (2, 64, 128, 32, "bf16", 0), (4, 33, 128, 16, "bf16", 0), (8, 16, 64, 16, "fp8", 0), (8, 32, 128, 16, "bf16", 0),
    (4, 32, 128, 16, "bf16", 40000), (8, 32, 128, 1, "bf16", 30000),   # rows with far more room: a work list
])
def test_windows(r, w, d, b, dtype, room):
    from paper_2410_00161_amd.session import KvcSession
    # chunk and tile edges (the pool here is small: chunks of 1024), a head shorter than the window, an empty one
    shape, cache, real = make(2, 2, 2, r, d, b, [1024, 1025, 63, 64, 65, 0, max(1, w // 2), 2049], dtype, room)
    st = oracle_state(cache)
    before = cache.metric.numpy().astype(np.float64)
    q = queries(shape, w)
    O.window_metric(st, q.double().numpy(), w, 5)
    sess = KvcSession(cache)
    sess.window_metric(q.to(sess.device), w, 5)
    torch.cuda.synchronize()
    m = sess.cache.metric.cpu().numpy().astype(np.float64)
    np.testing.assert_allclose(m[real], st.metric[real], rtol=0, atol=2e-3)
    big = real & (st.metric > 1e-3)
    np.testing.assert_allclose(m[big], st.metric[big], rtol=2e-2, atol=0)
    np.testing.assert_array_equal(m[~real], before[~real])


@pytest.mark.parametrize("r,w,first,exclude,d,b,dtype,room", [
    (4, 65, 300, 0, 128, 16, "bf16", 0),       # 260 rows: a second pass of one query
    (4, 64, 1000, 3, 128, 16, "bf16", 0),      # 256 rows: one pass
    (8, 127, 0, 10, 64, 16, "fp8", 0),         # the prompt's first queries, all rows at once
    (3, 300, 900, 64, 128, 4, "bf16", 0),      # rows that no pass divides
    (4, 700, 200, 10, 128, 16, "bf16", 0),     # several passes: what all rows at once would leave does not fit the workspace
    (4, 130, 500, 10, 128, 16, "fp8", 50000),  # several passes over a work list, for rows with far more room
    (1, 513, 10, 0, 64, 1, "bf16", 0),
])
def test_blocks_of_queries(r, w, first, exclude, d, b, dtype, room):
    from paper_2410_00161_amd.session import KvcSession
    shape, cache, real = make(1, 2, 2, r, d, b, [1030, 257, 0, 700], dtype, room)
    st = oracle_state(cache)
    before = cache.metric.numpy().astype(np.float64)
    q = queries(shape, w)
    O.query_block_metric(st, q.double().numpy(), w, first, exclude)
    sess = KvcSession(cache)
    sess.query_block_metric(q.to(sess.device), w, first, exclude)
    check(sess, st, real, before)


@pytest.mark.parametrize("r,w,lse,d,dtype,lengths", [
    (4, 32, False, 128, "bf16", [5200, 4097]), (4, 32, True, 128, "fp8", [5200, 0]),        # 128 rows, six chunks a row
    (8, 32, False, 64, "bf16", [5120, 1024]), (2, 16, False, 128, "bf16", [4200, 5200]),    # 256 and 32 rows
])
def test_windows_over_long_rows(r, w, lse, d, dtype, lengths):
    """Rows of more than four chunks that the heads nearly fill: items from an index grid."""
    from paper_2410_00161_amd.session import KvcSession
    shape, cache, real = make(2, 1, 2, r, d, 16, [n for n in lengths for _ in range(2)], dtype, 0)
    chunks = -(-shape.max_blocks_per_head * 16 // 1024)
    pool = shape.num_blocks * 16 // 1024 + 4
    assert chunks >= 5 and 4 * chunks <= 2 * min(pool, 4 * chunks)
    st = oracle_state(cache)
    before = cache.metric.numpy().astype(np.float64)
    q = queries(shape, w)
    row_lse = None
    if lse:
        row_lse = np.zeros((2, 1, 2 * r, w))
        for g in range(4):
            n, o = O.slots_of(st, g)
            C = len(n)
            for hq in range(r if C else 0):
                sc = q.double().numpy()[g // 2, 0, (g % 2) * r + hq] @ st.k_cache[n, o].T / np.sqrt(d)
                sc[np.arange(C)[None, :] > (C - w + np.arange(w))[:, None]] = -np.inf
                top = sc.max(1)
                row_lse[g // 2, 0, (g % 2) * r + hq] = top + np.log(np.exp(sc - top[:, None]).sum(1))
        row_lse = row_lse.astype(np.float32)
    O.window_metric(st, q.double().numpy(), w, 7, row_lse=row_lse)
    sess = KvcSession(cache)
    sess.window_metric(q.to(sess.device), w, 7, row_lse=None if row_lse is None else torch.from_numpy(row_lse).to(sess.device))
    torch.cuda.synchronize()
    m = sess.cache.metric.cpu().numpy().astype(np.float64)
    big = real & (st.metric > 1e-6)
    np.testing.assert_allclose(m[big], st.metric[big], rtol=1e-4, atol=0)
    np.testing.assert_array_equal(m[~real], before[~real])


def test_logits_that_outgrow_the_first_tiles():
    """Keys grow along the sequence until their logits stand hundreds of powers of two above the
    first ones, and shrink again: the running maxima of a block in several passes and of a window
    have to follow."""
    from paper_2410_00161_amd.session import KvcSession
    shape, cache, real = make(1, 1, 2, 4, 128, 16, [1500, 900], "bf16", 0)
    st = oracle_state(cache)
    for g in range(2):
        n, o = O.slots_of(st, g)
        j = np.arange(len(n))
        scale = np.where(j < 700, np.exp2(j / 100.0), np.exp2((1400 - j) / 150.0))
        rows = torch.from_numpy(st.k_cache[n, o] * scale[:, None]).to(torch.bfloat16)
        cache.k_cache[torch.from_numpy(n), torch.from_numpy(o)] = rows
    st = oracle_state(cache)
    before = cache.metric.numpy().astype(np.float64)
    q = queries(shape, 100)
    O.query_block_metric(st, q.double().numpy(), 100, 800, 0)
    sess = KvcSession(cache)
    sess.query_block_metric(q.to(sess.device), 100, 800, 0)
    check(sess, st, real, before)
    st = oracle_state(cache)
    qw = queries(shape, 32, seed=6)
    O.window_metric(st, qw.double().numpy(), 32, 1)
    sess = KvcSession(cache)
    sess.window_metric(qw.to(sess.device), 32, 1)
    torch.cuda.synchronize()
    np.testing.assert_allclose(sess.cache.metric.cpu().numpy()[real], st.metric[real], rtol=0, atol=2e-3)
