"""Blocks of many query rows of the all-queries metric: which calls the streamed launches take (the
rule is repeated here, so that a case that leaves them fails instead of passing for nothing), and
that what they add is as exact as the same block worked off in calls of at most 256 query rows."""
import numpy as np
import pytest
import torch

from paper_2410_00161_amd import binding as B
from paper_2410_00161_amd import workloads as W

pytestmark = pytest.mark.gpu

DEV = "cuda:0"


def streamed_chunk(shape, w, first, lse, layers=None):
    """Tokens per chunk of the streamed launches for this call, 0 where the block is worked off in
    passes of at most 256 query rows."""
    r, d, b = shape.group_size, shape.head_dim, shape.block_size
    rows, tiles = w * r, -(-w // 64)
    row_blocks = -(-rows // 256)
    if rows <= 256 or tiles * 64 * 8 > 9 * w or row_blocks * 256 * 8 > 9 * rows:
        return 0
    gsel = shape.num_seqs * (shape.num_layers if layers is None else layers) * shape.num_kv_heads
    pool = shape.num_blocks * b
    reach = min(shape.max_blocks_per_head * b, first + w)
    T = 4096
    while T > 1024 and min(gsel * reach, pool) // T * row_blocks < 2048:
        T //= 2
    chunks = -(-reach // T)
    if gsel * chunks > 2 * (pool // T + gsel):
        return 0
    pairs = 0 if lse else -(-gsel * chunks * rows * 8 // 256) * 256
    room = (pool // 64 + shape.G + 1) * r * d * 4
    return T if pairs + gsel * r * tiles * 64 * 4 <= room else 0


def prompt(S, Lyr, Hk, r, d, b, lengths, dtype, seed, slack=1.3):
    """A cache of prompts (one length per sequence) with blocks all over the pool, on the GPU."""
    per = Lyr * Hk
    ctx = torch.tensor(lengths, dtype=torch.int32).repeat_interleave(per)
    shape = W.Shape(S, Lyr, Hk, r, d, b, W.pool_size(ctx, b, slack, 5), -(-max(lengths) // b) + 1, dtype)
    cache = W.make_cache(shape, ctx, seed, placement="fragmented").to(DEV)
    used = torch.zeros(shape.num_blocks * b, dtype=torch.bool, device=DEV)   # the rest must never leak in
    for g, C in enumerate(ctx.tolist()):
        j = torch.arange(C, device=DEV)
        used[cache.block_table.view(len(ctx), -1)[g, j // b].long() * b + j % b] = True
    rows = cache.k_cache.view(-1, d)
    if dtype == "fp8":
        rows.view(torch.uint8)[~used] = 0x7F
    else:
        rows[~used] = float("nan")
    return cache


def queries(shape, w, scale=1.0, seed=5):
    g = torch.Generator().manual_seed(seed)
    q = scale * torch.randn((shape.num_seqs, shape.num_layers, shape.num_q_heads, w, shape.head_dim), generator=g)
    return q.to(torch.bfloat16).to(DEV)


def in_64_bits(cache, q, w, first, exclude, mode="l2"):
    """Per head instance its physical slots, the increments of its keys and the log-sum-exp of its
    query rows, from plain matrix products in 64 bits."""
    sh = cache.shape
    r, d, b = sh.group_size, sh.head_dim, sh.block_size
    q = q.reshape(sh.G, r * w, d)
    table, ctx = cache.block_table.view(sh.G, -1).long(), cache.ctx_len.view(-1).tolist()
    rows = cache.k_cache.view(-1, d)
    at = first + torch.arange(w, device=DEV)
    for g in range(sh.G):
        C = ctx[g]
        j = torch.arange(C, device=DEV)
        slots = table[g, j // b] * b + j % b
        K = rows[slots].float().double() if sh.kv_dtype != "fp8" else rows.view(torch.uint8)[slots].view(torch.float8_e4m3fn).float().double()
        s = (q[g].double() @ K.T.contiguous()).view(r, w, C) * d ** -0.5
        s.masked_fill_(j > at.view(w, 1), -torch.inf)
        lse = torch.logsumexp(s, -1)
        p = torch.exp(s - lse.unsqueeze(-1))
        p = p * p if mode == "l2" else p
        p.masked_fill_(j > (at - exclude).view(w, 1), 0.0)
        yield g, slots, p.sum((0, 1)), lse


def errors_against_short_calls(cache, q, w, first, lse):
    """Distance from 64 bits (2-norm of the difference over 2-norm) of the block in one call, and of the
    same block in calls of at most 256 query rows."""
    from paper_2410_00161_amd.session import KvcSession
    sh = cache.shape
    want = torch.zeros(sh.num_blocks * sh.block_size, dtype=torch.float64, device=DEV)
    row_lse = torch.empty((sh.num_seqs, sh.num_layers, sh.num_q_heads, w), device=DEV)
    for g, slots, inc, l in in_64_bits(cache, q, w, first, 0):
        want[slots] += inc
        row_lse.view(sh.G, sh.group_size, w)[g] = l.float()
    step = min(64, 256 // sh.group_size)
    out = []
    for parts in ([(0, w)], [(i, min(step, w - i)) for i in range(0, w, step)]):
        c = cache.clone()
        c.metric.zero_()
        sess = KvcSession(c)
        for i, n in parts:
            sess.query_block_metric(q[:, :, :, i:i + n].contiguous(), n, first + i, 0,
                                    row_lse=row_lse[:, :, :, i:i + n].contiguous() if lse else None)
        got = sess.cache.metric.double().view(-1)
        out.append(float((got - want).norm() / want.norm()))
    return out


# A tenth above the short calls' own error is the most two correct forms differ by here: both round
# max + log2(sum) of a row once, at the size of its largest logit, and that is most of the error.
@pytest.mark.parametrize("r,d,dtype,w,scale", [
    (4, 64, "fp8", 512, 1.0), (8, 128, "bf16", 256, 1.0), (4, 128, "bf16", 1024, 4.0), (4, 128, "bf16", 512, 12.0),
])
def test_row_sums_are_as_exact_as_a_running_maximum_keeps_them(r, d, dtype, w, scale):
    cache = prompt(1, 2, 4, r, d, 16, [8192], dtype, 21)
    first = 4096
    assert streamed_chunk(cache.shape, w, first, False)
    one, short = errors_against_short_calls(cache, queries(cache.shape, w, scale), w, first, False)
    assert one <= 1.1 * short


# (the log-sum-exp of every row is given, rounded once from 64 bits: what differs is the order of the sum)
@pytest.mark.parametrize("r,d,dtype,w", [(8, 128, "bf16", 4096), (4, 64, "fp8", 4096), (1, 128, "bf16", 8192)])
def test_long_sums_are_as_exact_as_short_ones(r, d, dtype, w):
    cache = prompt(1, 1, 2, r, d, 16, [8192], dtype, 22)
    first = 8192 - w
    assert streamed_chunk(cache.shape, w, first, True)
    one, short = errors_against_short_calls(cache, queries(cache.shape, w), w, first, True)
    assert one <= 1.1 * short


@pytest.mark.parametrize("d,dtype,b", [(128, "bf16", 16), (64, "bf16", 8), (128, "fp8", 64)])
def test_references_follow_the_logits(d, dtype, b):
    """Keys grow along the sequence until their logits stand far above the first ones, and shrink again,
    over several chunks and between the queries' own positions."""
    from paper_2410_00161_amd.session import KvcSession
    lengths, w, first = [3000, 1500, 700], 256, 1200
    cache = prompt(3, 1, 2, 4, d, b, lengths, dtype, 31)
    assert streamed_chunk(cache.shape, w, first, False) == 1024   # three chunks
    rows, ctx = cache.k_cache.view(-1, d), cache.ctx_len.view(-1).tolist()
    for g, C in enumerate(ctx):
        j = torch.arange(C, device=DEV)
        grow = torch.exp2(torch.where(j < 1100, j / 260.0, (1500 - j) / 95.0).clamp(-4.0, 4.5))
        slots = cache.block_table.view(len(ctx), -1)[g, j // b].long() * b + j % b
        if dtype == "fp8":
            old = rows.view(torch.uint8)[slots].view(torch.float8_e4m3fn).float()
            rows.view(torch.uint8)[slots] = (old * grow.view(-1, 1)).to(rows.dtype).view(torch.uint8)
        else:
            rows[slots] = (rows[slots].float() * grow.view(-1, 1)).to(rows.dtype)
    cache.metric.zero_()
    q = queries(cache.shape, w)
    sess = KvcSession(cache)
    sess.query_block_metric(q, w, first, 0)
    got = sess.cache.metric.double().view(-1)
    seen_large = 0.0
    for g, slots, inc, lse in in_64_bits(cache, q, w, first, 0):
        # the row's constant and an exp's argument are each rounded to half a last bit at the size of the
        # largest logits; the square doubles it
        size = float(lse.abs().max()) * 1.4427
        seen_large = max(seen_large, size)
        assert float((got[slots] - inc).norm() / inc.norm()) <= 2 * 0.6931 * size * 2.0 ** -23, g
        assert torch.equal(got[slots][inc == 0], inc[inc == 0])
    assert seen_large > 100


# (S, Lyr, Hk, r, d, b, lengths, dtype, w, first, exclude, lse, mode, chunk)
BLOCKS = [
    (3, 1, 2, 4, 128, 16, [3000, 1500, 700], "bf16", 256, 1200, 10, False, "l2", 1024),    # ragged, up to three chunks
    (1, 2, 2, 4, 128, 16, [5000], "bf16", 128, 4800, 0, False, "l2", 1024),                # tiles without a mask, the queries at the end
    (1, 2, 2, 4, 128, 16, [5000], "bf16", 128, 4990, 0, True, "l2", 1024),                 # queries past the last key
    (1, 1, 3, 8, 128, 64, [2049], "bf16", 57, 1000, 100, False, "l2", 1024),               # few of a tile's rows padded; far back keys only
    (1, 1, 3, 8, 64, 32, [2049], "bf16", 57, 1000, 0, False, "l1", 1024),
    (2, 1, 2, 4, 64, 8, [1300, 0], "bf16", 192, 0, 0, False, "l2", 1024),                  # blocks of half a load; no KV; a prompt's first queries
    (2, 1, 2, 4, 128, 1, [1300, 64], "bf16", 190, 500, 3, False, "l2", 1024),              # a block per token; a head that ends in front of the queries
    (1, 1, 2, 2, 128, 1024, [2500], "bf16", 256, 2000, 0, False, "l1", 1024),
    (2, 1, 2, 4, 128, 16, [3000, 2000], "fp8", 256, 1500, 10, False, "l2", 1024),
    (2, 1, 2, 8, 64, 4, [3000, 1100], "fp8", 128, 1000, 0, True, "l1", 1024),
    (1, 1, 2, 1, 128, 16, [1500], "bf16", 512, 900, 64, True, "l2", 1024),                 # one query head
    (1, 2, 8, 8, 128, 16, [8300], "bf16", 1024, 7200, 10, False, "l2", 2048),
    (1, 4, 8, 8, 64, 16, [8300], "bf16", 512, 7700, 0, False, "l2", 2048),
    (1, 4, 8, 8, 128, 16, [8300], "bf16", 1024, 7276, 0, False, "l2", 4096),
    (1, 4, 8, 8, 128, 16, [8300], "fp8", 1024, 7276, 10, True, "l1", 4096),
]


@pytest.mark.parametrize("S,Lyr,Hk,r,d,b,lengths,dtype,w,first,exclude,lse,mode,chunk", BLOCKS)
def test_streamed_blocks(S, Lyr, Hk, r, d, b, lengths, dtype, w, first, exclude, lse, mode, chunk):
    from paper_2410_00161_amd.session import KvcSession
    cache = prompt(S, Lyr, Hk, r, d, b, lengths, dtype, 41)
    assert streamed_chunk(cache.shape, w, first, lse) == chunk
    cache.metric.zero_()
    q = queries(cache.shape, w)
    want = torch.zeros(cache.shape.num_blocks * b, dtype=torch.float64, device=DEV)
    row_lse = torch.empty((S, Lyr, Hk * r, w), device=DEV)
    size = 1.0
    for g, slots, inc, l in in_64_bits(cache, q, w, first, exclude, mode):
        want[slots] += inc
        row_lse.view(cache.shape.G, r, w)[g] = l.float()
        if len(slots):
            size = max(size, float(l.abs().max()) * 1.4427)
    sess = KvcSession(cache, metric_mode=B.KVC_L1 if mode == "l1" else B.KVC_L2)
    sess.query_block_metric(q, w, first, exclude, row_lse=row_lse if lse else None)
    got = sess.cache.metric.double().view(-1)
    # rounding of a row's constant and of an exp's argument, each half a last bit at the size of the
    # largest logits and doubled by the square, and a few last bits of the sums
    bound = 2 * 0.6931 * size * 2.0 ** -23 + 4 * 2.0 ** -23
    assert float((got - want).norm() / want.norm()) <= bound
    large = want > 1e-3 * want.max()
    assert float(((got - want)[large] / want[large]).abs().max()) <= 4 * bound
    assert torch.equal(got[want == 0], want[want == 0])


def test_a_streamed_block_of_some_layers():
    """Layers 1 and 2 of 4; the metrics of the others stay, and what was there is added to."""
    from paper_2410_00161_amd.session import KvcSession
    cache = prompt(2, 4, 2, 4, 128, 16, [2600, 1400], "bf16", 43)
    w, first = 256, 1100
    assert streamed_chunk(cache.shape, w, first, False, layers=2)
    before = cache.metric.uniform_(0.5, 1.0).double().view(-1).clone()
    q = queries(cache.shape, w)
    want = before.clone()
    for g, slots, inc, _ in in_64_bits(cache, q, w, first, 0):
        if (g // 2) % 4 in (1, 2):
            want[slots] += inc
    sess = KvcSession(cache)
    sess.query_block_metric(q, w, first, 0, layer_begin=1, layer_end=3)
    got = sess.cache.metric.double().view(-1)
    assert float(((got - want) / want).abs().max()) <= 4e-6
    assert torch.equal(got[want == before], before[want == before])


@pytest.mark.parametrize("d,b", [(128, 16), (64, 8)])
def test_infinite_keys(d, b):
    """A query row with a logit of +inf: NaN at that key, nothing added anywhere else by that row (its
    denominator is infinite).  Over three chunks, the keys in different lanes."""
    from paper_2410_00161_amd.session import KvcSession
    cache = prompt(1, 1, 4, 4, d, b, [3000], "bf16", 33)
    w, first = 256, 2700
    assert streamed_chunk(cache.shape, w, first, False) == 1024
    rows, table = cache.k_cache.view(-1, d), cache.block_table.view(4, -1).long()
    for g, j in ((0, 0), (1, 7), (1, 2047), (2, 1030), (2, 2990)):
        rows[table[g, j // b] * b + j % b, (5 * j) % d] = (-1) ** g * float("inf")
    cache.metric.zero_()
    q = queries(cache.shape, w)
    row_lse = torch.empty((1, 1, 16, w), device=DEV)
    for g, _, _, lse in in_64_bits(cache, q, w, first, 0):
        row_lse.view(4, 4, w)[g] = torch.where(torch.isfinite(lse), lse, torch.inf).float()
    got = []
    for lse in (None, row_lse):
        sess = KvcSession(cache.clone())
        sess.query_block_metric(q, w, first, 0, row_lse=lse)
        got.append(sess.cache.metric.cpu())
    assert int(torch.isnan(got[1]).sum()) >= 4 and not bool(torch.isinf(got[1]).any())
    torch.testing.assert_close(got[0], got[1], rtol=1e-4, atol=1e-4 * float(got[1].nan_to_num().max()), equal_nan=True)
