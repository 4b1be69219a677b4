"""Kept work lists for caches whose rows have room for more chunks than a pool of compressed heads
fills: accepted as long as lists of 256-token chunks of full rows fit the workspace, and the same
numbers as plain calls, whichever layers hold the tokens."""
import numpy as np
import pytest
import torch

from paper_2410_00161_amd import binding as B
from paper_2410_00161_amd import workloads as W

pytestmark = pytest.mark.gpu


def records(shape, chunk):
    """(records that lists of such chunks of full rows take, records the workspace holds)"""
    heads = shape.num_seqs * shape.num_kv_heads
    pool, row = shape.num_blocks * shape.block_size, shape.max_blocks_per_head * shape.block_size
    T = 3456 if shape.group_size >= 8 else 6144
    most = min(max(min(pool, heads * row) // T, 410) + heads, heads * -(-row // chunk))
    return most * shape.num_layers, pool // 64 + shape.G + 1


@pytest.mark.parametrize("S,Lyr,Hk,r,row,dtype,full,spare", [
    (1, 32, 8, 4, 1024, "bf16", (0, 31), 100),      # heads that find their own item in a plain call
    (16, 13, 8, 4, 544, "bf16", (12,), 2500),        # 128 heads a layer
    (3, 14, 8, 8, 700, "fp8", (0, 1, 2), 100),      # the tokens in the first layers: later lists start far behind
])
def test_lists_of_rows_with_room(S, Lyr, Hk, r, row, dtype, full, spare):
    from paper_2410_00161_amd.session import KvcSession
    G = S * Lyr * Hk
    ctx = (row / 4 * torch.rand(G, generator=torch.Generator().manual_seed(4))).to(torch.int32).view(S, Lyr, Hk)
    for l in full:
        ctx[:, l] = row - 1
    ctx[0, 3, 1] = 0
    ctx = ctx.reshape(-1)
    N = W.pool_size(ctx, 16, 1.0, spare)
    shape = W.Shape(S, Lyr, Hk, r, 128, 16, N, -(-row // 16), dtype)
    (old, room), (new, _) = records(shape, 256), records(shape, 128)
    assert old <= room < new
    cache = W.make_cache(shape, ctx, 3, placement="fragmented", init_metric="prefill")
    sess, ref = KvcSession(cache.clone()), KvcSession(cache.clone())
    q = W.make_query(shape, 3).to(sess.device)
    for ctx_plus in (0, 1):
        if ctx_plus:
            k, v = (t.to(sess.device) for t in W.make_new_kv(shape, 3))
            sess.decode_plan(ctx_plus=1)
            sess.append(k, v)
            ref.append(k, v)
        else:
            sess.decode_plan()
        sess.out.fill_(5.0)
        for l in reversed(range(Lyr)):
            sess.paged_decode_planned(q, l)
            ref.paged_decode(q, layer_begin=l, layer_end=l + 1)
        torch.cuda.synchronize()
        assert B.kvc_poll_status(sess.cfg, sess.ws) == B.KVC_OK
        np.testing.assert_array_equal(sess.out.cpu().numpy(), ref.out.cpu().numpy())
        np.testing.assert_array_equal(sess.cache.metric.cpu().numpy(), ref.cache.metric.cpu().numpy())


def test_rows_with_far_more_room_are_refused():
    from paper_2410_00161_amd.session import KvcSession
    shape = W.Shape(1, 8, 8, 4, 128, 16, 600, 2048, "bf16")
    old, room = records(shape, 256)
    assert old > room
    sess = KvcSession(W.make_cache(shape, torch.full((64,), 100, dtype=torch.int32), 3))
    with pytest.raises(B.KvcError) as e:
        sess.decode_plan()
    assert e.value.code == B.KVC_ERR_UNSUPPORTED


@pytest.mark.parametrize("row", [512, 1000, 64])
def test_no_record_reaches_past_a_full_row(row):
    """Full heads, the cache's last one among them, planned one token longer: what the list holds ends
    with the row (a decode reads a record's block ids before it compares the length).  The append is
    refused, the decode from the list leaves the heads alone and says so."""
    from paper_2410_00161_amd.session import KvcSession
    S, Hk, b = 2, 8, 16
    row = -(-row // b) * b
    ctx = torch.tensor([row if g in (3, S * Hk - 1) else g * row // 20 for g in range(S * Hk)], dtype=torch.int32)
    shape = W.Shape(S, 1, Hk, 4, 128, b, W.pool_size(ctx, b, 1.2, 40), row // b, "bf16")
    cache = W.make_cache(shape, ctx, 3, placement="fragmented", init_metric="prefill")
    sess = KvcSession(cache)
    sess.decode_plan(ctx_plus=1)
    torch.cuda.synchronize()
    # the workspace: header, the layer's header block, tile sums, two scans over the heads, blocks held, then the records
    ws = sess.ws.view(torch.uint8).cpu()
    at = 512 + 512
    for words in (max(shape.num_blocks, shape.G) // 2048 + 3, shape.G + 1, shape.G + 1, shape.G):
        at += -(-4 * words // 256) * 256
    n = int(ws[512:1024].view(torch.int32)[3])
    records = ws[at:at + 32 * n].view(torch.int32).view(n, 8).numpy()
    assert sorted(set(records[:, 0])) == list(range(S * Hk)) and set(records[records[:, 0] == 3][:, 5]) == {row + 1}
    ends = records[:, 1] + records[:, 2]
    assert ends.max() == row and (records[:, 1] >= 0).all() and (records[:, 2] > 0).all()
    for g in range(S * Hk):
        assert ends[records[:, 0] == g].max() == min(int(ctx[g]) + 1, row)
    k, v = (t.to(sess.device) for t in W.make_new_kv(shape, 3))
    with pytest.raises(B.KvcError) as e:
        sess.append(k, v)
    assert e.value.code == B.KVC_ERR_TABLE_FULL
    sess.out.fill_(5.0)
    sess.paged_decode_planned(W.make_query(shape, 3).to(sess.device), 0)
    torch.cuda.synchronize()
    assert B.kvc_poll_status(sess.cfg, sess.ws) == B.KVC_ERR_ARG
    written = (sess.out.view(S * Hk, -1) != 5.0).any(1).cpu()
    assert written.nonzero().view(-1).tolist() == [0]        # (nothing in it, a row of zeros)
    np.testing.assert_array_equal(sess.cache.metric.cpu().numpy(), cache.metric.cpu().numpy())
