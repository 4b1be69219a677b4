"""Decode calls over few head instances, where every workgroup finds its own item from the lengths
(up to 64 heads) and a head's chunks share the work of combining it: against the CPU oracle at the
edges of both (2e-3 max-abs, the bar of the other decode tests)."""
import dataclasses

import numpy as np
import pytest
import torch

from oracle import kvc_oracle as O
from paper_2410_00161_amd import binding as B
from paper_2410_00161_amd import workloads as W
from helpers import oracle_state

pytestmark = pytest.mark.gpu

CASES = [
    # more chunks (of 128 tokens) than the 64 whose weights stay in LDS, and one of their edges
    ("one_head_157_chunks", dict(S=1, Lyr=1, Hk=1, r=4, d=128, kv_dtype="bf16"), [20000]),
    ("one_head_65_chunks_r1_d64", dict(S=1, Lyr=1, Hk=1, r=1, d=64, kv_dtype="f32"), [64 * 128 + 1]),
    ("chunk_edges_r2", dict(S=1, Lyr=1, Hk=6, r=2, d=64, kv_dtype="bf16"), [128, 129, 256, 1, 127, 257]),
    ("empty_heads_r8", dict(S=2, Lyr=1, Hk=4, r=8, d=128, kv_dtype="bf16"), [0, 700, 0, 0, 33, 1, 1500, 0]),
    ("all_whole_fp8", dict(S=1, Lyr=1, Hk=2, r=4, d=128, kv_dtype="fp8"), [100, 128]),
    ("63_heads", dict(S=9, Lyr=1, Hk=7, r=4, d=64, kv_dtype="bf16"), None),
    ("64_heads_fp8_b4", dict(S=8, Lyr=1, Hk=8, r=8, d=128, kv_dtype="fp8", b=4), None),
    ("65_heads", dict(S=13, Lyr=1, Hk=5, r=4, d=128, kv_dtype="bf16"), None),   # a work list again
]


@pytest.mark.parametrize("name,kw,lengths", CASES, ids=[c[0] for c in CASES])
def test_few_heads(name, kw, lengths):
    from paper_2410_00161_amd.session import KvcSession
    b = kw.get("b", 16)
    G = kw["S"] * kw["Lyr"] * kw["Hk"]
    g0 = torch.Generator().manual_seed(9)
    ctx = torch.tensor(lengths, dtype=torch.int32) if lengths else (600 * torch.rand(G, generator=g0) ** 3).to(torch.int32)
    if not lengths:
        ctx[G // 2] = 3000
    maxb = -(-int(ctx.max()) // b) + 2
    shape = W.Shape(kw["S"], kw["Lyr"], kw["Hk"], kw["r"], kw["d"], b, W.pool_size(ctx, b, 1.3, 9), maxb, kw["kv_dtype"])
    # two more layers on either side, so that the call picks one of three
    wide = dataclasses.replace(shape, num_layers=3, num_blocks=3 * shape.num_blocks)
    ctx3 = torch.stack([ctx.flip(0), ctx, ctx // 2], 0).view(3, kw["S"], kw["Hk"]).permute(1, 0, 2).reshape(-1)
    cache = W.make_cache(wide, ctx3, 13, placement="fragmented", init_metric="prefill")
    st = oracle_state(cache)
    q = W.make_query(wide, 13)
    sess = KvcSession(cache)
    sess.out.fill_(7.0)
    for turn in range(2):
        want = O.paged_decode(st, q.double().numpy(), layer_begin=1, layer_end=2)
        out = sess.paged_decode(q.to(sess.device), layer_begin=1, layer_end=2)
        torch.cuda.synchronize()
        got = out.cpu().numpy().astype(np.float64)
        np.testing.assert_allclose(got[:, 1], want[:, 1], rtol=0, atol=2e-3)
        assert (got[:, [0, 2]] == 7.0).all(), "rows of other layers were written"
        live = st.free_map == 0
        np.testing.assert_allclose(sess.cache.metric.cpu().numpy().astype(np.float64)[live], st.metric[live], rtol=0, atol=2e-3)


def test_recorded_calls_have_no_time_for_a_launch_that_does_not_exist():
    """Two launches are recorded, of the long items and of the short ones; the third output is zeros."""
    from paper_2410_00161_amd.session import KvcSession
    ctx = torch.tensor([9000, 300], dtype=torch.int32)
    shape = W.Shape(1, 1, 2, 4, 128, 16, W.pool_size(ctx, 16, 1.1, 3), 600, "bf16")
    sess = KvcSession(W.make_cache(shape, ctx, 3))
    q = W.make_query(shape, 3).to(sess.device)
    B.kvc_profile_begin(4)
    try:
        for _ in range(3):
            sess.paged_decode(q)
        chunk, short, combine = B.kvc_profile_collect(4)
    finally:
        B.kvc_profile_begin(0)
    assert len(chunk) == len(short) == len(combine) == 3
    assert min(chunk) > 0 and combine == [0.0] * 3
