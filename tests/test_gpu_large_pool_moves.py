"""Compactions in a pool of 2 GiB, whose moves read past the caches: the states that the same tables leave
in a small pool, byte for byte, by each of the launches that move (a head's own workgroup, slices of a head;
block and rank mode), with one or two KVs at a time and blocks of one token to 32."""
import dataclasses

import numpy as np
import pytest
import torch

from paper_2410_00161_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("mode", ["block", "rank"])
@pytest.mark.parametrize("G,most,b,dtype,d", [(12, 2600, 16, "bf16", 128), (600, 700, 8, "fp8", 64), (1100, 300, 32, "bf16", 64),
                                               (40, 900, 1, "f32", 128)])
def test_same_state_as_in_a_small_pool(mode, G, most, b, dtype, d):
    from paper_2410_00161_amd.session import KvcSession
    g0 = torch.Generator().manual_seed(6)
    ctx = (most * torch.rand(G, generator=g0)).to(torch.int32)
    ctx[0], ctx[1] = most, 0
    small = W.Shape(2, 1, G // 2, 2, d, b, W.pool_size(ctx, b, 1.1, 5), -(-most // b) + 2, dtype)
    cache = W.make_cache(small, ctx, 3, placement="fragmented", init_metric="prefill")
    bytes_per_block = 2 * b * d * small.kv_bytes
    n = -(-(2 << 30) // bytes_per_block) + 7
    assert n > small.num_blocks and small.num_blocks * bytes_per_block < 2 << 30
    big = dataclasses.replace(small, num_blocks=n)
    here = KvcSession(cache.clone())
    grow = lambda t, fill: torch.cat([t, torch.full((1,) + tuple(t.shape[1:]), fill, dtype=t.dtype, device=t.device).expand(n - t.shape[0], *t.shape[1:])])  # noqa: E731
    c = here.cache
    raw = lambda t: t.view(torch.uint8) if t.dtype == torch.float8_e4m3fn else t  # noqa: E731
    back = lambda t, like: t.view(like.dtype) if like.dtype == torch.float8_e4m3fn else t  # noqa: E731
    there = KvcSession(W.Cache(big, back(grow(raw(c.k_cache), 0), c.k_cache), back(grow(raw(c.v_cache), 0), c.v_cache), grow(c.metric, 0.0),
                               grow(c.pos, -1), c.block_table.clone(), c.ctx_len.clone(), grow(c.free_map, 0)))
    budget = torch.tensor([int(x) for x in (-(-ctx.view(2, -1) // b)).sum(1) * 2 // 5], dtype=torch.int32)
    for _ in range(2):
        freed = []
        for s in (here, there):
            if mode == "block":
                s.metric_reduce()
                s.evict_select(budget)
                freed.append(int(s.compact().item()))
            else:
                s.evict_rank_select(budget)
                freed.append(int(s.compact_rank().item()))
        assert freed[0] == freed[1] == int(budget.sum())
        for name in ("block_table", "ctx_len"):
            assert torch.equal(getattr(here.cache, name), getattr(there.cache, name)), name
        for name in ("k_cache", "v_cache", "metric", "pos", "free_map"):
            a, z = raw(getattr(here.cache, name)), raw(getattr(there.cache, name))[:small.num_blocks]
            assert torch.equal(a.contiguous().view(torch.uint8), z.contiguous().view(torch.uint8)), name
