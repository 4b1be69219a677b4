"""kvc_block_alloc where the requests of heads meet the tiles of the free map in every way (heads of many
requests across tiles, many heads in a tile, long runs of heads without one), with what an earlier call
left in the workspace: the k-th lowest free block to the k-th request in ascending head order."""
import statistics

import pytest
import torch

from paper_2410_00161_amd import binding as B

pytestmark = pytest.mark.gpu

DEV = "cuda:0"


class Pool:
    def __init__(self, S, Lyr, Hk, N, maxb, held, free_share, seed, align=0):
        G = S * Lyr * Hk
        g = torch.Generator(device=DEV)
        g.manual_seed(seed)
        self.held = torch.randint(0, held + 1, (G,), generator=g, device=DEV)
        total = int(self.held.sum())
        perm = torch.randperm(N, generator=g, device=DEV)
        self.table = torch.full((G, maxb), -1, dtype=torch.int32, device=DEV)
        self.table[torch.arange(maxb, device=DEV)[None] < self.held[:, None]] = perm[:total].int()
        self.free = torch.zeros(N, dtype=torch.uint8, device=DEV)
        self.free[perm[total:total + int(free_share * (N - total))]] = 1
        self.ctx = (self.held * 16).int()
        self.now = [self.table.clone(), self.ctx.clone(), torch.empty(N + align, dtype=torch.uint8, device=DEV)[align:]]
        self.cfg = B.make_config(S, Lyr, Hk, 1, 8, 16, N, maxb, "bf16", B.KVC_L2)
        kv = torch.zeros((N, 16, 8), dtype=torch.bfloat16, device=DEV)
        metric = torch.zeros((N, 16), device=DEV)
        self.keep = (kv, metric)
        self.st = B.make_state(kv, kv, metric, None, *self.now)
        self.ws = B.new_workspace(self.cfg, torch.device(DEV))

    def alloc(self, n):
        for t, was in zip(self.now, (self.table, self.ctx, self.free)):
            t.copy_(was)
        B.kvc_block_alloc(self.cfg, self.st, n, self.ws, flags=B.KVC_ASYNC)

    def check(self, n):
        torch.cuda.synchronize()
        assert B.kvc_poll_status(self.cfg, self.ws) == B.KVC_OK
        total = int(n.sum())
        ids = torch.nonzero(self.free)[:total, 0]
        off = torch.cumsum(n, 0) - n
        g = torch.repeat_interleave(torch.arange(len(n), device=DEV), n.long())
        want = self.table.clone()
        want[g, self.held[g] + torch.arange(total, device=DEV) - off[g]] = ids.int()
        assert torch.equal(self.now[0], want) and torch.equal(self.now[1], self.ctx)
        left = self.free.clone()
        left[ids] = 0
        assert torch.equal(self.now[2], left)


@pytest.mark.parametrize("S,Lyr,Hk,N,maxb,held,free_share,align", [
    (1, 1, 1, 5000, 4200, 40, 1.0, 0), (1, 1, 3, 9001, 2600, 5, 0.9, 1), (1, 1, 65, 20480, 300, 9, 0.5, 0),
    (3, 43, 5, 150007, 900, 20, 0.4, 0), (17, 16, 16, 200000, 200, 12, 0.6, 3),
])
def test_requests_against_tiles(S, Lyr, Hk, N, maxb, held, free_share, align):
    G = S * Lyr * Hk
    p = Pool(S, Lyr, Hk, N, maxb, held, free_share, 7, align)
    room, n_free = maxb - held, int(p.free.sum())
    g = torch.Generator().manual_seed(2)
    asks = [
        torch.ones(G), (torch.rand(G, generator=g) < 0.05).float(), torch.randint(0, 9, (G,), generator=g),
        torch.where(torch.arange(G) % 50 == G % 50, min(room, n_free // (G // 50 + 1)), 0),       # a few heads of many
        torch.where(torch.rand(G, generator=g) < 0.02, min(room, 100), torch.randint(0, 2, (G,), generator=g)),
        torch.zeros(G), (torch.arange(G) == G - 1) * min(room, n_free),                            # the last head alone
    ]
    for n in asks + asks[::-1]:
        n = n.to(DEV, torch.int32)
        if int(n.sum()) > n_free:
            continue
        p.alloc(n)
        p.check(n)


def test_few_requests_among_many_heads_cost_little_more_than_none():
    """16 384 heads, 1000 of them asking for a block (a search through all heads' offsets for each took
    more than twice as long as no request at all)."""
    p = Pool(64, 32, 8, 1350000, 512, 60, 0.3, 3)
    some = (torch.rand(16384, generator=torch.Generator().manual_seed(1)) < 0.06).to(DEV, torch.int32)
    took = []
    for n in (torch.zeros_like(some), some):
        times = []
        for _ in range(30):
            p.alloc(torch.zeros_like(some))   # (puts the state back; its own launches are done before the clock starts)
            for t, was in zip(p.now, (p.table, p.ctx, p.free)):
                t.copy_(was)
            torch.cuda._sleep(40000)
            a, e = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            B.kvc_block_alloc(p.cfg, p.st, n, p.ws, flags=B.KVC_ASYNC)
            e.record()
            torch.cuda.synchronize()
            times.append(a.elapsed_time(e))
        p.check(n)
        took.append(statistics.median(times))
    # 16.0 and 21.3 us, a ratio of 1.33 to 1.34 in five runs; with the search 15.4 and 43.3 us, 2.8: the line is
    # between the two, near their geometric mean (1.9)
    assert took[1] <= 2 * took[0], took
