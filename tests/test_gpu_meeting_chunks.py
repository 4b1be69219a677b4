"""Heads of several chunks, whose workgroups wait for one another and finish the head together: few and
many chunks, more than their pairs' room in LDS, more than the chip runs at once (the first ones then
leave their exps, and the last ones finish for them), from every kind of list; the same bits each time."""
import numpy as np
import pytest
import torch

from oracle import kvc_oracle as O
from paper_2410_00161_amd import binding as B
from paper_2410_00161_amd import workloads as W
from helpers import oracle_state

pytestmark = pytest.mark.gpu

CASES = [
    # chunk length, shape, lengths
    ("two_chunks_each", 64, dict(S=1, Lyr=1, Hk=4, r=8, d=128, kv_dtype="bf16"), [65, 128, 64, 127]),
    ("around_64_chunks", 64, dict(S=1, Lyr=1, Hk=3, r=4, d=128, kv_dtype="fp8"), [64 * 64, 64 * 64 + 1, 63 * 64 + 5]),
    ("pairs_beyond_lds", 64, dict(S=1, Lyr=1, Hk=2, r=1, d=64, kv_dtype="bf16"), [64 * 300 + 9, 64 * 128]),
    ("more_than_run_at_once_r1", 64, dict(S=1, Lyr=1, Hk=2, r=1, d=64, kv_dtype="bf16"), [64 * 2600 + 3, 700]),
    ("more_than_run_at_once_r4", 64, dict(S=1, Lyr=1, Hk=1, r=4, d=64, kv_dtype="f32"), [64 * 2100]),
    ("more_than_run_at_once_r2_b4", 64, dict(S=1, Lyr=1, Hk=1, r=2, d=64, kv_dtype="fp8", b=4), [64 * 2600 - 1]),
    ("picked_on_the_device", 0, dict(S=3, Lyr=2, Hk=8, r=4, d=128, kv_dtype="bf16"), None),
    ("two_pass_list", 512, dict(S=40, Lyr=4, Hk=8, r=2, d=64, kv_dtype="bf16"), None),
]


@pytest.mark.parametrize("name,chunk,kw,lengths", CASES, ids=[c[0] for c in CASES])
def test_split_heads(name, chunk, kw, lengths):
    from paper_2410_00161_amd.session import KvcSession
    b, G = kw.get("b", 16), kw["S"] * kw["Lyr"] * kw["Hk"]
    g0 = torch.Generator().manual_seed(4)
    ctx = torch.tensor(lengths, dtype=torch.int32) if lengths else (1 + 2500 * torch.rand(G, generator=g0) ** 3).to(torch.int32)
    shape = W.Shape(kw["S"], kw["Lyr"], kw["Hk"], kw["r"], kw["d"], b, W.pool_size(ctx, b, 1.1, 3), -(-int(ctx.max()) // b) + 1,
                    kw["kv_dtype"])
    cache = W.make_cache(shape, ctx, 13, placement="fragmented")
    st = oracle_state(cache)
    q = W.make_query(shape, 13)
    want = O.paged_decode(st, q.double().numpy())
    live = st.free_map == 0
    first = None
    B.kvc_set_decode_chunk(chunk)
    try:
        for turn in range(3):
            sess = KvcSession(cache.clone())
            out = sess.paged_decode(q.to(sess.device))
            assert B.kvc_poll_status(sess.cfg, sess.ws) == B.KVC_OK
            again = sess.paged_decode(q.to(sess.device), accumulate_metric=False, out=torch.empty_like(out))
            torch.cuda.synchronize()
            got, metric = out.cpu().numpy(), sess.cache.metric.cpu().numpy()
            np.testing.assert_array_equal(again.cpu().numpy(), got)   # (the counts are back at zero, the list is gone)
            if turn == 0:
                first = got, metric
                # f32 sums (3e-7 measured); where two 16-bit parts of a probability go into a matrix product, the 16 bits
                # that they carry move an output by up to 2^-16 of the values' weighted mean
                parts = kw["d"] == 128 and b >= 16 and (kw["r"] == 8 or kw["kv_dtype"] == "fp8")
                assert np.linalg.norm(got - want.reshape(got.shape)) <= (2.0 ** -16 if parts else 2e-6) * np.linalg.norm(want)
                np.testing.assert_allclose(metric[live], st.metric[live], rtol=0, atol=kw["r"] * 2.0 ** -15)   # exps of 16 bits
            # whoever finished a chunk, the bits are the same
            np.testing.assert_array_equal(got, first[0])
            np.testing.assert_array_equal(metric, first[1])
    finally:
        B.kvc_set_decode_chunk(0)


def test_kept_lists_meet_again():
    """A layer's kept list serves any number of decodes: its meeting words are back at zero after each."""
    from paper_2410_00161_amd.session import KvcSession
    ctx = torch.tensor([3000, 1, 900, 129, 4000, 128, 2000, 640] * 4, dtype=torch.int32)
    shape = W.Shape(2, 2, 8, 4, 128, 16, W.pool_size(ctx, 16, 1.1, 3), 260, "bf16")
    cache = W.make_cache(shape, ctx, 5)
    q = W.make_query(shape, 5)
    plain, sess = KvcSession(cache.clone()), KvcSession(cache.clone())
    sess.decode_plan()
    for turn in range(3):
        for layer in range(2):
            want = plain.paged_decode(q.to(plain.device), layer_begin=layer, layer_end=layer + 1)
            got = sess.paged_decode_planned(q.to(sess.device), layer)
        np.testing.assert_array_equal(got.cpu().numpy(), want.cpu().numpy())
        np.testing.assert_array_equal(sess.cache.metric.cpu().numpy(), plain.cache.metric.cpu().numpy())
    assert B.kvc_poll_status(sess.cfg, sess.ws) == B.KVC_OK


@pytest.mark.parametrize("r,d,dtype", [(8, 64, "bf16"), (8, 128, "fp8"), (4, 64, "fp8")])
def test_few_heads_are_counted_in_the_same_chunks_everywhere(r, d, dtype):
    """Whether a call has few heads for the room of its rows, and can have a kept list, does not depend on how
    many workgroups share a CU: rows of five chunks, 1024 heads a layer."""
    from paper_2410_00161_amd.session import KvcSession
    two = 3456 if r == 8 else 6144
    maxb = 5 * two // 16   # 1024 rows of five chunks are few, of the ten or more shorter ones they would not be
    ctx = torch.full((1024,), 40, dtype=torch.int32)
    ctx[7], ctx[500], ctx[1023] = 9000, 0, 3000
    shape = W.Shape(128, 1, 8, r, d, 16, W.pool_size(ctx, 16, 1.1, 3), maxb, dtype)
    cache = W.make_cache(shape, ctx, 5)
    q = W.make_query(shape, 5)
    plain, sess = KvcSession(cache.clone()), KvcSession(cache.clone())
    assert B.kvc_get_decode_chunk(sess.cfg) < two
    sess.decode_plan()   # (refused: an exception)
    want = plain.paged_decode(q.to(plain.device))
    got = sess.paged_decode_planned(q.to(sess.device), 0)
    assert B.kvc_poll_status(sess.cfg, sess.ws) == B.KVC_OK
    np.testing.assert_array_equal(got.cpu().numpy(), want.cpu().numpy())
    np.testing.assert_array_equal(sess.cache.metric.cpu().numpy(), plain.cache.metric.cpu().numpy())


@pytest.mark.parametrize("layers", [1, 2, 5, 70])
def test_meeting_words_beside_kept_lists(layers):
    """Decodes without a list meet in the header blocks of the layers' kept lists: neither disturbs the other."""
    from paper_2410_00161_amd.session import KvcSession
    ctx = torch.tensor([1500, 1, 900, 129, 2000, 128, 640, 300], dtype=torch.int32).repeat(layers)
    shape = W.Shape(2, layers, 4, 4, 64, 16, W.pool_size(ctx, 16, 1.1, 3), 130, "bf16")
    cache = W.make_cache(shape, ctx, 5)
    q = W.make_query(shape, 5)
    plain, sess = KvcSession(cache.clone()), KvcSession(cache.clone())
    sess.decode_plan()
    for layer in {0, layers // 2, layers - 1}:
        want = plain.paged_decode(q.to(plain.device), layer_begin=layer, layer_end=layer + 1, accumulate_metric=False).clone()
        for turn in range(2):
            got = torch.zeros_like(want)
            sess.paged_decode_planned(q.to(sess.device), layer, accumulate_metric=False, out=got)
            again = torch.zeros_like(want)
            sess.paged_decode(q.to(sess.device), layer_begin=layer, layer_end=layer + 1, accumulate_metric=False, out=again)
            rows = slice(None), slice(layer, layer + 1)
            view = (2, layers, -1)
            np.testing.assert_array_equal(got.view(view)[rows].cpu().numpy(), want.view(view)[rows].cpu().numpy())
            np.testing.assert_array_equal(again.view(view)[rows].cpu().numpy(), want.view(view)[rows].cpu().numpy())
    assert B.kvc_poll_status(sess.cfg, sess.ws) == B.KVC_OK


def _words_of(shape):
    """Where the temporaries of a decode begin in the workspace, in 32-bit words."""
    S, Lyr, G = shape.num_seqs, shape.num_layers, shape.G
    items = shape.num_blocks * shape.block_size // 64 + G + 1
    sizes = dict(header=512, plan_hdr=512 * Lyr, tile_sums=4 * ((max(shape.num_blocks, G) + 1) // 2048 + 2), off_a=4 * (G + 1),
                 off_b=4 * (G + 1), held=4 * G, items=32 * items, slot_word=4 * items, part_ml=8 * shape.group_size * items)
    at, out = 0, {}
    for name, n in sizes.items():
        out[name] = at // 4
        at += -(-n // 256) * 256
    return out


def test_chunks_that_leave_in_calls_of_few_heads():
    """More chunks than the chip has places for, at the library's own chunk length: without a list and from a kept one
    some chunks leave, the others finish for them, twice in a row and with the same bits."""
    from paper_2410_00161_amd.session import KvcSession
    S, Hk, r, d = 2, 4, 8, 64   # (8-bit rows: chunks of 1664 tokens, 1024 places; a head of 1322 chunks among shorter ones)
    ctx = torch.tensor([70000, 2200003, 1665, 40, 3329, 90017, 1664, 130000], dtype=torch.int32)
    shape = W.Shape(S, 1, Hk, r, d, 16, W.pool_size(ctx, 16, 1.01, 3), -(-int(ctx.max()) // 16) + 1, "fp8")
    cache = W.make_cache(shape, ctx, 21, device="cuda:0")
    q = W.make_query(shape, 21).cuda()
    want, p2 = torch.empty(S * Hk, r, d, dtype=torch.float64), torch.zeros(shape.num_blocks, 16, dtype=torch.float64, device="cuda:0")
    for g in range(S * Hk):
        C, ids = int(ctx[g]), cache.block_table.view(S * Hk, -1)[g]
        ids = ids[ids >= 0].long()
        k, v = ((t.view(torch.uint8)[ids].view(torch.float8_e4m3fn).to(torch.float64).reshape(-1, d)[:C]) for t in (cache.k_cache, cache.v_cache))
        p = torch.softmax(q.view(S * Hk, r, d)[g].double() @ k.t().contiguous() / d ** 0.5, dim=1)
        want[g] = (p @ v).cpu()
        sq = torch.zeros(ids.numel() * 16, dtype=torch.float64, device="cuda:0")
        sq[:C] = (p * p).sum(0)
        p2[ids] = sq.view(-1, 16)
    first = None
    for kept in (False, True):
        sess = KvcSession(cache.clone())
        if kept:
            sess.decode_plan()
        marks = sess.ws.view(torch.int32)[_words_of(shape)["part_ml"]:][:sum(n for n in (-(-int(c) // 1664) for c in ctx) if n > 1) * r * 2].view(-1, r, 2)
        for turn in range(2):
            marks.zero_()
            out = sess.paged_decode_planned(q, 0) if kept else sess.paged_decode(q)
            left = int((marks[:, 0, 1] < 0).sum())
            print(f"[case] kept={kept} turn={turn}: {left} of {marks.shape[0]} chunks left", flush=True)
            assert B.kvc_poll_status(sess.cfg, sess.ws) == B.KVC_OK
            assert 0 < left < marks.shape[0] and bool((marks[:, :, 1] != 0).all())
            got, metric = out.cpu().numpy().reshape(S * Hk, r, d), sess.cache.metric.double()
            assert np.linalg.norm(got - want.numpy()) <= 2e-6 * np.linalg.norm(want.numpy())   # f32 sums
            # exps of 16 bits: an increment is off by a few of their halves at most, and the sum over a head by what these cancel to
            assert float((metric - (turn + 1) * p2).norm() / p2.norm()) <= (turn + 1) * 2.0 ** -12
            np.testing.assert_allclose(metric.cpu().numpy(), (turn + 1) * p2.cpu().numpy(), rtol=0, atol=(turn + 1) * r * 2.0 ** -15)
            bits = got, metric.cpu().numpy() / (turn + 1)
            first = bits if first is None else first
            np.testing.assert_array_equal(bits[0], first[0])
            if turn == 0:
                np.testing.assert_array_equal(bits[1], first[1])
        del sess, marks


@pytest.mark.parametrize("kept", [False, True], ids=["no_list", "kept_list"])
@pytest.mark.parametrize("word", [1 << 16, 3 << 16, 1, 2, 0x10001, 0x20002, 0x50003, 7 << 16, -1, -(1 << 16), 0x5a5a5a5a], ids=hex)
def test_words_that_are_not_zero_are_reported(word, kept):
    """Counts left by something else, as in a workspace that was never reset or that two calls at once have used: never
    an unfinished head with the status OK.  A reset (and, of a kept list, a new plan) makes the workspace good again."""
    from paper_2410_00161_amd.session import KvcSession
    ctx = torch.tensor([3000, 1, 900, 1290, 4000, 128, 2000, 640], dtype=torch.int32)   # (up to 32 chunks)
    shape = W.Shape(1, 1, 8, 4, 128, 16, W.pool_size(ctx, 16, 1.1, 3), 260, "bf16")
    cache = W.make_cache(shape, ctx, 5)
    q = W.make_query(shape, 5)
    sess = KvcSession(cache)

    def call():
        out = torch.full_like(sess.out, 7.0)
        if kept:
            return sess.paged_decode_planned(q.to(sess.device), 0, accumulate_metric=False, out=out).cpu().numpy()
        return sess.paged_decode(q.to(sess.device), accumulate_metric=False, out=out).cpu().numpy()

    if kept:
        sess.decode_plan()
    want = call()
    words = sess.ws.view(torch.int32)
    # the words of the list's partial-result slots, or the second halves of the header block and of the first layer's
    at, n = (_words_of(shape)["slot_word"], shape.num_blocks * 16 // 64 + 8 + 1) if kept else (64, 192)
    planted = words[at:at + n].clone()
    if kept:
        planted += word
    else:
        planted[:64] += word
        planted[128:] += word
    words[at:at + n] = planted
    for turn in range(2):
        got = call()
        reported = B.kvc_poll_status(sess.cfg, sess.ws) == B.KVC_ERR_ARG
        assert reported or np.array_equal(got, want)
        assert reported or turn == 0
        words[0] = 0   # (the status alone)
    B.kvc_workspace_reset(sess.cfg, sess.ws)
    if kept:
        sess.decode_plan()
    np.testing.assert_array_equal(call(), want)
    assert B.kvc_poll_status(sess.cfg, sess.ws) == B.KVC_OK


@pytest.mark.parametrize("kept", [False, True], ids=["list", "kept_list"])
def test_long_chunks_have_places_at_once(kept):
    """32-bit rows of d = 128 with eight query heads leave one workgroup a CU, 256 in all: 72 heads, cut by the fraction of
    their tokens into some 320 chunks of nearly one length, are cut longer; few short heads more or less do not count."""
    from paper_2410_00161_amd.session import KvcSession
    g0 = torch.Generator().manual_seed(2)
    ctx = (1100 + 2000 * torch.rand(72, generator=g0)).to(torch.int32)
    ctx[3], ctx[40], ctx[71] = 0, 1, 130
    shape = W.Shape(9, 1, 8, 8, 128, 16, W.pool_size(ctx, 16, 1.1, 3), 200, "f32")
    cache = W.make_cache(shape, ctx, 5)
    st = oracle_state(cache)
    q = W.make_query(shape, 5)
    want = O.paged_decode(st, q.double().numpy())
    sess = KvcSession(cache)
    if kept:
        sess.decode_plan()
        out = sess.paged_decode_planned(q.to(sess.device), 0).cpu().numpy()
    else:
        out = sess.paged_decode(q.to(sess.device)).cpu().numpy()
    assert B.kvc_poll_status(sess.cfg, sess.ws) == B.KVC_OK
    assert np.linalg.norm(out - want.reshape(out.shape)) <= 2e-6 * np.linalg.norm(want)
    live = st.free_map == 0
    np.testing.assert_allclose(sess.cache.metric.cpu().numpy()[live], st.metric[live], rtol=0, atol=8 * 2.0 ** -15)
    items = int(sess.ws.view(torch.int32)[_words_of(shape)["plan_hdr"] + 3 if kept else 3])   # items listed
    tokens = int(ctx.sum())
    assert -(-tokens // 512) > 256 and 72 < items <= 256 + 3


@pytest.mark.parametrize("heads,two", [(376, False), (392, True), (512, True), (520, False)])
def test_rows_of_one_chunk_of_two_workgroups(heads, two):
    """Rows that a chunk for two workgroups a CU holds whole, one for three does not: whole where all heads then have
    places at once, and halves would not."""
    cfg = B.make_config(heads // 8, 1, 8, 8, 128, 16, heads * 204, 204, "fp8")   # 3264 tokens
    assert B.kvc_get_decode_chunk(cfg) == (3456 if two else 1920)
