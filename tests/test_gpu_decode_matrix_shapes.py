"""Decode shapes that run on the matrix cores with blocks shorter than 16 tokens or rows of 64
dimensions, against the CPU oracle: outputs as near to 64 bits as the plain ALUs leave them."""
import numpy as np
import pytest
import torch

from oracle import kvc_oracle as O
from paper_2410_00161_amd import binding as B
from paper_2410_00161_amd import workloads as W
from helpers import oracle_state
from test_gpu_window_paths import make

pytestmark = pytest.mark.gpu
LENGTHS = [1, 2, 15, 16, 17, 0, 31, 33, 63, 64, 65, 200, 1300, 700, 9, 512]


@pytest.mark.parametrize("r,d,b,dtype", [
    (8, 64, 16, "bf16"), (8, 64, 8, "bf16"), (8, 64, 64, "fp8"), (8, 64, 2, "fp8"),
    (8, 128, 8, "bf16"), (8, 128, 1, "bf16"), (8, 128, 4, "fp8"), (4, 128, 8, "fp8"), (4, 128, 2, "fp8"),
])
@pytest.mark.parametrize("chunk", [0, 128, 2048])   # picked on the device; split heads; one-wavefront items
def test_outputs_near_64_bits(r, d, b, dtype, chunk):
    """Three parts of a probability carry all its bits and the logits are sums of exact products in f32:
    2.5e-7 (2-norm) measured here as on the plain ALUs; two parts (16 bits of a probability) leave 1.0e-6,
    so 6e-7 tells them apart.  Metric: the exps' 16-bit record moves a probability by 2^-17."""
    from paper_2410_00161_amd.session import KvcSession
    shape, cache, real = make(2, 2, 4, r, d, b, LENGTHS, dtype, 0)
    for t in (cache.v_cache,):      # empty slots may hold anything
        if dtype == "fp8":
            t.view(torch.uint8)[~torch.from_numpy(real)] = 0x7F
        else:
            t[~torch.from_numpy(real)] = float("nan")
    st = oracle_state(cache)
    q = W.make_query(shape, 3)
    before = cache.metric.numpy().astype(np.float64)
    want = O.paged_decode(st, q.double().numpy())
    B.kvc_set_decode_chunk(chunk)
    try:
        sess = KvcSession(cache)
        out = sess.paged_decode(q.to(sess.device))
        torch.cuda.synchronize()
    finally:
        B.kvc_set_decode_chunk(0)
    got = out.double().cpu().numpy().reshape(want.shape)
    assert np.linalg.norm(got - want) <= 6e-7 * np.linalg.norm(want)
    m = sess.cache.metric.cpu().numpy().astype(np.float64)
    np.testing.assert_allclose(m[real], st.metric[real], rtol=0, atol=r * 2.0 ** -15)
    np.testing.assert_array_equal(m[~real], before[~real])


@pytest.mark.parametrize("r,d,b", [(8, 64, 16), (8, 64, 8), (8, 128, 8), (8, 128, 1)])
@pytest.mark.parametrize("chunk", [0, 128, 2048])
def test_infinite_values_stay_infinite(r, d, b, chunk):
    """An infinite value times a probability, however few bits that has, is infinite; the other dimensions
    and the metric do not notice.  (8-bit floats have no infinities.)"""
    from paper_2410_00161_amd.session import KvcSession
    shape, cache, real = make(2, 2, 4, r, d, b, LENGTHS, "bf16", 0)
    clean = cache.clone()
    table = cache.block_table.reshape(shape.G, -1)
    sign = np.zeros((shape.G, d))
    for g, j, k, x in ((0, 0, 7, 1), (3, 7, 5, 1), (3, 15, 6, -1), (8, 62, 9, 1), (12, 1000, 3, -1), (12, 40, 3, -1), (15, 511, 0, 1)):
        cache.v_cache[int(table[g, j // b]), j % b, k] = x * float("inf")
        sign[g, k] = x
    q = W.make_query(shape, 3)
    B.kvc_set_decode_chunk(chunk)
    try:
        sess, ref = KvcSession(cache), KvcSession(clean)
        got, want = (s.paged_decode(q.to(s.device)).cpu().numpy().reshape(shape.G, r, d) for s in (sess, ref))
    finally:
        B.kvc_set_decode_chunk(0)
    hit = np.broadcast_to((sign != 0)[:, None], got.shape)
    np.testing.assert_array_equal(got[hit], (np.broadcast_to(sign[:, None], got.shape)[hit] * np.inf).astype(np.float32))
    np.testing.assert_array_equal(got[~hit], want[~hit])
    np.testing.assert_array_equal(sess.cache.metric.cpu().numpy(), ref.cache.metric.cpu().numpy())
