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
