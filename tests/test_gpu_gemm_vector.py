"""GPU parity of the GeMM kernel for one to four tokens on the vector ALUs: K of one load, of a piece of 256 bytes and one more,
of fewer pieces than waves, of one to four pieces a wave and of several rounds; few rows, and more workgroups than run at once."""
import numpy as np
import pytest
import torch

import zq_inputs
from helpers import assert_bit_equal, dev, host
from test_gpu_gemm import SIMPLE, _case, _check, _run, orc, zq  # noqa: F401 (fixtures)
from test_gpu_gemm_gelu import _check_fused

pytestmark = pytest.mark.gpu

ZQ_MAX_K, ZQ_MAX_K_W4 = 133143, 132104          # include/zq.h

# (M, N, K, groups); one and two tokens for both weight types, more for INT8 against few rows and a long K
SHAPES = [
    (1, 16, 16, 1), (1, 16, 32, 1), (1, 48, 256, 3), (1, 2064, 288, 129), (1, 400, 1024, 25), (1, 400, 1056, 5), (1, 4112, 2080, 257),
    (1, 10256, 544, 641), (1, 1616, 6432, 101), (1, 272, 8224, 17), (1, 144, 16416, 3), (1, 48, 40992, 3), (1, 16, 132096, 1),
    (2, 16, 32, 1), (2, 2048, 1056, 128), (2, 1040, 2560, 65), (2, 528, 12320, 11), (2, 6160, 1632, 35), (2, 32, 33312, 2),
    (3, 16, 2560, 1), (3, 2048, 2576, 128), (4, 1040, 4128, 13), (4, 784, 9248, 49),
]


def _kernel(zq, bits, M, N, K):
    """The kernel of a call with the class "simple", which is what _run(..., SIMPLE, ...) makes."""
    before = zq.force_gemm_variant(SIMPLE)
    try:
        return zq.gemm_kernel(M, N, K, bits)
    finally:
        zq.force_gemm_variant(before)


@pytest.mark.parametrize("bits", [8, 4])
@pytest.mark.parametrize("M,N,K,g", SHAPES)
def test_vector_against_oracle(zq, orc, bits, M, N, K, g):
    if bits == 4 and (K % 32 or M > 2):
        pytest.skip("not this kernel")
    print("vector", bits, M, N, K, g, flush=True)
    assert _kernel(zq, bits, M, N, K) == "vector"
    xq, s_tok, s_w, bias, codes, wq = _case(zq_inputs.rng_for(4, 9000 + M + N + K + bits), M, N, K, g, bits)
    if M == 1:
        xq[:] = np.where(xq < 0, -127, 127)                     # activations at full size
    res = _run(zq, bits, SIMPLE, xq, s_tok, wq, s_w, bias)
    _check(orc, res, xq, s_tok, codes, s_w, bias, "vector %d-bit %dx%dx%d" % (bits, M, N, K))


@pytest.mark.parametrize("bits", [8, 4])
@pytest.mark.parametrize("approx", [False, True])
def test_vector_without_bias_and_with_gelu(zq, orc, bits, approx):
    M, N, K, g = 2, 1024, 2080, 64
    xq, s_tok, s_w, bias, codes, wq = _case(zq_inputs.rng_for(4, 9100 + bits), M, N, K, g, bits)
    gemm = zq.zq_gemm_i8_dequant if bits == 8 else zq.zq_gemm_w4a8_dequant
    out, acc, _, _ = gemm(dev(xq), dev(s_tok), dev(wq), dev(s_w), want_acc=True)
    assert_bit_equal(host(acc), orc.matmul_i32(xq, codes), "acc")
    want = (host(acc).astype(np.float32) * (s_tok[:, None] * np.repeat(s_w, N // g)[None, :])).astype(np.float16)
    assert_bit_equal(host(out), want, "out")
    s_tok = (s_tok * (3.0 / (np.sqrt(K) * 40.0 * float(s_tok.mean()) * float(s_w.mean())))).astype(np.float32)
    res = zq.zq_gemm_gelu_quant_tokenwise(dev(xq), dev(s_tok), dev(wq), dev(s_w), dev(bias), approx_tanh=approx)
    torch.cuda.synchronize()
    _check_fused(orc, *(host(t) for t in res), xq, s_tok, codes, s_w, bias, approx, "vector gelu")


@pytest.mark.parametrize("M", [1, 2, 4])
@pytest.mark.parametrize("bits", [8, 4])
def test_vector_largest_sums(zq, orc, bits, M):
    """The longest K there is, every product of a row with the same sign and at full size: with INT4 weights the accumulators,
    which carry the factor 16, come within 0.01 % of 2^31."""
    if bits == 4 and M > 2:
        pytest.skip("not this kernel")
    N, g = 48, 3
    K = ZQ_MAX_K // 16 * 16 if bits == 8 else ZQ_MAX_K_W4 // 32 * 32
    print("vector largest", bits, M, K, flush=True)
    assert zq.gemm_schedule(M, N, K + (16 if bits == 8 else 32), bits) is None
    assert _kernel(zq, bits, M, N, K) == "vector"
    rng = zq_inputs.rng_for(4, 9200 + M + bits)
    sign = np.where(rng.random((1, K)) < 0.5, -1, 1)
    xq = np.repeat(127 * sign, M, axis=0).astype(np.int8)
    xq[M - 1] = -127                                            # the last token, with the rows of -8 (-127) below: all products +1016
    codes = np.empty((N, K), dtype=np.int8)
    codes[0::3] = 127 * sign if bits == 8 else np.where(sign < 0, -8, 7)
    codes[1::3] = -127 * sign if bits == 8 else np.where(sign < 0, 7, -8)
    codes[2::3] = -127 if bits == 8 else -8
    if bits == 8:
        wq = codes
    else:
        u = codes.astype(np.uint8) & 0xF
        wq = (u[:, 0::2] | (u[:, 1::2] << 4)).astype(np.uint8)
    s_tok, s_w = zq_inputs.random_scales(rng, M, 5e-3, 0.3), zq_inputs.random_scales(rng, g, 1e-8, 1e-7)
    bias = zq_inputs.bias(rng, N)
    res = _run(zq, bits, SIMPLE, xq, s_tok, wq, s_w, bias)
    _check(orc, res, xq, s_tok, codes, s_w, bias, "vector largest sums %d-bit" % bits)
    assert abs(int(host(res[1])[M - 1, 2])) * (1 if bits == 8 else 16) > 0.9998 * 2 ** 31
