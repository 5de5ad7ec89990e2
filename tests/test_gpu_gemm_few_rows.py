"""GPU parity of the two forms of the direct GeMM kernel for few weight rows: eight tokens by eight rows twice in a matrix
instruction (up to 8 tokens, 2048 rows, K beyond 1024), and activations that are permuted after contiguous loads (12 to 32 tokens, 4096
rows, K a multiple of 256, or of 64 from 2048 on); K of a few values past a half, a stage and a round of them."""
import pytest
import torch

import zq_inputs
from helpers import dev, host
from test_gpu_gemm import SIMPLE, _case, _check, _run, orc, zq  # noqa: F401 (fixtures)
from test_gpu_gemm_a16 import _check as _check_a16

pytestmark = pytest.mark.gpu

# (M, N, K, groups)
SHAPES = [
    (3, 16, 1056, 1), (8, 2048, 1312, 128), (5, 1040, 1536, 65), (7, 272, 2080, 17), (8, 528, 3104, 11), (4, 112, 4128, 7),
    (6, 1616, 4640, 101), (8, 16, 12320, 1),
    (12, 16, 256, 1), (16, 4096, 512, 256), (17, 2064, 1024, 3), (32, 1040, 1280, 13), (27, 400, 2112, 25), (31, 4000, 2304, 250),
    (24, 80, 4160, 5), (13, 272, 6400, 17),
]


@pytest.mark.parametrize("bits", [8, 4])
@pytest.mark.parametrize("M,N,K,g", SHAPES)
def test_few_rows_against_oracle(zq, orc, bits, M, N, K, g):
    print("few rows", bits, M, N, K, g, flush=True)
    xq, s_tok, s_w, bias, codes, wq = _case(zq_inputs.rng_for(4, 9500 + M + N + K + bits), M, N, K, g, bits)
    res = _run(zq, bits, SIMPLE, xq, s_tok, wq, s_w, bias)
    _check(orc, res, xq, s_tok, codes, s_w, bias, "few rows %d-bit %dx%dx%d" % (bits, M, N, K))


@pytest.mark.parametrize("M,N,K,g", [(1, 2048, 1040, 128)] + SHAPES)
def test_few_rows_a16_against_oracle(zq, orc, M, N, K, g):
    """FP16 activations; the values behind the last row's end are not finite, so a load that runs over the end shows.  (Some of
    the shapes stream; those of FORMS do not.)"""
    print("few rows a16", M, N, K, g, zq.gemm_schedule(M, N, K, 8, 0, x_bits=16), flush=True)
    rng = zq_inputs.rng_for(9, 9500 + M + N + K)
    x = zq_inputs.activations(rng, M, K, outlier_frac=0.01, outlier_scale=15.0)
    codes = zq_inputs.random_codes(rng, (N, K))
    s_w, bias = zq_inputs.random_scales(rng, g, 1e-4, 1e-2), zq_inputs.bias(rng, N)
    buf = torch.full((M * K + 4096,), float("nan"), dtype=torch.float16, device="cuda")
    xd = buf[: M * K].view(M, K)
    xd.copy_(dev(x))
    out = zq.zq_gemm_w8a16_dequant(xd, dev(codes), dev(s_w), dev(bias))
    out2 = zq.zq_gemm_w8a16_dequant(xd, dev(codes), dev(s_w), dev(bias))
    torch.cuda.synchronize()
    _check_a16(orc, host(out), x, codes, s_w, bias, "few rows a16 %dx%dx%d" % (M, N, K))
    assert torch.equal(out.view(torch.int16), out2.view(torch.int16))


# (kernel, M, N, K, groups) through the default dispatch, per weight bits; 16: FP16 activations
FORMS = {
    8: [("direct_pairs", 3, 16, 1056, 1), ("direct_pairs", 8, 2048, 1312, 128), ("direct_pairs", 7, 272, 2080, 17),
        ("direct_pairs", 5, 1616, 4640, 101), ("direct_pairs", 8, 16, 12320, 1), ("direct_permuted", 12, 4096, 768, 256),
        ("direct_permuted", 17, 2064, 1024, 3), ("direct_permuted", 32, 1040, 1280, 13), ("direct_permuted", 27, 400, 2176, 25),
        ("direct_permuted", 24, 1024, 3072, 64), ("direct_permuted", 16, 80, 4224, 5)],
    4: [("direct_pairs", 3, 16, 1056, 1), ("direct_pairs", 8, 2048, 1312, 128), ("direct_pairs", 4, 112, 4128, 7),
        ("direct_pairs", 5, 1616, 4640, 101), ("direct_pairs", 8, 16, 12320, 1), ("direct_permuted", 16, 4096, 1024, 256),
        ("direct_permuted", 17, 2064, 1024, 3), ("direct_permuted", 31, 4000, 2304, 250), ("direct_permuted", 27, 400, 2176, 25),
        ("direct_permuted", 13, 272, 6400, 17)],
    16: [("direct_pairs", 1, 2048, 1040, 128), ("direct_pairs", 4, 112, 4128, 7), ("direct_pairs", 8, 2048, 1312, 128),
         ("direct_pairs", 5, 1616, 4640, 101), ("direct_pairs", 8, 16, 12320, 1), ("direct_permuted", 16, 1024, 1024, 64),
         ("direct_permuted", 17, 2064, 1024, 3), ("direct_permuted", 31, 4000, 2112, 250), ("direct_permuted", 13, 272, 4096, 17),
         ("direct_permuted", 24, 80, 4160, 5)],
}


@pytest.mark.parametrize("bits,kernel,M,N,K,g", [(b,) + c for b in (8, 4, 16) for c in FORMS[b]])
def test_every_form_is_reached(zq, orc, bits, kernel, M, N, K, g):
    assert zq.gemm_kernel(M, N, K, 4 if bits == 4 else 8, 0, x_bits=16 if bits == 16 else 8) == kernel
    if bits == 16:
        test_few_rows_a16_against_oracle(zq, orc, M, N, K, g)
        return
    print("form", kernel, bits, M, N, K, g, flush=True)
    xq, s_tok, s_w, bias, codes, wq = _case(zq_inputs.rng_for(4, 9700 + M + N + K + bits), M, N, K, g, bits)
    res = _run(zq, bits, -1, xq, s_tok, wq, s_w, bias)
    _check(orc, res, xq, s_tok, codes, s_w, bias, "%s %d-bit %dx%dx%d" % (kernel, bits, M, N, K))
