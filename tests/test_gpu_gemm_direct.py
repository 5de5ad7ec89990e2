"""GPU parity of the direct GeMM kernel (K divided over the waves of a workgroup) at the sizes where it can go wrong:
token tiles and weight strips that are full, one over and one short, K tails of one 16-byte load, fewer stages than
waves, a last round of stages that is partly empty, more token tiles than a workgroup holds."""
import pytest
import torch

import zq_inputs
from helpers import dev, host
from test_gpu_gemm import SIMPLE, _case, _check, _run, orc, zq  # noqa: F401 (fixtures)
from test_gpu_gemm_a16 import _check as _check_a16

pytestmark = pytest.mark.gpu

# (M, N, K, groups)
SHAPES = [
    (1, 16, 16, 1), (8, 2048, 32, 8), (9, 4112, 272, 257), (16, 6160, 2080, 35), (17, 8208, 1056, 27),
    (32, 1616, 4128, 101), (33, 2064, 1312, 3), (64, 400, 2592, 25), (5, 8192, 2048, 128), (3, 10256, 544, 1),
    (4, 2064, 4096, 3), (65, 1040, 800, 65), (144, 272, 1024, 17), (200, 784, 160, 49),
]


@pytest.mark.parametrize("bits", [8, 4])
@pytest.mark.parametrize("M,N,K,g", SHAPES)
def test_direct_against_oracle(zq, orc, bits, M, N, K, g):
    if bits == 4 and K % 32:
        pytest.skip("INT4 needs K % 32 == 0")
    print("direct", bits, M, N, K, g, flush=True)
    xq, s_tok, s_w, bias, codes, wq = _case(zq_inputs.rng_for(4, 5000 + M + N + K + bits), M, N, K, g, bits)
    res = _run(zq, bits, SIMPLE, xq, s_tok, wq, s_w, bias)
    _check(orc, res, xq, s_tok, codes, s_w, bias, "direct %d-bit %dx%dx%d" % (bits, M, N, K))


@pytest.mark.parametrize("M,N,K,g", [s for s in SHAPES if s[0] <= 64])
def test_direct_a16_against_oracle(zq, orc, M, N, K, g):
    """FP16 activations on the same kernel (K no multiple of 256, or few tokens); the values behind the last row's end
    are not finite, so an activation load that runs over the end shows."""
    print("direct a16", M, N, K, g, flush=True)
    rng = zq_inputs.rng_for(9, 5000 + M + N + K)
    x = zq_inputs.activations(rng, M, K, outlier_frac=0.01, outlier_scale=15.0)
    codes = zq_inputs.random_codes(rng, (N, K))
    s_w, bias = zq_inputs.random_scales(rng, g, 1e-4, 1e-2), zq_inputs.bias(rng, N)
    buf = torch.full((M * K + 4096,), float("nan"), dtype=torch.float16, device="cuda")
    xd = buf[: M * K].view(M, K)
    xd.copy_(dev(x))
    out = zq.zq_gemm_w8a16_dequant(xd, dev(codes), dev(s_w), dev(bias))
    out2 = zq.zq_gemm_w8a16_dequant(xd, dev(codes), dev(s_w), dev(bias))
    torch.cuda.synchronize()
    _check_a16(orc, host(out), x, codes, s_w, bias, "direct a16 %dx%dx%d" % (M, N, K))
    assert torch.equal(out.view(torch.int16), out2.view(torch.int16))
