"""GPU parity of the small-tile GeMM kernel (33 to some hundred tokens) at the sizes where it can go wrong: one token and
one strip over and short of a tile, each of its tiles at the most workgroups it takes, K of fewer stages than waves, a
last round of stages that is partly empty, K tails of one load, and the automatic choice around its limits."""
import pytest
import torch

import zq_inputs
from helpers import dev, host
from test_gpu_gemm import SIMPLE, _case, _check, _run, orc, zq  # noqa: F401 (fixtures)
from test_gpu_gemm_a16 import _check as _check_a16

pytestmark = pytest.mark.gpu

# (M, N, K, groups)
SHAPES = [
    (33, 272, 32, 17), (64, 8192, 288, 8), (65, 5104, 1056, 29), (129, 2032, 544, 127), (63, 8208, 2080, 27),
    (128, 4096, 3104, 16), (250, 4112, 672, 1), (257, 3216, 1312, 67), (1024, 1024, 800, 2), (40, 16384, 160, 256),
    (97, 784, 6656, 49),
]
EDGES = [(64, 4096, 4096, 4), (64, 4112, 4096, 1), (65, 2048, 2048, 8), (128, 1024, 4096, 4), (192, 2048, 6656, 2)]


@pytest.mark.parametrize("forced", [SIMPLE, -1])
@pytest.mark.parametrize("bits", [8, 4])
@pytest.mark.parametrize("M,N,K,g", SHAPES + EDGES)
def test_small_tiles_against_oracle(zq, orc, bits, M, N, K, g, forced):
    print("mid", bits, M, N, K, g, forced, flush=True)
    xq, s_tok, s_w, bias, codes, wq = _case(zq_inputs.rng_for(4, 7000 + M + N + K + bits), M, N, K, g, bits)
    res = _run(zq, bits, forced, xq, s_tok, wq, s_w, bias)
    _check(orc, res, xq, s_tok, codes, s_w, bias, "small tiles %d-bit %dx%dx%d" % (bits, M, N, K))


@pytest.mark.parametrize("M,N,K,g", SHAPES + EDGES)
def test_small_tiles_a16_against_oracle(zq, orc, M, N, K, g):
    """FP16 activations; the values behind the last row's end are not finite, so a load that runs over the end shows."""
    print("mid a16", M, N, K, g, flush=True)
    rng = zq_inputs.rng_for(9, 7000 + M + N + K)
    x = zq_inputs.activations(rng, M, K, outlier_frac=0.01, outlier_scale=15.0)
    codes = zq_inputs.random_codes(rng, (N, K))
    s_w, bias = zq_inputs.random_scales(rng, g, 1e-4, 1e-2), zq_inputs.bias(rng, N)
    buf = torch.full((M * K + 4096,), float("nan"), dtype=torch.float16, device="cuda")
    xd = buf[: M * K].view(M, K)
    xd.copy_(dev(x))
    out = zq.zq_gemm_w8a16_dequant(xd, dev(codes), dev(s_w), dev(bias))
    out2 = zq.zq_gemm_w8a16_dequant(xd, dev(codes), dev(s_w), dev(bias))
    torch.cuda.synchronize()
    _check_a16(orc, host(out), x, codes, s_w, bias, "small tiles a16 %dx%dx%d" % (M, N, K))
    assert torch.equal(out.view(torch.int16), out2.view(torch.int16))


# both depths of the 32 x 32 and 64 x 32 tiles: INT4 from four stages a wave on, INT8 on 64 x 32 from six; two tiles of
# 32 x 32 on every compute unit
DEPTHS = [(40, 272, 4096, 17), (40, 272, 5152, 17), (100, 1040, 8192, 65), (245, 784, 6208, 7), (245, 1536, 5152, 96), (390, 768, 3104, 48),
          (36, 16384, 1024, 64), (70, 8208, 544, 27), (120, 4112, 1056, 257), (36, 8192, 1024, 64)]


@pytest.mark.parametrize("bits", [8, 4])
@pytest.mark.parametrize("M,N,K,g", DEPTHS)
def test_small_tile_depths(zq, orc, bits, M, N, K, g):
    test_small_tiles_against_oracle(zq, orc, bits, M, N, K, g, SIMPLE)


# INT4, more than one 32 x 32 tile per compute unit: four waves with two stages in flight; K of a stage, of fewer than waves, of
# an odd and an even count of stages a wave, with a tail of 32 values
@pytest.mark.parametrize("M,N,K,g", [(65, 2768, 32, 173), (80, 5136, 416, 107), (72, 4608, 1056, 96), (96, 4112, 1536, 257),
                                     (70, 4112, 2080, 257), (80, 5440, 3104, 10), (66, 4112, 5120, 257)])
def test_int4_on_four_waves(zq, orc, M, N, K, g):
    before = zq.force_gemm_variant(SIMPLE)
    try:
        assert zq.gemm_kernel(M, N, K, 4) == "small32x32_4waves"
    finally:
        zq.force_gemm_variant(before)
    test_small_tiles_against_oracle(zq, orc, 4, M, N, K, g, SIMPLE)
