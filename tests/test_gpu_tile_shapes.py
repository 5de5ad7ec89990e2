"""GPU parity of every tile shape of the tiled GeMM, at edges in M, N and K, in one round of workgroups and in several.
The shape a call takes follows from its sizes; the sizes below reach all of them (128x64, 128x128, 192x128, 256x128,
256x192, 256x256) for INT8 and INT4 weights and for FP16 activations."""
import pytest
import torch

import zq_inputs
from helpers import dev, host
from test_gpu_gemm import TILE128, TILE256, TILE256X128, TILE256X192, _case, _check, _run, orc, zq  # noqa: F401
from test_gpu_gemm_a16 import _check as _check_a16

pytestmark = pytest.mark.gpu

# (variant, M, N, K, groups)
SHAPES = [
    (TILE128, 129, 80, 1056, 5), (TILE128, 333, 1040, 2080, 65), (TILE128, 200, 64, 32, 4),      # 128x64
    (TILE128, 1300, 3088, 544, 193),                                                             # 128x128
    (TILE256X128, 193, 144, 672, 9), (TILE256X128, 333, 1040, 2080, 65), (TILE256X128, 192, 128, 96, 8),   # 192x128
    (TILE256X128, 2060, 4112, 160, 257),                                                         # 256x128, two rounds
    (TILE256X128, 2048, 4096, 544, 64),                                                          # 256x128, one round
    (TILE256X192, 257, 208, 416, 13), (TILE256, 513, 272, 416, 17),
]


@pytest.mark.parametrize("bits", [8, 4])
@pytest.mark.parametrize("variant,M,N,K,g", SHAPES)
def test_tile_shape_against_oracle(zq, orc, bits, variant, M, N, K, g):
    print("tile shape", variant, bits, M, N, K, g, flush=True)
    xq, s_tok, s_w, bias, codes, wq = _case(zq_inputs.rng_for(4, 6000 + M + N + K + bits), M, N, K, g, bits)
    res = _run(zq, bits, variant, xq, s_tok, wq, s_w, bias)
    _check(orc, res, xq, s_tok, codes, s_w, bias, "tile %d %d-bit %dx%dx%d" % (variant, bits, M, N, K))


# FP16 activations choose among the same shapes (above 64 tokens, K no multiple of 256): 128x64, 192x128, 128x128,
# 256x128, 256x192, 256x256
@pytest.mark.parametrize("M,N,K,g", [(129, 1040, 1040, 65), (333, 8208, 528, 27), (1025, 3088, 272, 193),
                                     (2040, 4112, 400, 257), (2048, 6144, 208, 128), (4080, 4112, 208, 257)])
def test_tile_shape_a16_against_oracle(zq, orc, M, N, K, g):
    print("tile shape a16", M, N, K, g, flush=True)
    rng = zq_inputs.rng_for(9, 6000 + M + N + K)
    x = zq_inputs.activations(rng, M, K, outlier_frac=0.01, outlier_scale=15.0)
    codes = zq_inputs.random_codes(rng, (N, K))
    s_w, bias = zq_inputs.random_scales(rng, g, 1e-4, 1e-2), zq_inputs.bias(rng, N)
    out = zq.zq_gemm_w8a16_dequant(dev(x), dev(codes), dev(s_w), dev(bias))
    torch.cuda.synchronize()
    _check_a16(orc, host(out), x, codes, s_w, bias, "tile a16 %dx%dx%d" % (M, N, K))
