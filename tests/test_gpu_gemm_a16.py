"""GPU parity of the W8A16 GeMM (FP16 activations x group-wise INT8 weights, Sec. 5) against the
fp64 oracle, through the C ABI.  Accumulation is fp32 on the matrix cores, so the bar is the FP16
tolerance of the task (2e-3 of the terms' magnitude) plus the fp32 accumulation bound."""
import numpy as np
import pytest
import torch

import zq_inputs
from helpers import dev, host
from test_gpu_gemm import orc, zq  # noqa: F401 (fixtures)

pytestmark = pytest.mark.gpu


def _check(orc, out16, x, codes, s_w, bias, what, rows=None):
    K = x.shape[1]
    acc, absacc = orc.matmul_f16_i8(x, codes, rows=rows)
    ref, mag = orc.dequant_w(acc, s_w, bias)
    gs = codes.shape[0] // s_w.size
    sw_col = np.repeat(s_w.astype(np.float64), gs)[None, :]
    # one FP16 rounding of the result (4.9e-4 relative, inside the task's 2e-3), and at most one fp32
    # rounding per 16-deep matrix-core step on partial sums no larger than the sum of |products|
    tol = 2e-3 * mag + (K / 16 + 8) * 2.0 ** -24 * absacc * sw_col + 2.0 ** -25
    got = out16.astype(np.float64) if rows is None else out16[rows].astype(np.float64)
    err = np.abs(got - ref)
    assert (err <= tol).all(), "%s: %d bad, worst err %.3e at tol %.3e" % (
        what, int((err > tol).sum()), err.max(), tol[np.unravel_index(err.argmax(), err.shape)])
    # the accumulation term must not be what makes the test pass: typical error is far below it
    assert np.median(err / np.maximum(mag, 1e-30)) < 5e-4, what


SHAPES = [
    # (M, N, K, groups): few tokens or few rows, K of one load to many stages ...
    (1, 16, 16, 1), (17, 768, 784, 48), (129, 96, 1024, 2), (70, 272, 208, 17),
    (1, 64, 256, 4), (8, 6144, 2048, 128), (33, 144, 1792, 9), (64, 1024, 1536, 64), (16, 33040, 512, 5),
    (50, 16, 256, 1),
    # ... some hundred tokens and more, ragged edges, K not a multiple of the stage depth ...
    (300, 400, 384, 25), (515, 1024, 1024, 64), (129, 272, 2048, 17), (2500, 4112, 512, 257),
    (515, 1024, 400, 64), (300, 1040, 1008, 65),
    (2300, 7152, 336, 3),                              # 256x256 tiles (one round of 252), ragged in M, N and K
    # ... a long K
    (32, 2048, 8192, 128), (7, 528, 24576, 11), (64, 4112, 16384, 1), (1, 2048, 8192, 128),
    (130, 1024, 4096, 64), (300, 400, 2048, 25), (256, 2064, 2000, 3), (129, 272, 8192, 17),
    # 65 to 128 tokens
    (65, 1024, 1536, 64), (100, 6144, 2048, 128), (128, 2064, 512, 3), (90, 2048, 8192, 128), (128, 528, 24576, 11),
]
# (schedule, workspace, M, N, K, groups); the workspace is the one that is asked for, none, or the streaming K split's only
ROUTES = [
    # the streaming schedule, one to four token tiles, uneven strips ...
    ("stream", "asked", 2, 6576, 2816, 137), ("stream", "asked", 12, 544, 5632, 2), ("stream", "asked", 31, 528, 4352, 11),
    ("stream", "asked", 60, 1040, 3584, 13), ("stream", "asked", 50, 4112, 2304, 1), ("stream", "none", 24, 144, 9728, 9),
    # ... and with a K split (fp32 partials, added in the order of K)
    ("stream_splitk", "asked", 11, 272, 9728, 17), ("stream_splitk", "asked", 27, 272, 5888, 1),
    ("stream_splitk", "asked", 44, 528, 12032, 11),
    # 65 to 128 tokens: two streaming launches over row halves (second half one row, ragged, full), also with a K split
    ("stream_halves", "asked", 65, 19088, 768, 1193), ("stream_halves", "asked", 98, 12384, 768, 3),
    ("stream_halves", "none", 128, 528, 9728, 33), ("stream_splitk_halves", "stream", 90, 2048, 8192, 128),
    ("stream_splitk_halves", "stream", 65, 528, 24576, 11),
    # the tiled schedule that splits K over workgroups (fp32 partials, second kernel)
    ("tile128x128_splitk", "asked", 101, 528, 9728, 11), ("tile128x128_splitk", "asked", 245, 400, 5728, 25),
    ("tile128x128_splitk", "asked", 129, 2064, 8192, 3), ("tile128x128_splitk", "asked", 300, 1024, 6000, 64),
]


@pytest.mark.parametrize("M,N,K,g", SHAPES)
def test_w8a16_against_oracle(zq, orc, M, N, K, g):
    _against_oracle(zq, orc, M, N, K, g, zq.gemm_w8a16_workspace_bytes(M, N, K))


@pytest.mark.parametrize("name,workspace,M,N,K,g", ROUTES)
def test_w8a16_reaches(zq, orc, name, workspace, M, N, K, g):
    nbytes = {"asked": zq.gemm_w8a16_workspace_bytes(M, N, K), "none": 0,
              "stream": zq.gemm_w8a16_workspace_bytes(64, N, K)}[workspace]
    assert zq.gemm_schedule(M, N, K, 8, nbytes, x_bits=16) == name
    _against_oracle(zq, orc, M, N, K, g, nbytes)


def _against_oracle(zq, orc, M, N, K, g, nbytes):
    print("w8a16", M, N, K, g, zq.gemm_schedule(M, N, K, 8, nbytes, x_bits=16), flush=True)
    rng = zq_inputs.rng_for(9, M + N + K)
    x = zq_inputs.activations(rng, M, K, outlier_frac=0.01, outlier_scale=15.0)
    codes = zq_inputs.random_codes(rng, (N, K))
    s_w = zq_inputs.random_scales(rng, g, 1e-4, 1e-2)
    bias = zq_inputs.bias(rng, N)
    ws = zq.new_workspace(nbytes)
    out = zq.zq_gemm_w8a16_dequant(dev(x), dev(codes), dev(s_w), dev(bias), workspace=ws)
    out2 = zq.zq_gemm_w8a16_dequant(dev(x), dev(codes), dev(s_w), dev(bias), workspace=ws)
    torch.cuda.synchronize()
    _check(orc, host(out), x, codes, s_w, bias, "w8a16 %dx%dx%d" % (M, N, K))
    assert torch.equal(out.view(torch.int16), out2.view(torch.int16)), "result depends on arrival order"
    # without a workspace (no K split) and without bias
    out3 = zq.zq_gemm_w8a16_dequant(dev(x), dev(codes), dev(s_w), None)
    torch.cuda.synchronize()
    _check(orc, host(out3), x, codes, s_w, None, "w8a16 no ws/bias %dx%dx%d" % (M, N, K))


def test_w8a16_integer_inputs_are_exact(zq, orc):
    """Integer-valued activations make every partial sum an integer below 2^24: fp32 accumulation is
    exact, so the result equals the INT8 x INT8 product dequantized with unit token scales."""
    rng = zq_inputs.rng_for(9, 4)
    M, N, K, g = 24, 256, 768, 16
    xq = zq_inputs.random_codes(rng, (M, K))
    codes = zq_inputs.random_codes(rng, (N, K))
    s_w = np.full(g, 2.0 ** -12, np.float32)
    out = zq.zq_gemm_w8a16_dequant(dev(xq.astype(np.float16)), dev(codes), dev(s_w), None)
    torch.cuda.synchronize()
    acc = orc.matmul_i32(xq, codes).astype(np.float64)
    assert np.abs(acc).max() < 2 ** 24
    want = (acc * 2.0 ** -12).astype(np.float16)          # one rounding, as the kernel does
    assert np.array_equal(host(out).view(np.uint16), want.view(np.uint16))


@pytest.mark.parametrize("name,M", [("c5_qkv", 64), ("c4_qkv", 16), ("c4_qkv", 128), ("c3_qkv", 1), ("c3_qkv", 2048), ("c4_qkv", 4096)])
def test_w8a16_full_size_sampled_rows(zq, orc, name, M):
    """QKV linears at workload size in the launch configuration the benchmark times; sampled rows."""
    K, N, g, bits = zq_inputs.LINEARS[name]
    gen = torch.Generator(device="cuda").manual_seed(99)
    x = (torch.randn((M, K), generator=gen, device="cuda") *
         torch.exp(torch.empty((M, 1), device="cuda").uniform_(-0.7, 0.7, generator=gen))).half()
    codes = torch.randint(-127, 128, (N, K), generator=gen, device="cuda", dtype=torch.int8)
    s_w = (torch.rand(g, generator=gen, device="cuda") * 1e-3 + 1e-4)
    bias = (torch.randn(N, generator=gen, device="cuda") * 0.01).half()
    nbytes = zq.gemm_w8a16_workspace_bytes(M, N, K)
    ws = zq.new_workspace(nbytes)
    out = zq.zq_gemm_w8a16_dequant(x, codes, s_w, bias, workspace=ws)
    torch.cuda.synchronize()
    rows = sorted(set([0, M - 1, M // 2, min(M - 1, 15), min(M - 1, 16), min(M - 1, 255), min(M - 1, 256)]))
    _check(orc, host(out), host(x), host(codes), host(s_w), host(bias), "w8a16 %s M=%d" % (name, M), rows=rows)
