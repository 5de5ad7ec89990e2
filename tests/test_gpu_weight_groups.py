"""GPU parity of the one-pass group-wise weight quantizer, bit for bit, at the sizes where it can go wrong: a group of one
slice, exactly full and one vector over, each number of vectors per thread, a short last slice, the most slices and one
more than that, both sides of the line to the two-pass quantizer, with and without waiting for the other slices of a
group, and in a replayed graph."""
import numpy as np
import pytest
import torch

import zq_inputs
from helpers import assert_bit_equal, dev, host

pytestmark = pytest.mark.gpu

# (N, K, groups); a slice holds at most 32768 weights
SHAPES = [
    (32, 512, 2), (48, 544, 3), (16, 1024, 1), (32, 1056, 2),       # one slice, up to 4 / 8 / 16 vectors per thread
    (64, 2048, 4), (64, 2080, 4),                                   # exactly full; a second slice
    (16, 4096, 1), (48, 8192, 3), (64, 4096, 4), (512, 2080, 1),                    # 2, 3 x 4, 4 x 2, 33 slices
    (4096, 3328, 2), (3328, 4096, 2), (6656, 4096, 4), (7680, 4096, 4), (5040, 3584, 7),  # 2 x 208; 4 x 208, 240; 7 x 79
    (6400, 1600, 100), (4800, 2080, 300), (4096, 4096, 16),
    (4080, 2048, 1), (4096, 2048, 1), (8160, 2048, 2),              # 255 slices; 256: read twice; 2 x 255
]


@pytest.fixture(scope="module")
def zq():
    import paper_2206_01861_amd as z
    z.lib()
    return z


@pytest.fixture(scope="module")
def orc():
    from oracle import zq_oracle
    return zq_oracle


def _weights(N, K, g, seed):
    """Groups whose largest value stands first, last, in the middle or nowhere (all zero), in turn."""
    w = zq_inputs.weights(zq_inputs.rng_for(1, seed), N, K)
    flat = w.reshape(g, -1)
    for i in range(g):
        if i % 4 == 3:
            flat[i] = 0
        else:
            at = (0, flat.shape[1] - 1, flat.shape[1] // 2)[i % 4]
            flat[i, at] = np.float16(-3.0 - 0.25 * (i % 7))
    return w


@pytest.mark.parametrize("wait", [True, False])
@pytest.mark.parametrize("bits", [8, 4])
@pytest.mark.parametrize("N,K,g", SHAPES)
def test_weight_groups_bit_exact(zq, orc, bits, N, K, g, wait):
    print("weight groups", bits, N, K, g, wait, flush=True)
    w = _weights(N, K, g, 500 + N + K + g)
    wq_o, s_o, _ = orc.quantize_weight_groupwise(w, g, bits)
    wd = dev(w)
    before = zq.set_in_kernel_quant(wait)
    try:
        got = [zq.zq_quantize_weight_groupwise(wd, g, bits) for _ in range(3)]
    finally:
        zq.set_in_kernel_quant(before)
    for wq, s_w in got:
        assert_bit_equal(host(s_w), s_o, "s_w")
        assert_bit_equal(host(wq), wq_o, "wq")


@pytest.mark.parametrize("bits", [8, 4])
def test_weight_groups_in_a_replayed_graph(zq, orc, bits):
    N, K, g = 1600, 2080, 20
    print("weight groups graph", bits, flush=True)
    wd = dev(_weights(N, K, g, 1))
    zq.zq_quantize_weight_groupwise(wd, g, bits)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        wq, s_w = zq.zq_quantize_weight_groupwise(wd, g, bits)
    for seed in range(2, 5):
        w = _weights(N, K, g, seed)
        wd.copy_(dev(w))
        graph.replay()
        torch.cuda.synchronize()
        wq_o, s_o, _ = orc.quantize_weight_groupwise(w, g, bits)
        assert_bit_equal(host(s_w), s_o, "s_w")
        assert_bit_equal(host(wq), wq_o, "wq")
