"""The binding's native calls (_zq_host) against its ctypes path: the same tensors out of the same calls, on torch's current
stream, and the same errors."""
import pytest
import torch

from test_gpu_quant import zq  # noqa: F401 (fixture)

pytestmark = pytest.mark.gpu


@pytest.fixture()
def calls(zq):
    gen = torch.Generator(device="cuda").manual_seed(5)
    rnd = lambda *s: torch.randn(s, generator=gen, device="cuda").half()
    M, N, K, g = 70, 1024, 512, 16
    x, w, gamma, beta, bias = rnd(M, K), rnd(N, K), rnd(K), rnd(K), rnd(N)
    ws = zq.new_workspace(max(zq.gemm_quant_workspace_bytes(M, N, K, b) for b in (8, 4)))
    xq, st, _ = zq.zq_layernorm_quant_tokenwise(x, gamma, beta, 1e-5)
    w8, s8 = zq.zq_quantize_weight_groupwise(w, g, 8)
    w4, s4 = zq.zq_quantize_weight_groupwise(w, g, 4)
    out = [lambda b=b: zq.zq_quantize_weight_groupwise(w, g, b) for b in (8, 4)]
    out += [lambda y=y, p=p: zq.zq_layernorm_quant_tokenwise(x, torch.nn.Parameter(gamma), p, 1e-5, y_dtype=y)
            for y in (None, torch.float16, torch.float32) for p in (beta, None)]
    out += [lambda y=y, p=p, t=t: zq.zq_gelu_quant_tokenwise(x, p, approx_tanh=t, y_dtype=y)
            for y in (None, torch.float16, torch.float32) for p in (gamma, None) for t in (False, True)]
    out += [lambda: zq.zq_quantize_tokenwise(x), lambda: zq.zq_gemm_w8a16_dequant(x, w8, s8, bias, workspace=ws),
            lambda: zq.zq_gemm_w8a16_dequant(x, w8, s8)]
    for call, wq, sw in ((zq.zq_gemm_i8_dequant, w8, s8), (zq.zq_gemm_w4a8_dequant, w4, s4)):
        out += [lambda c=call, a=(xq, st, wq, sw), p=p, r=r, s=s: c(*a, p, requant=r, workspace=s)
                for p in (bias, None) for r in (False, True) for s in (ws, None)]
        out += [lambda a=(xq, st, wq, sw), t=t, k=k: zq.zq_gemm_gelu_quant_tokenwise(*a, bias, approx_tanh=t, workspace=ws if not k else None,
                                                                                    keep_g=k)
                for t in (False, True) for k in ((True, False) if zq.gemm_quantizes_in_kernel(M, N, K, 8, ws.numel()) else (True,))]
    return out


def _flat(r):
    return r if isinstance(r, tuple) else (r,)


def test_native_calls_equal_the_ctypes_path(zq, calls, monkeypatch):
    from paper_2206_01861_amd import binding
    native = binding._host
    taken = []

    class Spy:
        def __getattr__(self, name):
            def call(*args):
                r = getattr(native, name)(*args)
                taken.append(r is not None)
                return r
            return call
    side = torch.cuda.Stream()
    for i, call in enumerate(calls):
        monkeypatch.setattr(binding, "_host", Spy())
        side.wait_stream(torch.cuda.current_stream())
        with torch.cuda.stream(side):
            got = _flat(call())
        side.synchronize()
        assert taken == [True] * (i + 1), i
        monkeypatch.setattr(binding, "_host", None)
        want = _flat(call())
        assert len(got) == len(want)
        for a, b in zip(got, want):
            assert (a is None) == (b is None)
            if a is not None:
                assert a.dtype == b.dtype and a.shape == b.shape and torch.equal(a, b), i


def test_native_calls_leave_the_errors_to_the_ctypes_path(zq):
    x = torch.zeros((4, 64), dtype=torch.float16, device="cuda")
    xq, st = zq.zq_quantize_tokenwise(x)
    wq, sw = zq.zq_quantize_weight_groupwise(torch.zeros((32, 64), dtype=torch.float16, device="cuda"), 2, 8)
    with pytest.raises(TypeError):
        zq.zq_quantize_tokenwise(x.float())
    with pytest.raises(TypeError):
        zq.zq_quantize_tokenwise(torch.zeros((64, 4), dtype=torch.float16, device="cuda").t())
    with pytest.raises(TypeError):
        zq.zq_layernorm_quant_tokenwise(x, None, None, 1e-5)
    with pytest.raises(TypeError):
        zq.zq_layernorm_quant_tokenwise(x, x[0], None, 1e-5, y_dtype=torch.int8)
    with pytest.raises(ValueError):
        zq.zq_gemm_i8_dequant(xq, st, wq[:, :32].contiguous(), sw)
    with pytest.raises(ValueError):
        zq.zq_gemm_i8_dequant(xq, st[:3], wq, sw)
    with pytest.raises(ValueError):
        zq.zq_gemm_i8_dequant(xq, st, wq, sw, torch.zeros(16, dtype=torch.float16, device="cuda"))
    for bad in (lambda: zq.zq_gemm_i8_dequant(xq, st, wq, sw[:1].expand(3).contiguous()),
                lambda: zq.zq_layernorm_quant_tokenwise(x, x[0], None, -1.0),
                lambda: zq.zq_quantize_tokenwise(torch.zeros((4, 24), dtype=torch.float16, device="cuda")),
                lambda: zq.zq_quantize_weight_groupwise(torch.zeros((32, 64), dtype=torch.float16, device="cuda"), 3, 8)):
        with pytest.raises(zq.ZQError):
            bad()
    # integers where floats and truth values are usual go the other way, with the same result
    a = zq.zq_layernorm_quant_tokenwise(x, x[0], None, 1)
    b = zq.zq_layernorm_quant_tokenwise(x, x[0], None, 1.0)
    assert torch.equal(a[0], b[0])
