"""The native call path of the binding against the checks in Python: the same results,
and the same refusals, for calls that it takes, leaves to Python, or must refuse."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


class _PythonOnly:
    """A binding that takes no call."""

    def __getattr__(self, name):
        return lambda *a: None


def _both(fa, monkeypatch, call):
    """(result or exception type and text) through the native path and through Python."""
    got = []
    native = fa.api._binding
    for binding in (native, _PythonOnly()):
        monkeypatch.setattr(fa.api, "_binding", binding)
        try:
            r = call()
            torch.cuda.synchronize()
            got.append(r)
        except Exception as e:   # noqa: BLE001 - the type and the text are compared
            got.append((type(e), str(e)))
    monkeypatch.setattr(fa.api, "_binding", native)
    return got


def _same(a, b):
    if isinstance(a, torch.Tensor):
        return isinstance(b, torch.Tensor) and a.dtype == b.dtype and torch.equal(a, b)
    if isinstance(a, tuple) and a and isinstance(a[0], torch.Tensor):
        return len(a) == len(b) and all(_same(x, y) for x, y in zip(a, b))
    return a == b


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
def test_native_calls_equal_the_python_path(monkeypatch, dtype):
    import paper_2609_04105_amd as fa
    g = torch.Generator(device="cuda").manual_seed(3)
    q, k, v = (torch.randn((2, 3, 256, 64), device="cuda", generator=g).to(dtype) for _ in range(3))
    plain, anchored, fp8 = (fa.quantize_qkv(q, k, v, **o) for o in ({}, {"anchored": True}, {"pv_fp8": True}))
    lse = torch.empty((2, 3, 256), device="cuda")
    out32, out16 = (torch.empty((2, 3, 256, 64), device="cuda", dtype=t) for t in (torch.float32, torch.bfloat16))
    odd = torch.empty(lse.numel() + 1, device="cuda")[1:].view_as(lse)          # not 16-byte aligned
    bad = plain[0][:, :, :128].contiguous()
    calls = [
        lambda: fa.quantize_qkv(q, k, v), lambda: fa.quantize_qkv(q, k, v, anchored=True),
        lambda: fa.quantize_qkv(q, k, v, pv_fp8=True), lambda: fa.quantize_qkv(q[0], k[0], v[0]),
        lambda: fa.quantize_qkv(q, k[:, :, :128].contiguous(), v), lambda: fa.quantize_qkv(q, k, v, anchored=1),
        lambda: fa.forward_mxfp4(*plain), lambda: fa.forward_mxfp4(*plain, out=out32),
        lambda: fa.forward_mxfp4(*plain, out=out16), lambda: fa.forward_mxfp4(*plain, out_dtype=torch.bfloat16),
        lambda: fa.forward_mxfp4(*plain, softmax_scale=0.2, affine_a=1.6, affine_b=0.95),
        lambda: fa.forward_mxfp4(*plain, softmax_scale=1), lambda: fa.forward_mxfp4(*plain, softmax_scale=np.float64(0.3)),
        lambda: fa.forward_mxfp4(*plain, causal=True, lse=lse), lambda: lse.clone(),
        lambda: fa.forward_mxfp4(*plain, ex2_pairs=4), lambda: fa.forward_mxfp4(*anchored, guard=(110, 16)),
        lambda: fa.forward_mxfp4(*fp8, pv_fp8=True), lambda: fa.forward_mxfp4(*plain, causal=1),
        lambda: fa.attention_mxfp4(q, k, v), lambda: fa.attention_mxfp4(q, k, v, guard=(110, 16), out=out16),
        lambda: fa.attention_mxfp4(q, k, v, pv_fp8=True, causal=True, lse=lse), lambda: lse.clone(),
        lambda: fa.attention_mxfp4(q, k, v, ex2_pairs=16, out_dtype=torch.bfloat16),
        lambda: fa.forward_bf16(q, k, v), lambda: fa.forward_bf16(q, k, v, softmax_scale=0.1, out=out16),
        lambda: fa.attention_mxfp4(q.requires_grad_(), k, v).requires_grad,
        # refused
        lambda: fa.forward_mxfp4(bad, *plain[1:]), lambda: fa.forward_mxfp4(plain[0].float(), *plain[1:]),
        lambda: fa.forward_mxfp4(*plain, out=out32[:, :, :128]), lambda: fa.forward_mxfp4(*plain, out=out32.double()),
        lambda: fa.forward_mxfp4(*plain, softmax_scale=-1.0), lambda: fa.forward_mxfp4(*plain, ex2_pairs=3),
        lambda: fa.forward_mxfp4(*plain, guard=(120, 16)), lambda: fa.forward_mxfp4(*plain, guard=(1, 2, 3)),
        lambda: fa.forward_mxfp4(*plain, lse=lse[:1]), lambda: fa.forward_mxfp4(*plain, lse=odd),
        lambda: fa.forward_mxfp4(*plain, pv_fp8=True), lambda: fa.forward_mxfp4(*plain, causal=True, ex2_pairs=2),
        lambda: fa.forward_mxfp4(*plain, out_dtype=torch.float16), lambda: fa.forward_mxfp4(*(t.cpu() for t in plain)),
        lambda: fa.attention_mxfp4(q, k, v, guard=(110, 16), pv_fp8=True), lambda: fa.attention_mxfp4(q, k, 5),
        lambda: fa.attention_mxfp4(q[:, :, :200].contiguous(), k, v),
        lambda: fa.attention_mxfp4(*(t[:, :, :192].contiguous() for t in (q, k, v))),
        lambda: fa.attention_mxfp4(q.transpose(1, 2), k, v), lambda: fa.forward_bf16(q, k[:1], v),
        lambda: fa.quantize_qkv(q, k, v, anchored=True, pv_fp8=True),
    ]
    for i, call in enumerate(calls):
        a, b = _both(fa, monkeypatch, call)
        assert _same(a, b), f"call {i}: {a} through the native path, {b} through Python"


def test_current_stream_and_replay(monkeypatch):
    """A call on another stream runs there, and a captured call replays."""
    import paper_2609_04105_amd as fa
    g = torch.Generator(device="cuda").manual_seed(4)
    q, k, v = (torch.randn((1, 2, 512, 128), device="cuda", generator=g).to(torch.bfloat16) for _ in range(3))
    want = fa.attention_mxfp4(q, k, v)
    s = torch.cuda.Stream()
    s.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(s):
        got = fa.attention_mxfp4(q, k, v)
    s.synchronize()
    assert torch.equal(got, want)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        got = fa.attention_mxfp4(q, k, v)
    for i in range(3):
        q.copy_(torch.randn(q.shape, device="cuda", generator=g))
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(got, fa.attention_mxfp4(q, k, v)), f"replay {i}"
