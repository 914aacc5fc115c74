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


class _Watched:
    """The native binding, recording whether its last call took the arguments."""

    def __init__(self, native):
        self.native, self.took = native, None

    def __getattr__(self, name):
        def call(*a):
            r = getattr(self.native, name)(*a)
            self.took = r is not None
            return r
        return call


class _Refused(tuple):
    """An exception's type and text."""


def _outcome(call, buffers):
    """The call's result and the caller's buffers after it (copies; the buffers are NaN
    before), or the exception."""
    for t in buffers:
        t.fill_(float("nan"))
    try:
        r = call()
        torch.cuda.synchronize()
    except Exception as e:   # noqa: BLE001 - the type and the text are compared
        return _Refused((type(e), str(e)))
    parts = r if isinstance(r, tuple) else (r,)
    owner = [next((i for i, b in enumerate(buffers) if b is t), None) for t in parts]   # the caller's own tensor
    return owner, [t.requires_grad for t in parts], [t.detach().clone() for t in (*parts, *buffers)]


def _same(a, b):
    if isinstance(a, _Refused) or isinstance(b, _Refused):
        return type(a) is type(b) and a == b
    same = [x.dtype == y.dtype and x.shape == y.shape and torch.equal(x.nan_to_num(nan=12345.0), y.nan_to_num(nan=12345.0))
            if x.is_floating_point() else x.dtype == y.dtype and torch.equal(x, y) for x, y in zip(a[2], b[2])]
    return a[:2] == b[:2] and len(a[2]) == len(b[2]) and all(same)


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
def test_native_calls_equal_the_python_path(monkeypatch, dtype):
    """Calls that the native path takes, calls that it leaves to Python and calls that are
    refused: the same results in the same tensors, the same exceptions, through both."""
    import paper_2609_04105_amd as fa
    g = torch.Generator(device="cuda").manual_seed(3)
    q, k, v = (torch.randn((2, 3, 256, 64), device="cuda", generator=g).to(dtype) for _ in range(3))
    grad = q.clone().requires_grad_()
    plain, anchored, fp8 = (fa.quantize_qkv(q, k, v, **o) for o in ({}, {"anchored": True}, {"pv_fp8": True}))
    lse = torch.empty((2, 3, 256), device="cuda")
    out32, out16 = (torch.empty((2, 3, 256, 64), device="cuda", dtype=t) for t in (torch.float32, torch.bfloat16))
    odd = torch.empty(lse.numel() + 1, device="cuda")[1:].view_as(lse)          # not 16-byte aligned
    bad = plain[0][:, :, :128].contiguous()
    bf16 = [lambda: fa.forward_bf16(q, k, v), lambda: fa.forward_bf16(q, k, v, softmax_scale=0.1, out=out16),
            lambda: fa.forward_bf16(q, k, v, out=out32)]
    taken = [
        lambda: fa.quantize_qkv(q, k, v), lambda: fa.quantize_qkv(q, k, v, anchored=True),
        lambda: fa.quantize_qkv(q, k, v, pv_fp8=True), lambda: fa.quantize_qkv(q[0], k[0], v[0]),
        lambda: fa.forward_mxfp4(*plain), lambda: fa.forward_mxfp4(*plain, out=out32),
        lambda: fa.forward_mxfp4(*plain, out=out16), lambda: fa.forward_mxfp4(*plain, out_dtype=torch.bfloat16),
        lambda: fa.forward_mxfp4(*plain, softmax_scale=0.2, affine_a=1.6, affine_b=0.95),
        lambda: fa.forward_mxfp4(*plain, causal=True, lse=lse), lambda: fa.forward_mxfp4(*plain, lse=lse, out=out32),
        lambda: fa.forward_mxfp4(*plain, ex2_pairs=4), lambda: fa.forward_mxfp4(*anchored, guard=(110, 16)),
        lambda: fa.forward_mxfp4(*fp8, pv_fp8=True), lambda: fa.attention_mxfp4(q, k, v),
        lambda: fa.attention_mxfp4(q, k, v, guard=(110, 16), out=out16),
        lambda: fa.attention_mxfp4(q, k, v, pv_fp8=True, causal=True, lse=lse),
        lambda: fa.attention_mxfp4(q, k, v, ex2_pairs=16, out_dtype=torch.bfloat16),
        lambda: fa.attention_mxfp4(grad, k, v),
    ]
    left = [
        lambda: fa.quantize_qkv(q, k[:, :, :128].contiguous(), v), lambda: fa.quantize_qkv(q, k, v, anchored=1),
        lambda: fa.forward_mxfp4(*plain, softmax_scale=1), lambda: fa.forward_mxfp4(*plain, softmax_scale=np.float64(0.3)),
        lambda: fa.forward_mxfp4(*plain, causal=1),
    ]
    refused = [
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
    if dtype == torch.bfloat16:
        taken += bf16
    else:
        refused += bf16
    native, buffers = fa.api._binding, (lse, out32, out16)
    for kind, calls in (("taken", taken), ("left", left), ("refused", refused)):
        for i, call in enumerate(calls):
            watched = _Watched(native)
            got = []
            for binding in (watched, _PythonOnly()):
                monkeypatch.setattr(fa.api, "_binding", binding)
                got.append(_outcome(call, buffers))
            a, b = got
            assert _same(a, b), f"{kind} call {i}: {a} through the native path, {b} through Python"
            assert isinstance(a, _Refused) == (kind == "refused"), f"{kind} call {i}: {a}"
            if kind != "refused":
                assert watched.took == (kind == "taken"), f"{kind} call {i}"
    monkeypatch.setattr(fa.api, "_binding", native)


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
