"""The Python entry points on torch tensors: the short way through the C++ module and the long way through binding.py's own
checks give the same results and the same errors."""
import pytest
import torch

import paper_2501_08071_amd as P
from paper_2501_08071_amd import binding

pytestmark = pytest.mark.gpu


class Sub(torch.Tensor):
    """A subclass goes the long way."""


@pytest.fixture(params=["short", "long"])
def way(request, monkeypatch):
    if request.param == "long":
        class Never:
            def __getattr__(self, name):
                return lambda *a: None
        monkeypatch.setattr(binding, "_fast", Never())
    return request.param


def rand(*shape, dtype=torch.float16, seed=0):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    return torch.randn(shape, generator=g, device="cuda").to(dtype)


@pytest.mark.parametrize("dtype", [torch.float16, torch.bfloat16])
def test_every_form_of_a_call(way, dtype):
    q, k, v = (rand(2, 3, 70, 64, dtype=dtype, seed=i) for i in range(3))
    o0, l0 = P.attn_fwd(q, k, v, True, 0.125)
    assert o0.dtype == l0.dtype == torch.float32 and o0.shape == q.shape and l0.shape == q.shape[:3] and not o0.requires_grad
    o, l = torch.empty_like(o0), torch.empty_like(l0)
    r = P.attn_fwd(q, k, v, True, 0.125, o=o, lse=l)
    assert r[0] is o and r[1] is l and torch.equal(o, o0) and torch.equal(l, l0)
    for args, kw in [((1, 0.125), {}), ((True, 0.125), {"stream": torch.cuda.current_stream()}), ((True, 0.125), {"want_lse": False}),
                     ((True, 0.125), {"lse": l})]:
        r = P.attn_fwd(q, k, v, *args, **kw)
        assert torch.equal(r[0], o0) and (r[1] is None if "want_lse" in kw else torch.equal(r[1], l0))
    h, _ = P.attn_fwd_o16(q, k, v, True, 0.125)
    assert h.dtype == dtype and torch.equal(h, o0.to(dtype))
    p = torch.nn.Parameter(q)
    assert torch.equal(P.attn_fwd(p, k, v, True, 0.125)[0], o0)
    assert torch.equal(P.attn_fwd(q.as_subclass(Sub), k, v, True, 0.125)[0].as_subclass(torch.Tensor), o0)
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        s1 = P.softmax_rows_fwd(k)
    s2 = P.softmax_rows_fwd(k, stream=side)
    y = torch.empty_like(k)
    side.synchronize()
    assert torch.equal(s1, s2) and P.softmax_rows_fwd(k, y=y) is y and torch.equal(y, s1)
    w = rand(64, dtype=dtype, seed=9)
    n = P.rmsnorm_fwd(k, w, 1e-6, y=y)
    assert n is y and torch.equal(P.rmsnorm_fwd(k, w, 1e-6), y) and torch.equal(P.rmsnorm_fwd(k, w, eps=0), P.rmsnorm_fwd(k, w, 0.0))
    a, b = rand(3, 40, 64, dtype=dtype), rand(3, 64, 24, dtype=dtype, seed=1)
    c = P.gemm_leakyrelu_fwd(a, b)
    assert c.shape == (3, 40, 24) and torch.equal(P.gemm_leakyrelu_fwd(a[1].contiguous(), b[1].contiguous(), 0.01), c[1])
    out = torch.empty_like(c)
    assert P.gemm_leakyrelu_fwd(a, b, c=out) is out and torch.equal(out, c)
    assert P.softmax_rows_fwd(k[:0]).shape == (0, 3, 70, 64) and P.gemm_leakyrelu_fwd(a[:, :0].contiguous(), b).shape == (3, 0, 24)


def test_what_is_refused(way):
    q, x, w = rand(1, 2, 8, 64), rand(4, 64), rand(64)
    f32 = q.float()
    bad = [(TypeError, lambda: P.attn_fwd(f32, f32, f32, False, 1.0)), (TypeError, lambda: P.attn_fwd(q, q.bfloat16(), q, False, 1.0)),
           (ValueError, lambda: P.attn_fwd(q, q, q[:, :1], False, 1.0)), (ValueError, lambda: P.attn_fwd(q.transpose(1, 2), q, q, False, 1.0)),
           (ValueError, lambda: P.attn_fwd(q.cpu(), q, q, False, 1.0)), (ValueError, lambda: P.attn_fwd(q, q, q, False, 1.0, o=q)),
           (ValueError, lambda: P.attn_fwd(q, q, q, False, 1.0, lse=f32)), (P.AttnError, lambda: P.attn_fwd(q, q, q, False, float("nan"))),
           (P.AttnError, lambda: P.attn_fwd(x[None, None, :, :48].contiguous(), *[x[None, None, :, :48].contiguous()] * 2, False, 1.0)),
           (ValueError, lambda: P.softmax_rows_fwd(x.t())), (ValueError, lambda: P.softmax_rows_fwd(x, y=x.float())), (TypeError, lambda: P.softmax_rows_fwd(f32)),
           (P.RowopsError, lambda: P.softmax_rows_fwd(x.view(-1)[1:65])), (P.RowopsError, lambda: P.rmsnorm_fwd(x, w, -1.0)),
           (ValueError, lambda: P.rmsnorm_fwd(x, w[:32], 1e-6)), (ValueError, lambda: P.gemm_leakyrelu_fwd(x, x)),
           (TypeError, lambda: P.gemm_leakyrelu_fwd(x, x[None])), (ValueError, lambda: P.gemm_leakyrelu_fwd(x, x.t())),
           (P.GemmError, lambda: P.gemm_leakyrelu_fwd(x, w.view(64, 1), float("inf"))), (ValueError, lambda: P.gemm_leakyrelu_fwd(x, w.view(64, 1), c=x))]
    for kind, call in bad:
        with pytest.raises(kind):
            call()
    torch.cuda.synchronize()
