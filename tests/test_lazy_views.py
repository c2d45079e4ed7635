"""PyTorch's lazy views: conj() and the imaginary part of a conjugate only mark
the tensor, whose memory holds the other sign.  Every entry point multiplies
the values; the call without allocation and every ``out`` refuse such a view."""
import pytest

from tests._gpu import gpu_available, note

if gpu_available():
    import torch
    import paper_cs_9809105_amd as hs
    from paper_cs_9809105_amd import autograd


def _c(shape, seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    return torch.randn(shape, generator=g, device="cuda", dtype=torch.complex64)


@pytest.mark.gpu
@pytest.mark.parametrize("stream", [False, True])
@pytest.mark.parametrize("dt", ["c32", "c32_split3_bf16", "c32_split2_f16"])
def test_conjugate_views(dt, stream):
    if not gpu_available():
        pytest.skip("no GPU")
    m, n, k = 37, 41, 50
    o = dict(dtype=dt, p=2, K=1)
    if stream:
        o["stream"] = torch.cuda.current_stream()
    A, At, Bm, G = _c((m, k + 3), 1)[:, 3:].conj(), _c((k, m), 2).conj(), _c((k, n), 3).conj(), _c((m, n), 4).conj()
    r = [t.resolve_conj() for t in (A, At, Bm, G)]
    assert A.is_conj() and not r[0].is_conj()
    note("conj", dt, stream)
    pairs = [(hs.hs_gemm(A, Bm, **o), hs.hs_gemm(r[0], r[2], **o)),
             (hs.hs_gemm(r[0], Bm, **o), hs.hs_gemm(r[0], r[2], **o)),
             (hs.hs_gemm_tn(At, Bm, **o), hs.hs_gemm_tn(r[1], r[2], **o))]
    pairs += list(zip(hs.hs_gemm_backward(A, Bm, G, **o), hs.hs_gemm_backward(r[0], r[2], r[3], **o)))
    if dt == "c32":
        x = _c((k,), 5).conj()
        pairs.append((hs.hs_gemv(A, x, **o), hs.hs_gemv(r[0], x.resolve_conj(), **o)))
    torch.cuda.synchronize()
    for got, ref in pairs:
        assert torch.equal(got, ref)
    C = torch.empty((m, n), device="cuda", dtype=torch.complex64)
    for call in (lambda: hs.hs_gemm(r[0], r[2], out=C.conj(), **o), lambda: hs.hs_gemm_tn(r[1], r[2], out=C.conj(), **o),
                 lambda: hs.hs_gemm_noalloc(A, r[2], C, **o), lambda: hs.hs_gemm_noalloc(r[0], Bm, C, **o),
                 lambda: hs.hs_gemm_noalloc(r[0], r[2], C.conj(), **o),
                 lambda: hs.hs_gemv(r[0], r[0][0], out=C[:, 0].conj().contiguous().conj(), **dict(o, dtype="c32"))):
        with pytest.raises(ValueError):
            call()


@pytest.mark.gpu
@pytest.mark.parametrize("stream", [False, True])
def test_negative_views(stream):
    if not gpu_available():
        pytest.skip("no GPU")
    o = dict(stream=torch.cuda.current_stream()) if stream else {}
    neg = torch._neg_view
    A, Bm = _c((30, 20), 6).real.contiguous(), _c((20, 25), 7).real.contiguous()
    x, bodies = _c((20,), 8).conj().imag, _c((40, 4), 9).conj().imag        # strided, marked
    assert x.is_neg() and bodies.is_neg() and neg(A).is_neg()
    note("neg", stream)
    pairs = [(hs.hs_gemm(neg(A), Bm, **o), hs.hs_gemm(-A, Bm, **o)),
             (hs.hs_gemv(A, x, **o), hs.hs_gemv(A, x.resolve_neg().contiguous(), **o)),
             (hs.hs_gemv(A, neg(Bm[:, 0].contiguous()), **o), hs.hs_gemv(A, -Bm[:, 0], **o)),
             (hs.hs_nbody(bodies, 0.1, **o), hs.hs_nbody(bodies.resolve_neg().contiguous(), 0.1, **o)),
             (hs.hs_nbody(neg(A[:, :4].contiguous()), 0.1, **o), hs.hs_nbody(-A[:, :4].contiguous(), 0.1, **o))]
    torch.cuda.synchronize()
    for got, ref in pairs:
        assert torch.equal(got, ref)
    with pytest.raises(ValueError):
        hs.hs_nbody(A[:, :4].contiguous(), 0.1, out=neg(torch.empty((30, 4), device="cuda")), **o)


@pytest.mark.gpu
def test_gradient_through_a_conjugate():
    """L = Re sum(conj(C) W): the gradient reaches the product as a conjugate
    view, and dL/dC = W."""
    if not gpu_available():
        pytest.skip("no GPU")
    A, Bm, W = _c((33, 40), 10).requires_grad_(), _c((40, 29), 11).requires_grad_(), _c((33, 29), 12)
    note("conj gradient")
    C = autograd.matmul(A, Bm, dtype="c32", p=2, K=2)
    (C.conj() * W).real.sum().backward()
    dA, dB = hs.hs_gemm_backward(A.detach(), Bm.detach(), W, dtype="c32", p=2, K=2)
    torch.cuda.synchronize()
    assert torch.equal(A.grad, dA) and torch.equal(Bm.grad, dB)
    A2 = A.detach().clone().requires_grad_()
    C2 = autograd.matmul(A2.conj(), Bm.detach(), dtype="c32")
    ref = hs.hs_gemm(A2.detach().conj().resolve_conj(), Bm.detach(), dtype="c32")
    assert torch.equal(C2.detach(), ref)
    C2.backward(W)
    dA2, _ = hs.hs_gemm_backward(A2.detach().conj().resolve_conj(), Bm.detach(), W, dtype="c32")
    assert torch.equal(A2.grad, dA2.conj().resolve_conj())
