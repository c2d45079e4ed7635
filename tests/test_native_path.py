"""The binding's native call path (csrc/hs_torch.cpp) against its general one
(taken when a stream is passed): the same bits for every entry point, form of
output and strided operand, and the same exception for arguments that either
refuses."""
import pytest

from paper_cs_9809105_amd import binding as B
from tests._gpu import gpu_available, note

if gpu_available():
    import torch
    import paper_cs_9809105_amd as hs


def test_cpu_tensors_are_refused():
    import torch
    x = torch.ones(3, 3)
    for f in (lambda: B.hs_gemm(x, x), lambda: B.hs_gemm_tn(x, x), lambda: B.hs_gemv(x, x[0]),
              lambda: B.hs_gemm_noalloc(x, x, x), lambda: B.hs_gemm_backward(x, x, x),
              lambda: B.hs_nbody(torch.ones(3, 4))):
        with pytest.raises(TypeError):
            f()


def _operands(dt, dev="cuda"):
    t = getattr(torch, B.IN_TYPES[B._dt(dt)])
    g = torch.Generator(device=dev)
    g.manual_seed(7)
    def mat(r, c, pad):
        x = torch.randn((r, c + pad), generator=g, device=dev, dtype=t if t.is_complex else torch.float32).to(t)
        return x[:, pad:]
    m, n, k = (64, 128, 192) if dt.startswith("fp8") else (45, 33, 70)
    return [[mat(m, k, p), mat(k, m, p), mat(k, n, p), mat(m, n, p)] for p in (0, 3)]


@pytest.mark.gpu
@pytest.mark.parametrize("dt", sorted(B.DTYPES))
def test_same_bits_as_the_general_path(dt):
    if not gpu_available():
        pytest.skip("no GPU")
    s = torch.cuda.current_stream()
    o = dict(dtype=dt, p=1, K=0)
    note("native path", dt)
    for A, At, Bm, G in _operands(dt):
        out_t = getattr(torch, B._out_type(B._dt(dt)))
        shape = (A.shape[0], Bm.shape[1])
        wide = torch.full((shape[0], shape[1] + 5), 7, device="cuda", dtype=out_t)[:, 2:2 + shape[1]]
        pairs = [(hs.hs_gemm(A, Bm, **o), hs.hs_gemm(A, Bm, stream=s, **o)),
                 (hs.hs_gemm(A, Bm, out=wide, **o), hs.hs_gemm(A, Bm, stream=s, **o)),
                 (hs.hs_gemm_tn(At, Bm, **o), hs.hs_gemm_tn(At, Bm, stream=s, **o)),
                 (hs.hs_gemm_noalloc(A, Bm, torch.empty(shape, device="cuda", dtype=out_t), **o),
                  hs.hs_gemm(A, Bm, stream=s, **o))]
        pairs += list(zip(hs.hs_gemm_backward(A, Bm, G, **o), hs.hs_gemm_backward(A, Bm, G, stream=s, **o)))
        if dt in ("f32", "f64", "c32"):
            x = Bm[:, :1].reshape(-1).contiguous()
            pairs.append((hs.hs_gemv(A, x, **o), hs.hs_gemv(A, x, stream=s, **o)))
        if dt in ("f32", "f64"):
            b = A[:, :4].contiguous()
            pairs.append((hs.hs_nbody(b, 1e-3, p=1), hs.hs_nbody(b, 1e-3, p=1, stream=s)))
        torch.cuda.synchronize()
        for got, ref in pairs:
            assert got.dtype == ref.dtype and got.shape == ref.shape and torch.equal(got, ref)
        dA, dB = hs.hs_gemm_backward(A, Bm, G, need_a=False, **o)
        assert dA is None and dB is not None


@pytest.mark.gpu
def test_same_refusals_as_the_general_path():
    if not gpu_available():
        pytest.skip("no GPU")
    s = torch.cuda.current_stream()
    A, Bm = torch.ones((8, 6), device="cuda"), torch.ones((6, 5), device="cuda")
    C = torch.ones((8, 5), device="cuda")
    calls = [lambda **k: hs.hs_gemm(A, Bm, p=4, K=3, **k),                  # K does not divide p
             lambda **k: hs.hs_gemm(A, Bm, dtype="f64", **k),
             lambda **k: hs.hs_gemm(A, Bm, dtype=99, **k),
             lambda **k: hs.hs_gemm(A, A, **k),                             # inner dimensions
             lambda **k: hs.hs_gemm(A.t(), A, **k),                         # column-major
             lambda **k: hs.hs_gemm(A[:1].expand(8, 6), Bm, **k),           # overlapping rows
             lambda **k: hs.hs_gemm(A, Bm, out=C[:, :4], **k),
             lambda **k: hs.hs_gemm(A, Bm, out=C.double(), **k),
             lambda **k: hs.hs_gemm(A, Bm, p=1.5, **k),
             lambda **k: hs.hs_gemm(A, Bm, dtype="fp8_e4m3", **k),          # not whole 64-element chunks
             lambda **k: hs.hs_gemm_tn(A, Bm, **k),
             lambda **k: hs.hs_gemm_noalloc(A, Bm, C[:4], **k),
             lambda **k: hs.hs_gemm_backward(A, Bm, Bm, **k),
             lambda **k: hs.hs_gemv(A, Bm[0], **k),
             lambda **k: hs.hs_gemv(A, A[0], dtype="split3_bf16", **k),
             lambda **k: hs.hs_nbody(A, **k),
             lambda **k: hs.hs_nbody(A[:, :4].contiguous(), -1.0, **k)]
    for i, f in enumerate(calls):
        seen = []
        for k in ({}, {"stream": s}):
            with pytest.raises(Exception) as e:
                f(**k)
            seen.append((type(e.value), str(e.value)))
        assert seen[0] == seen[1], i
    # empty matrices are no error on either
    assert hs.hs_gemm(A[:0], Bm).shape == (0, 5) and hs.hs_gemv(A[:, :0], A[0, :0]).abs().sum() == 0
