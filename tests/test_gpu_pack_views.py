"""Operands read along the contraction from views whose rows begin at any
element: odd leading dimensions and offsets, contraction blocks that do not
divide into 16-byte units, a block's end inside one, contractions shorter than
a unit, and views that end with their buffer."""
import numpy as np
import pytest

import oracle
from paper_cs_9809105_amd import inputs
from tests._gpu import STORAGE, check, gpu_available, host, note, poisoned, to_dev

if gpu_available():
    import torch
    import paper_cs_9809105_amd as hs

# (m, n, k, p, K, elements before the view's first, elements after its rows)
CASES = [(37, 29, 45, 1, 1, 1, 0), (64, 33, 77, 4, 2, 3, 2), (130, 70, 1001, 8, 2, 0, 5), (33, 40, 3, 1, 1, 2, 0),
         (65, 31, 129, 3, 3, 5, 1), (257, 260, 250, 2, 1, 7, 0)]


@pytest.mark.gpu
@pytest.mark.parametrize("dt", ["f64", "f32", "split3_bf16", "split2_f16", "bf16", "f16"])
@pytest.mark.parametrize("case", CASES)
def test_rows_at_any_element(dt, case):
    if not gpu_available():
        pytest.skip("no GPU")
    m, n, k, p, K, before, after = case
    A, A64 = to_dev(inputs.normal((m, k), seed=4300), dt)
    Bm, B64 = to_dev(inputs.normal((k, n), seed=4301), dt)
    # the surroundings hold NaN: a product that reads one of them shows it
    wide = torch.full((m * (k + after) + before,), float("nan"), dtype=getattr(torch, STORAGE[dt]), device="cuda")
    view = wide.as_strided((m, k), (k + after, 1), before)
    view.copy_(A)
    note("pack view", dt, case)
    out = torch.float64 if dt == "f64" else torch.float32
    C = hs.hs_gemm(view, Bm, dtype=dt, p=p, K=K, out=poisoned((m, n), out))
    torch.cuda.synchronize()
    check(host(C), oracle.gemm(A64, B64), dt, A64, B64, what="pack view %s" % (case,))
    C0 = hs.hs_gemm(A, Bm, dtype=dt, p=p, K=K, out=poisoned((m, n), out))
    torch.cuda.synchronize()
    assert np.array_equal(host(C), host(C0))


# packed operands of 64 MiB and more are laid out four units a thread: rows,
# columns and blocks that end inside a thread's four, each way of reading them
@pytest.mark.gpu
@pytest.mark.parametrize("dt", ["f32", "bf16", "f16"])
@pytest.mark.parametrize("m, n, k, p, K", [(4090, 4104, 4133, 3, 3), (4096, 4096, 4096, 4, 2)])
def test_four_units_a_thread(dt, m, n, k, p, K):
    if not gpu_available():
        pytest.skip("no GPU")
    A, A64 = to_dev(inputs.small_int((m, k), 4310, -4, 4), dt)
    At, _ = to_dev(np.ascontiguousarray(A64.T), dt)
    Bm, B64 = to_dev(inputs.small_int((k, n), 4311, -4, 4), dt)
    G, G64 = to_dev(inputs.small_int((m, n), 4312, -4, 4), "f32")
    note("four units", dt, m, n, k, p, K)
    C = hs.hs_gemm(A, Bm, dtype=dt, p=p, K=K, out=poisoned((m, n), torch.float32))
    Ct = hs.hs_gemm_tn(At, Bm, dtype=dt, p=p, K=K, out=poisoned((m, n), torch.float32))
    torch.cuda.synchronize()
    # sums of at most 4133 products of magnitude 16: exact in FP32 in any order
    a32, b32, g32 = (x.astype(np.float32) for x in (A64, B64, G64))
    ref = a32 @ b32
    assert np.array_equal(host(C), ref)
    assert np.array_equal(host(Ct), ref)
    if dt == "f32":
        dA, dB = hs.hs_gemm_backward(A, Bm, G, dtype=dt, p=p, K=K)
        torch.cuda.synchronize()
        assert np.array_equal(host(dA), g32 @ b32.T)
        assert np.array_equal(host(dB), a32.T @ g32)
