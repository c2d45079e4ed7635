"""The matrix-vector kernel at the edges of its groups of loads and of its
waves-per-row layouts, at every alignment of the rows, against the oracle; an A
of 256 MiB, which is read past the caches."""
import numpy as np
import pytest

import oracle
from paper_cs_9809105_amd import inputs
from tests._gpu import check, gpu_available, host, note, to_dev

pytestmark = pytest.mark.gpu

if gpu_available():
    import torch
    import paper_cs_9809105_amd as hs

# (m, n, p, K): one element short of, at and past a group of 256 lanes' loads
# (FP32 1024 elements; FP64 and complex 512), of two groups and of a single
# load; rows at every alignment; p > n and K = p; the lengths and row counts
# from which two and four waves share a row
CASES = [(5, 1, 1, 1), (5, 3, 1, 1), (5, 5, 4, 2), (5, 255, 3, 3), (5, 511, 2, 1), (5, 512, 2, 2), (5, 513, 2, 2),
         (3, 1023, 3, 3), (3, 1024, 4, 4), (3, 1025, 4, 1), (3, 2047, 1, 1), (3, 2051, 4, 2), (11, 3, 64, 8),
         (300, 500, 64, 8), (6, 900, 4096, 64), (399, 6143, 8, 2), (399, 6145, 8, 2), (401, 6144, 8, 2),
         (402, 12287, 4, 2), (403, 12289, 4, 4), (7, 12300, 1, 1)]


@pytest.mark.parametrize("dt", ["f32", "f64", "c32"])
@pytest.mark.parametrize("case", CASES)
def test_gemv_edges(dt, case):
    if not gpu_available():
        pytest.skip("no GPU")
    m, n, p, K = case
    note("gemv", dt, case)
    if dt == "c32":
        z = [inputs.normal(s, 5200 + i) + 1j * inputs.normal(s, 5210 + i) for i, s in enumerate([(m, n), (n,)])]
        A, x = (torch.from_numpy(v.astype(np.complex64)).cuda() for v in z)
        y = hs.hs_gemv(A, x, dtype=dt, p=p, K=K).cpu().numpy().astype(np.complex128)
        Ah, xh = (v.cpu().numpy().astype(np.complex128) for v in (A, x))
        check(y, oracle.complex_gemv(Ah, xh), "c32", Ah, xh[:, None], what="gemv %s" % (case,), vector=True)
        return
    A, A64 = to_dev(inputs.normal((m, n + 1), 5200), dt)
    A, A64 = A[:, 1:], A64[:, 1:]             # rows that start at an odd element
    x, x64 = to_dev(inputs.normal((n,), 5201), dt)
    y = hs.hs_gemv(A, x, dtype=dt, p=p, K=K)
    check(host(y), oracle.gemv(A64, x64), dt, A64, x64[:, None], what="gemv %s" % (case,), vector=True)
    Ai, Ai64 = to_dev(inputs.small_int((m, n), 5202), dt)
    xi, xi64 = to_dev(inputs.small_int((n,), 5203), dt)
    assert np.array_equal(host(hs.hs_gemv(Ai, xi, dtype=dt, p=p, K=K)), oracle.gemv(Ai64, xi64))


def test_gemv_of_256_mib():
    if not gpu_available():
        pytest.skip("no GPU")
    g = torch.Generator(device="cuda")
    g.manual_seed(3)
    A = torch.randint(-8, 9, (2048, 32768), generator=g, device="cuda").float()
    x = torch.randint(-8, 9, (32768,), generator=g, device="cuda").float()
    note("gemv 256 MiB")
    y = hs.hs_gemv(A, x, p=64, K=8)           # small integers: exact
    assert torch.equal(y.double(), A.double() @ x.double())
