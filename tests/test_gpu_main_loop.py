"""The 256 x 256 kernel (products whose tiles fill at least half of the chip):
fewer stages than its three LDS slots, as many, and more; contraction ends
inside a stage; last tiles of a few rows and columns beside whole ones, whose
sums are stored unchecked; stripes that a tile does not divide; several
partial results.  256 tiles each, so that no form takes the smaller tiles."""
import numpy as np
import pytest

import oracle
from oracle.metrics import err_row
from tests._gpu import ROW_TOL, check, gpu_available, host, note, poisoned, to_dev
from paper_cs_9809105_amd import inputs

if gpu_available():
    import torch
    import paper_cs_9809105_amd as hs

# contraction elements of one pipeline stage
STAGE = {"f32": 16, "split3_bf16": 16, "split2_f16": 16, "bf16": 64, "f16": 64, "fp8_e4m3": 128, "fp8_e4m3_r1": 64}
FP8 = ("fp8_e4m3", "fp8_e4m3_r1")
# (m, n, p, K, stages): p K blocks of `stages` stages, the last one short
CASES = [(4096, 4096, 1, 1, 1), (4090, 3850, 1, 1, 2), (3841, 3843, 1, 1, 3), (4090, 4096, 2, 1, 2),
         (4096, 3850, 2, 2, 1), (3900, 4001, 3, 3, 5), (4090, 3850, 1, 1, 4)]


@pytest.mark.gpu
@pytest.mark.parametrize("dt", list(STAGE))
@pytest.mark.parametrize("case", CASES)
def test_stages_and_ragged_tiles(dt, case):
    if not gpu_available():
        pytest.skip("no GPU")
    m, n, p, K, stages = case
    k = p * stages * STAGE[dt] - (3 if stages > 1 else 0)
    if dt in FP8:                       # what the form takes: blocks of whole 64s, stripes of whole 32s
        m, k = m + -m % (32 * p), k + -k % (64 * p)
    rows = sorted({r for t in range(0, m, 256) for r in (t, t + 31, t + 127, t + 255)} | {m - 2, m - 1})
    rows = [r for r in rows if r < m]
    A, A64 = to_dev(inputs.normal((m, k), seed=4200), dt)
    Bm, B64 = to_dev(inputs.normal((k, n), seed=4201), dt)
    note("main loop", dt, case, k)
    C = hs.hs_gemm(A, Bm, dtype=dt, p=p, K=K, out=poisoned((m, n), torch.float32))
    torch.cuda.synchronize()
    ref, got = oracle.gemm_rows(A64, B64, rows), host(C)
    assert np.isfinite(got).all()
    if dt in FP8:
        assert err_row(got[rows], ref) <= ROW_TOL[dt]
    else:
        check(got[rows], ref, dt, A64[rows], B64, what="main loop %s" % (case,))
    Ai, Ai64 = to_dev(inputs.small_int((m, k), 4202, -4, 4), dt)
    Bi, Bi64 = to_dev(inputs.small_int((k, n), 4203, -4, 4), dt)
    Ci = hs.hs_gemm(Ai, Bi, dtype=dt, p=p, K=K, out=poisoned((m, n), torch.float32))
    torch.cuda.synchronize()
    assert np.array_equal(host(Ci), Ai64 @ Bi64)         # exact in float64 in any order
