"""The 256 x 256 kernel at one stage, at as many as its three LDS slots hold,
at one more and at an odd number over several partial results, with the last
stage short and the last tiles ragged: the forms whose stages are shallow (32
contraction elements of BF16 and FP16, 64 of FP8), and FP32 with K = 3."""
import numpy as np
import pytest

import oracle
from oracle.metrics import err_row
from paper_cs_9809105_amd import binding as B
from paper_cs_9809105_amd import inputs
from tests._gpu import ROW_TOL, check, gpu_available, host, note, poisoned, to_dev
from tests._launches import launches

if gpu_available():
    import torch
    import paper_cs_9809105_amd as hs

STAGE = {"f32": 16, "bf16": 32, "f16": 32, "fp8_e4m3": 64}
# (m, n, p, K, stages of a block, 256 x 256 tiles)
SHAPES = [(4096, 4096, 1, 1, 1, 256), (4090, 3850, 1, 1, 2, 256), (3841, 3843, 1, 1, 3, 256), (4090, 3850, 1, 1, 4, 256),
          (4096, 3850, 2, 2, 1, 256), (3900, 3501, 3, 3, 5, 252)]
CASES = [(dt,) + s for dt in ("bf16", "f16", "fp8_e4m3") for s in SHAPES] + [("f32",) + SHAPES[-1]]


def _sizes(dt, m, n, p, stages):
    k = p * stages * STAGE[dt] - (3 if stages > 1 else 0)
    if dt == "fp8_e4m3":                # what the form takes: blocks of whole 64s, stripes of whole 32s
        m, k = m + -m % (32 * p), k + -k % (64 * p)
    return m, n, k


def test_cases_run_on_the_256_kernel_with_these_stages():
    sizes = [_sizes(dt, m, n, p, stages) for dt, m, n, p, _, stages, _ in CASES]
    got = launches([("gemm", m, n, k, B.DTYPES[c[0]], c[3], c[4]) for c, (m, n, k) in zip(CASES, sizes)])
    for c, r in zip(CASES, got):
        main = [x for x in r["launches"] if "mm_kernel" in x["kernel"]]
        assert r["status"] == 0 and len(main) == 1 and main[0]["grid"][0] == c[6], (c, r)
    # packed operands are padded to whole stages
    for dt, d in STAGE.items():
        if dt != "fp8_e4m3":
            one, two, also = (B.hs_workspace_size(B.HS_OP_GEMM, 4096, 4096, k, dt, 1, 1) for k in (d, d + 1, 2 * d))
            assert one < two == also == 2 * one, dt


@pytest.mark.gpu
@pytest.mark.parametrize("case", CASES)
def test_stage_counts(case):
    if not gpu_available():
        pytest.skip("no GPU")
    dt, m, n, p, K, stages, _ = case
    m, n, k = _sizes(dt, m, n, p, stages)
    rows = sorted({r for t in range(0, m, 256) for r in (t, t + 31, t + 127, t + 255) if r < m} | {m - 2, m - 1})
    A, A64 = to_dev(inputs.normal((m, k), seed=4400), dt)
    Bm, B64 = to_dev(inputs.normal((k, n), seed=4401), dt)
    note("stages", case, k)
    C = hs.hs_gemm(A, Bm, dtype=dt, p=p, K=K, out=poisoned((m, n), torch.float32))
    torch.cuda.synchronize()
    ref, got = oracle.gemm_rows(A64, B64, rows), host(C)
    assert np.isfinite(got).all()
    if dt == "fp8_e4m3":
        assert err_row(got[rows], ref) <= ROW_TOL[dt]
    else:
        check(got[rows], ref, dt, A64[rows], B64, what="stages %s" % (case,))
    Ai, Ai64 = to_dev(inputs.small_int((m, k), 4402, -4, 4), dt)
    Bi, Bi64 = to_dev(inputs.small_int((k, n), 4403, -4, 4), dt)
    Ci = hs.hs_gemm(Ai, Bi, dtype=dt, p=p, K=K, out=poisoned((m, n), torch.float32))
    torch.cuda.synchronize()
    assert np.array_equal(host(Ci), Ai64 @ Bi64)         # exact in float64 in any order
