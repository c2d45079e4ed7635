"""The wave-tile kernel (products whose 256 x 256 tiles would leave most of
the chip idle, and every FP64 product): its plan on the CPU, its results on
the GPU at the sizes where a tile, a class's last group, a chunk or a wave's
share of the chunks begins or ends."""
import numpy as np
import pytest

import oracle
from oracle.metrics import err_row
from paper_cs_9809105_amd import binding as B
from paper_cs_9809105_amd import inputs
from tests._gpu import ROW_TOL, check, gpu_available, host, note, poisoned, to_dev

if gpu_available():
    import torch
    import paper_cs_9809105_amd as hs

FORMS = ["f64", "f32", "split3_bf16", "split2_f16", "bf16", "f16"]


def _up(x, a):
    return -(-x // a) * a


def _tiled_bytes(m, n, k, dt, p):
    """Packed operands in whole 256 x 256 tiles (FP64 64 x 64) and whole
    pipeline stages: stripes of ceil(m / p) rows in groups of at most a tile,
    columns padded to a tile, contraction blocks to whole stages."""
    esz, pieces, tile, stage = {"f64": (8, 1, 64, 128), "f32": (4, 1, 256, 64), "bf16": (2, 1, 256, 128),
                                "split3_bf16": (2, 3, 256, 32), "split2_f16": (2, 2, 256, 32)}[dt]
    s_r, s_k = -(-m // p), -(-k // p)
    ms = min(tile, s_r)
    row = p * _up(s_k * esz, stage) * pieces
    side = 2 * _up(4 * m, 256) + _up(4 * n, 256) if dt == "split2_f16" else 0
    return _up(p * _up(s_r, ms) * row, 256) + _up(_up(n, tile) * row, 256) + side


@pytest.mark.parametrize("dt", ["f64", "f32", "split3_bf16", "split2_f16", "bf16"])
def test_workspace_is_at_most_that_of_whole_tiles(dt):
    """The wave kernel's operands are padded to smaller units, so that a call
    fits wherever whole tiles would fit (planes of a split step order: at
    most 4, and only for a contraction of 1024 or more)."""
    g = inputs.rng(2024)
    for _ in range(300):
        m, n, k = (int(x) for x in np.exp(g.uniform(np.log(1), np.log(3000), size=3)))
        p = int(g.choice([1, 2, 3, 4, 6, 8, 16, 64, 96]))
        K = int(g.choice([d for d in range(1, p + 1) if p % d == 0]))
        planes = 4 * m * n * (8 if dt == "f64" else 4) if k >= 1024 or p >= 64 else 0
        ws = B.hs_workspace_size(B.HS_OP_GEMM, m, n, k, dt, p, K)
        assert 0 < ws <= _tiled_bytes(m, n, k, dt, p) + planes, (m, n, k, p, K)


# (m, n, k, p, K): one row or column short of, at and past a small (32; FP64
# 16) and a large (64; FP64 32) tile, a class list of several stripes with a
# short last group, K = p, one chunk, fewer chunks than waves, many chunks on
# one tile, and products of enough tiles for the large one (900 FP32 tiles:
# 1920 x 1920)
CASES = [(31, 33, 40, 1, 1), (32, 32, 16, 1, 1), (33, 31, 8, 2, 1), (64, 64, 64, 4, 2), (65, 63, 130, 5, 5),
         (63, 65, 257, 4, 4), (17, 300, 515, 3, 1), (300, 15, 96, 12, 4), (1, 1, 1, 1, 1), (5, 7, 4100, 2, 2),
         (130, 66, 1030, 6, 2), (1290, 1300, 72, 10, 2), (1925, 1921, 40, 4, 2)]


@pytest.mark.gpu
@pytest.mark.parametrize("dt", FORMS)
@pytest.mark.parametrize("case", CASES)
def test_wave_products(dt, case):
    if not gpu_available():
        pytest.skip("no GPU")
    m, n, k, p, K = case
    out = torch.float64 if dt == "f64" else torch.float32
    A, A64 = to_dev(inputs.normal((m, k), seed=4100), dt)
    At, _ = to_dev(np.ascontiguousarray(A64.T), dt)
    Bm, B64 = to_dev(inputs.normal((k, n), seed=4101), dt)
    note("wave", dt, case)
    C = hs.hs_gemm(A, Bm, dtype=dt, p=p, K=K, out=poisoned((m, n), out))
    Ct = hs.hs_gemm_tn(At, Bm, dtype=dt, p=p, K=K, out=poisoned((m, n), out))
    torch.cuda.synchronize()
    ref = oracle.gemm(A64, B64)
    check(host(C), ref, dt, A64, B64, what="wave %s" % (case,))
    check(host(Ct), ref, dt, A64, B64, what="wave tn %s" % (case,))
    Ai, Ai64 = to_dev(inputs.small_int((m, k), 4102, -4, 4), dt)
    Bi, Bi64 = to_dev(inputs.small_int((k, n), 4103, -4, 4), dt)
    Ci = hs.hs_gemm(Ai, Bi, dtype=dt, p=p, K=K, out=poisoned((m, n), out))
    torch.cuda.synchronize()
    assert np.array_equal(host(Ci), oracle.gemm(Ai64, Bi64))


@pytest.mark.gpu
@pytest.mark.parametrize("dt", ["fp8_e4m3", "fp8_e4m3_r1"])
@pytest.mark.parametrize("case", [(32, 31, 64, 1, 1), (96, 65, 192, 3, 1), (64, 130, 128, 2, 2), (1408, 1290, 256, 4, 2),
                                  (160, 33, 2560, 5, 5)])
def test_wave_fp8(dt, case):
    """FP8 on stripes that end inside a 128-row scale tile: small integers
    exact, the form's own bound on real values."""
    if not gpu_available():
        pytest.skip("no GPU")
    m, n, k, p, K = case
    for ints in (True, False):
        gen = (lambda s, sd: inputs.small_int(s, sd, -4, 4)) if ints else (lambda s, sd: inputs.uniform(s, sd))
        A, A64 = to_dev(gen((m, k), 4110), dt)
        Bm, B64 = to_dev(gen((k, n), 4111), dt)
        note("wave fp8", dt, case, ints)
        C = hs.hs_gemm(A, Bm, dtype=dt, p=p, K=K, out=poisoned((m, n), torch.float32))
        torch.cuda.synchronize()
        ref = oracle.gemm(A64, B64)
        if ints:
            assert np.array_equal(host(C), ref)
        else:
            assert err_row(host(C), ref) <= ROW_TOL[dt]


# 96 x 64 tiles (two-round counts of 64 x 64 ones): last groups of 65, 1 and 96
# rows, eight waves and the four that eight chunks allow; 64 x 96 tiles with last
# columns of 56, 96 and 4; 128 x 64 tiles (split
# forms): 512 tiles of two waves, 800 of one, last groups of 127, 98 and 1 rows
TALL = ([(dt, c) for dt in ("bf16", "f16", "split3_bf16", "split2_f16")
         for c in [(1090, 961, 250, 2, 2), (1537, 700, 113, 1, 1), (2016, 577, 516, 3, 3),
                   (1000, 1400, 113, 2, 2), (1000, 1152, 200, 10, 10), (995, 1060, 333, 10, 10)]] +
        [(dt, c) for dt in ("split3_bf16", "split2_f16")
         for c in [(2047, 2010, 2050, 2, 1), (2500, 2500, 2100, 4, 2), (1281, 2500, 2049, 1, 1)]])


@pytest.mark.gpu
@pytest.mark.parametrize("dt, case", TALL)
def test_wave_tall_tiles(dt, case):
    if not gpu_available():
        pytest.skip("no GPU")
    m, n, k, p, K = case
    rows = sorted({r for t in range(0, m, 96) for r in (t, t + 31, t + 95) if r < m} | {m - 2, m - 1})
    A, A64 = to_dev(inputs.normal((m, k), seed=4120), dt)
    Bm, B64 = to_dev(inputs.normal((k, n), seed=4121), dt)
    note("wave tall", dt, case)
    C = hs.hs_gemm(A, Bm, dtype=dt, p=p, K=K, out=poisoned((m, n), torch.float32))
    torch.cuda.synchronize()
    assert np.isfinite(host(C)).all()
    check(host(C)[rows], oracle.gemm_rows(A64, B64, rows), dt, A64[rows], B64, what="wave tall %s" % (case,))
    Ai, Ai64 = to_dev(inputs.small_int((m, k), 4122, -4, 4), dt)
    Bi, Bi64 = to_dev(inputs.small_int((k, n), 4123, -4, 4), dt)
    Ci = hs.hs_gemm(Ai, Bi, dtype=dt, p=p, K=K, out=poisoned((m, n), torch.float32))
    torch.cuda.synchronize()
    assert np.array_equal(host(Ci), Ai64 @ Bi64)         # exact in float64 in any order
