"""The row amaxes of the two-piece FP16 form at every length of a row's and a
column block's tail, of rows at any alignment and of tall sources: each row
holds one value that overflows FP16 unless its amax is found."""
import numpy as np
import pytest

import oracle
from paper_cs_9809105_amd import inputs
from tests._gpu import gpu_available, host, note, poisoned

if gpu_available():
    import torch
    import paper_cs_9809105_amd as hs

# (m, n, k): contraction and columns of every remainder mod 4, one column, a block
# of 32 columns and one past it, one wave's 256 elements and one past them, and
# over 8192 rows on one, five and more than 1024 columns (two blocks side by side)
CASES = [(5, 1, 1), (9, 2, 2), (33, 3, 3), (31, 32, 70), (7, 33, 255), (18, 34, 256), (8, 35, 257), (70, 129, 131),
         (3, 33, 8193), (33, 130, 8195), (66, 36, 4100), (2, 1026, 8200), (2, 1055, 8193), (2, 3, 8200), (1, 5, 8449), (3, 37, 90)]


def _spiked(rows, k, seed):
    """rows x k small integers with 2^20 at one place of each row, its last for row 0."""
    x = inputs.small_int((rows, k), seed, -3, 3)
    x[np.arange(rows), (k - 1 + 7 * np.arange(rows)) % k] = 2.0 ** 20
    return x


def _view(x, pad):
    """x on the device as a view whose rows start `pad` elements into wider ones."""
    w = torch.full((x.shape[0], x.shape[1] + pad), 3.0e38, dtype=torch.float32, device="cuda")
    w[:, pad:] = torch.from_numpy(x)
    return w[:, pad:]


@pytest.mark.gpu
@pytest.mark.parametrize("case", CASES)
@pytest.mark.parametrize("pad", [0, 1, 2, 3])
def test_spikes(case, pad):
    if not gpu_available():
        pytest.skip("no GPU")
    m, n, k = case
    # 2^20 times at most 3, plus k products of at most 9: exact in FP32
    A, Bm = _spiked(m, k, 4500), inputs.small_int((k, n), 4501, -3, 3)
    A2, B2 = inputs.small_int((m, k), 4502, -3, 3), np.ascontiguousarray(_spiked(n, k, 4503).T)
    note("row amax", case, pad)
    for a, b in ((A, Bm), (A2, B2)):
        ref = oracle.gemm(a, b)
        for C in (hs.hs_gemm(_view(a, pad), _view(b, pad), dtype="split2_f16", out=poisoned((m, n), torch.float32)),
                  hs.hs_gemm_tn(_view(np.ascontiguousarray(a.T), pad), _view(b, pad), dtype="split2_f16",
                                out=poisoned((m, n), torch.float32))):
            torch.cuda.synchronize()
            assert np.array_equal(host(C), ref)


@pytest.mark.gpu
@pytest.mark.parametrize("ld", [16384, 16387])
def test_spikes_of_a_source_larger_than_the_cache(ld):
    """16384 x 4100 (256 MiB and more), rows on 128-byte lines and not."""
    if not gpu_available():
        pytest.skip("no GPU")
    m, n, k = 3, 16384, 4100
    g = torch.Generator(device="cuda")
    g.manual_seed(5)
    W = torch.full((k, ld), 3.0e38, device="cuda")
    Bm = W[:, ld - n:]
    Bm.copy_(torch.randint(-3, 4, (k, n), generator=g, device="cuda"))
    j = torch.arange(n, device="cuda")
    Bm[(k - 1 + 7 * j) % k, j] = 2.0 ** 20
    A = torch.randint(-3, 4, (m, k), generator=g, device="cuda").float()
    note("row amax large", ld)
    C = hs.hs_gemm(A, Bm, dtype="split2_f16")
    assert torch.equal(C.double(), A.double() @ Bm.double())
