"""The matrix-vector kernel's variants: matrices read past the caches (those of
which too little stays there for the next product with the same matrix), and many
short rows, four to a wave."""
import pytest

from paper_cs_9809105_amd import binding as B
from tests._gpu import gpu_available, note
from tests._launches import launches

if gpu_available():
    import torch
    import paper_cs_9809105_amd as hs


def test_a_matrix_near_the_cache_size_is_read_through_it():
    calls = [("f32", 8192, 8192, 0), ("f32", 8192, 9216, 0), ("f64", 4096, 8192, 0), ("c32", 4096, 9216, 0),
             ("f32", 8192, 9728, 1), ("f32", 16384, 16384, 1), ("f64", 8192, 8192, 1), ("c32", 8192, 8192, 1)]
    for (dt, m, n, past), r in zip(calls, launches([("gemv", m, n, 0, B.DTYPES[dt], 64, 8) for dt, m, n, _ in calls])):
        assert r["status"] == 0 and "ELi%dELi64EEE" % past in r["launches"][0]["kernel"], (dt, m, n, r)


@pytest.mark.gpu
@pytest.mark.parametrize("dt", ["f32", "f64", "c32"])
def test_gemv_past_the_caches(dt):
    if not gpu_available():
        pytest.skip("no GPU")
    m, n = (2049, 40003) if dt == "f32" else (2049, 20003)
    g = torch.Generator(device="cuda")
    g.manual_seed(3)
    def ints(*shape):
        x = [torch.randint(-8, 9, shape, generator=g, device="cuda").double() for _ in range(2)]
        return torch.complex(*x) if dt == "c32" else x[0]
    A, x = ints(m, n), ints(n)
    note("gemv past the caches", dt)
    t = getattr(torch, B.IN_TYPES[B.DTYPES[dt]])
    y = hs.hs_gemv(A.to(t), x.to(t), dtype=dt, p=64, K=8)     # small integers: exact
    assert torch.equal(y.to(A.dtype), A @ x)


def test_many_short_rows_share_a_wave():
    calls = [("f32", 8192, 1536, 16), ("f32", 8191, 1536, 64), ("f32", 8192, 1537, 64), ("f64", 8192, 768, 16),
             ("c32", 9000, 769, 64), ("f32", 700000, 122, 16), ("f32", 1000, 777, 64)]
    for (dt, m, n, lanes), r in zip(calls, launches([("gemv", m, n, 0, B.DTYPES[dt], 1, 1) for dt, m, n, _ in calls])):
        x = r["launches"][0]
        assert r["status"] == 0 and "ELi%dEEE" % lanes in x["kernel"], (dt, m, n, x)
        assert x["grid"][0] == -(-m // (256 // lanes)) and x["block"][0] == 256, (dt, m, n, x)


@pytest.mark.gpu
@pytest.mark.parametrize("dt", ["f32", "f64", "c32"])
@pytest.mark.parametrize("n", [1, 2, 3, 5, 63, 64, 65, 127, 128, 129, 255, 256, 257, 511, 513, 767, 768])
def test_short_rows(dt, n):
    """One element short of, at and past a load, a group of loads and the longest
    row of the type's; rows at any alignment; a last workgroup of one to 16 rows."""
    if not gpu_available():
        pytest.skip("no GPU")
    g = torch.Generator(device="cuda")
    g.manual_seed(n)
    t = getattr(torch, B.IN_TYPES[B.DTYPES[dt]])
    def ints(*shape):
        x = [torch.randint(-8, 9, shape, generator=g, device="cuda").double() for _ in range(2)]
        return torch.complex(*x) if dt == "c32" else x[0]
    k = 2 * n if dt == "f32" else n
    for m, pad in ((8192, 0), (8193, 1), (8207, 2), (8208, 3)):
        W, x = ints(m, k + pad), ints(k)
        note("gemv short rows", dt, m, k, pad)
        y = hs.hs_gemv(W.to(t)[:, pad:], x.to(t), dtype=dt, p=4, K=2)     # small integers: exact
        assert torch.equal(y.to(W.dtype), W[:, pad:] @ x)


@pytest.mark.gpu
def test_short_rows_past_the_caches():
    if not gpu_available():
        pytest.skip("no GPU")
    g = torch.Generator(device="cuda")
    g.manual_seed(6)
    A = torch.randint(-8, 9, (700001, 122), generator=g, device="cuda").float()
    x = torch.randint(-8, 9, (122,), generator=g, device="cuda").float()
    note("gemv short rows past the caches")
    assert torch.equal(hs.hs_gemv(A, x).double(), A.double() @ x.double())
