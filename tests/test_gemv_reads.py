"""Which matrices the matrix-vector kernel reads past the caches: those of which
too little stays there for the next product with the same matrix."""
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
        assert r["status"] == 0 and "ELi%dEEE" % past in r["launches"][0]["kernel"], (dt, m, n, r)


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
