"""How many waves of a workgroup share the travelling bodies: fewer where a
schedule of many replicas leaves few of them and fills the chip without."""
import pytest

import oracle
from paper_cs_9809105_amd import binding as B
from paper_cs_9809105_amd import inputs
from tests._gpu import gpu_available, note
from tests._launches import launches

# (n, p, K, waves)
CASES = [(5000, 64, 64, 1), (4000, 60, 30, 1), (8000, 32, 32, 2), (16384, 64, 32, 4), (16384, 64, 8, 8), (3000, 16, 4, 16),
         (2000, 16, 16, 4)]


def test_waves():
    for c, r in zip(CASES, launches([("nbody", n, 0, 0, B.HS_F32, p, K) for n, p, K, _ in CASES])):
        main = [x for x in r["launches"] if "nbody_kernel" in x["kernel"]][0]
        assert r["status"] == 0 and main["block"][0] == 64 * c[3], (c, main)


@pytest.mark.gpu
@pytest.mark.parametrize("dt", ["f32", "f64"])
@pytest.mark.parametrize("case", CASES[:3])
def test_few_travelling_bodies(dt, case):
    if not gpu_available():
        pytest.skip("no GPU")
    from tests.test_gpu_nbody import _bounds, _eps2, _errors, _run, _stored
    n, p, K, _ = case
    Xd, X64 = _stored(inputs.plummer(n, seed=4700, unequal=True), dt)
    e2 = _eps2(1e-4, dt)
    note("nbody waves", dt, case)
    ref, scale = oracle.nbody(X64, e2, with_scale=True)
    ea, ep = _errors(_run(Xd, e2, dt, p, K), ref, scale)
    ta, tp = _bounds(n, K, dt)
    assert ea <= ta and ep <= tp, (ea, ta, ep, tp)
