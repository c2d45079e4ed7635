"""Both operands are prepared in one launch; together they can pass the 2^32
threads that a grid may have, and are then prepared in two."""
from paper_cs_9809105_amd import binding as B
from tests._launches import launches

# (op, m, n, k, dtype, p, K), kernel, launches of it: FP64 stripes of 33 rows in 32-row
# tiles, 3.3 billion threads (3.1 read across rows) beside 1.8; row amaxes of 2^26 - 8
# rows beside 64; small ones
CASES = [(("gemm", 31680, 36864, 94080, "f64", 960, 960), "pack_kernel", 2),
         (("tn", 31680, 36864, 94080, "f64", 960, 960), "pack_kernel", 2),
         (("gemm", (1 << 26) - 8, 64, 64, "split2_f16", 1, 1), "row_amax_kernel", 2),
         (("gemm", 3000, 2000, 1000, "split2_f16", 1, 1), "row_amax_kernel", 1),
         (("gemm", 3000, 2000, 1000, "split2_f16", 1, 1), "pack_kernel", 1)]


def test_accepted_sizes_launch():
    got = launches([(op, m, n, k, B.DTYPES[dt], p, K) for (op, m, n, k, dt, p, K), _, _ in CASES])
    for (call, kernel, count), r in zip(CASES, got):
        assert r["workspace"] and r["status"] == B.HS_OK, (call, r)
        mine = [x for x in r["launches"] if kernel in x["kernel"]]
        assert len(mine) == count, (call, mine)
        for x in r["launches"]:
            assert x["grid"][0] * x["block"][0] < 1 << 32, (call, x)


def test_nbody_size_limit():
    """p ceil(S / 256) K below 2^31, pairs of replicas counted once (S = ceil(n / p))."""
    for n, p, K, ok in [((1 << 28) - 4096 * 256, 4096, 4096, True), (1 << 28, 4096, 4096, False),
                        ((1 << 29) - (1 << 20), 4096, 2048, True), (1 << 29, 4096, 2048, False),
                        ((1 << 31) - 1, 4096, 512, False), ((1 << 31) - 1, 4096, 256, True),
                        ((1 << 31) - 1, 1024, 1024, False), ((1 << 31) - 1, 3, 3, True)]:
        for dt in ("f32", "f64"):
            assert (B.hs_workspace_size(B.HS_OP_NBODY, n, 0, 0, dt, p, K) != B.SIZE_MAX) == ok, (n, p, K, dt)
