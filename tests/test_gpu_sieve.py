"""GPU parity of the threshold-first batch search (large enough mk_knn_search
calls) against the float64 oracle: tile edges, every dimension class, and data
on which a query's result cannot be proven and the fused search takes over."""
import numpy as np
import pytest

import oracle
from band import check_rows

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def api():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1702_08734_amd import api as a
    a.lib()
    return a


def dev(x):
    return torch.from_numpy(np.ascontiguousarray(x)).cuda()


def mixture(rng, n, d):
    mu = 2.0 * np.random.default_rng(d).standard_normal((50, d))
    return (mu[rng.integers(0, 50, n)] + rng.standard_normal((n, d))).astype(np.float32)


def check(api, xq, xb, k, metric, yn=None, rows=None):
    print(f"sieve nq={len(xq)} nb={len(xb)} d={xb.shape[1]} k={k} {metric}", flush=True)
    D, I = api.knn_search(dev(xq), dev(xb), k, metric, yn)
    torch.cuda.synchronize()
    rows = np.unique(np.linspace(0, len(xq) - 1, 24).astype(int)) if rows is None else rows
    fails = check_rows(D.cpu().numpy()[rows], I.cpu().numpy()[rows], xq, xb, rows, k, metric)
    assert not fails, fails[:10]
    return D, I


# every padded class and its edges, odd and unaligned dimensions, query counts
# at and beside a workgroup's 256 (128 for d > 128), database sizes that fill
# no tile, k at the edges of the 64-entry queues
@pytest.mark.parametrize("metric", ["l2", "ip"])
@pytest.mark.parametrize("nq,nb,d,k", [
    (1024, 16384, 17, 1), (64, 262_145, 32, 48), (257, 70_001, 33, 49), (512, 32_769, 64, 112),
    (300, 60_013, 90, 113), (256, 66_000, 96, 10), (255, 70_007, 100, 240), (1025, 20_000, 128, 7),
    (129, 131_073, 129, 32), (128, 140_000, 200, 5), (385, 50_001, 256, 100),
    (600, 30_011, 128, 1008), (513, 40_000, 64, 1009), (300, 65_537, 128, 1024)])
def test_sieve_shapes(api, nq, nb, d, k, metric):
    rng = np.random.default_rng(nq + nb + d + k)
    check(api, mixture(rng, nq, d), mixture(rng, nb, d), k, metric)


def test_sieve_unaligned_base(api):
    # rows that start 4 bytes off a 16-byte boundary
    rng = np.random.default_rng(1)
    xb, xq = mixture(rng, 40_000, 64), mixture(rng, 500, 64)
    flat = torch.empty(40_000 * 64 + 1, device="cuda")
    flat[1:] = dev(xb).flatten()
    D, I = api.knn_search(dev(xq), flat[1:].view(40_000, 64), 10)
    D2, I2 = api.knn_search(dev(xq), dev(xb), 10)
    assert torch.equal(I, I2) and torch.allclose(D, D2, rtol=1e-6)


@pytest.mark.parametrize("metric", ["l2", "ip"])
@pytest.mark.parametrize("k", [10, 1000])
def test_sieve_sorted_rows(api, k, metric):
    # rows and queries in the order of their clusters: thresholds from the
    # sample, tiles full of one query's candidates
    rng = np.random.default_rng(2)
    mu = 2.0 * rng.standard_normal((40, 48))
    xb = (np.repeat(mu, 2000, axis=0) + rng.standard_normal((80_000, 48))).astype(np.float32)
    check(api, xb[:512] + np.float32(0.01), xb, k, metric)


@pytest.mark.parametrize("metric", ["l2", "ip"])
@pytest.mark.parametrize("k", [1, 40, 600])
def test_sieve_integer_ties(api, k, metric):
    # small integers, thousands of exact ties at rank k: no proof is possible,
    # the fused search answers, lower index first
    rng = np.random.default_rng(3 + k)
    xb = rng.integers(-1, 2, size=(70_000, 12)).astype(np.float32)
    xq = rng.integers(-1, 2, size=(256, 12)).astype(np.float32)
    D, I = api.knn_search(dev(xq), dev(xb), k, metric)
    torch.cuda.synchronize()
    rows = np.arange(0, 256, 9)
    Do, Io = oracle.knn(xq[rows], xb, k, oracle.METRIC_L2 if metric == "l2" else oracle.METRIC_IP)
    np.testing.assert_array_equal(I.cpu().numpy()[rows], Io)
    np.testing.assert_array_equal(D.cpu().numpy()[rows].astype(np.float64), Do)


def test_sieve_equal_rows(api):
    xb = np.ones((70_000, 20), np.float32)
    D, I = api.knn_search(dev(xb[:256]), dev(xb), 30)
    assert (D == 0).all() and torch.equal(I, torch.arange(30, device="cuda").expand(256, 30))


def test_sieve_graded_columns(api):
    # one column 2^60 times another, queries along the small one: FP16 planes
    # cannot hold it, the proof fails and the fused search answers
    rng = np.random.default_rng(4)
    xb = rng.standard_normal((70_000, 8)).astype(np.float32)
    xb[:, 0] *= 2.0 ** 30
    xb[:, 1] *= 2.0 ** -30
    xq = np.zeros((256, 8), np.float32)
    xq[:, 1] = rng.standard_normal(256)
    check(api, xq, xb, 20, "ip")


@pytest.mark.parametrize("scale", [1e-18, 1e15])
def test_sieve_scales(api, scale):
    # magnitudes outside what the split rows take
    rng = np.random.default_rng(5)
    xb = (mixture(rng, 70_000, 24) * np.float32(scale)).astype(np.float32)
    xq = (mixture(rng, 256, 24) * np.float32(scale)).astype(np.float32)
    check(api, xq, xb, 10, "ip")


def test_sieve_products_underflow(api):
    # inner products (about 1e-60) that no FP32 value holds: the fused search's
    # answer, which the allocation-free call gives
    rng = np.random.default_rng(5)
    xb, xq = (dev(mixture(rng, n, 24) * np.float32(1e-30)) for n in (70_000, 256))
    D, I = api.knn_search(xq, xb, 10, "ip")
    D2, I2 = api.knn_search_noalloc(xq, xb, 10, "ip")
    assert torch.equal(I, I2) and torch.equal(D, D2)


def test_sieve_far_from_origin(api):
    # norms a million times the distances between neighbours
    rng = np.random.default_rng(6)
    xb = (rng.standard_normal((70_000, 16)) + 300.0).astype(np.float32)
    check(api, xb[:256] + np.float32(0.25), xb, 10, "l2")


def test_sieve_supplied_norms(api):
    # rows whose supplied norm is infinite are left out
    rng = np.random.default_rng(7)
    xb, xq = mixture(rng, 70_000, 40), mixture(rng, 300, 40)
    yn = api.norms(dev(xb))
    keep = np.arange(0, 70_000, 2)
    yn[1::2] = float("inf")
    D, I = api.knn_search(dev(xq), dev(xb), 12, "l2", yn)
    rows = np.arange(0, 300, 17)
    fails = check_rows(D.cpu().numpy()[rows], I.cpu().numpy()[rows] // 2, xq,
                       np.ascontiguousarray(xb[keep]), rows, 12, "l2")
    assert not fails and (I % 2 == 0).all(), fails[:10]


@pytest.mark.parametrize("value", [float("nan"), float("inf")])
def test_sieve_rows_not_finite(api, value):
    # a row that is not finite hides no other row's neighbours
    rng = np.random.default_rng(8)
    xb, xq = mixture(rng, 70_000, 40), mixture(rng, 256, 40)
    D0, I0 = api.knn_search(dev(xq), dev(xb), 5)
    used = set(I0.cpu().numpy().ravel().tolist())
    spare = next(i for i in range(70_000) if i not in used)
    xb[spare, 3] = value
    D, I = api.knn_search(dev(xq), dev(xb), 5)
    assert torch.equal(I, I0) and torch.equal(D, D0)


def test_sieve_batches_alike(api):
    # a query's result does not depend on the batch it comes in
    rng = np.random.default_rng(9)
    xb, xq = dev(mixture(rng, 100_000, 64)), dev(mixture(rng, 700, 64))
    D, I = api.knn_search(xq, xb, 20)
    for lo, hi in ((0, 64), (200, 500), (690, 700)):
        d, i = api.knn_search(xq[lo:hi].contiguous(), xb, 20)
        assert torch.equal(d, D[lo:hi]) and torch.equal(i, I[lo:hi])


# low-precision batches against calls of 32 queries, which the fused search
# answers: the same candidates, so the same results bit for bit
@pytest.mark.parametrize("metric", ["l2", "ip"])
@pytest.mark.parametrize("prec", ["bf16", "fp8"])
@pytest.mark.parametrize("nq,nb,d,k,R", [(300, 60_013, 17, 5, 40), (513, 33_000, 64, 20, 80),
                                         (260, 70_001, 90, 100, 400), (257, 66_000, 128, 10, 64),
                                         (200, 90_007, 200, 7, 28), (100, 400_000, 96, 256, 1024)])
def test_sieve_lowp_equals_small_batches(api, nq, nb, d, k, R, prec, metric):
    print(f"lowp sieve nq={nq} nb={nb} d={d} R={R} {prec} {metric}", flush=True)
    rng = np.random.default_rng(nq + nb + d)
    xb, xq = dev(mixture(rng, nb, d)), dev(mixture(rng, nq, d))
    lp, inv = api.quantize_rows(xb, prec)
    D, I = api.knn_search_lowp(xq, xb, lp, inv, k, R, prec, metric)
    for lo in (0, 64, nq - 32):
        q = xq[lo:lo + 32].contiguous()
        d2, i2 = api.knn_search_lowp(q, xb, lp, inv, k, R, prec, metric)
        assert torch.equal(I[lo:lo + 32], i2) and torch.equal(D[lo:lo + 32], d2)


# nearest row (k = 1) of many queries among few rows: class edges, row counts
# around a tile and a group of four, duplicate rows (lower index first), rows
# equal to queries
@pytest.mark.parametrize("n,K,d", [(8192, 4096, 128), (9001, 4099, 33), (16_385, 2305, 96),
                                   (131_072, 256, 8), (131_073, 257, 64), (8200, 5001, 200),
                                   (8192, 65_536, 17)])
def test_nearest_rows(api, n, K, d):
    print(f"nearest n={n} K={K} d={d}", flush=True)
    rng = np.random.default_rng(n + K + d)
    x, c = mixture(rng, n, d), mixture(rng, K, d)
    c[K - 1] = c[3]
    c[K // 2] = c[7]
    x[5], x[6], x[n - 1] = c[3], c[7], c[K - 2]
    a, dist = api.kmeans_assign(dev(x), dev(c))
    rows = np.unique(np.concatenate([np.linspace(0, n - 1, 60).astype(int), [5, 6, n - 1]]))
    fails = check_rows(dist.cpu().numpy()[rows, None], a.cpu().numpy()[rows, None], x, c, rows, 1)
    assert not fails, fails[:10]
    assert a[5] == 3 and a[6] == 7 and a[n - 1] == K - 2 and dist[5] == 0
    # the same bits as small batches (fused search)
    a2, d2 = api.kmeans_assign(dev(x[:200]), dev(c))
    assert torch.equal(a[:200], a2) and torch.equal(dist[:200], d2)


def test_nearest_ties_and_bad_rows(api):
    # integer rows: thousands of ties for the nearest; then a row that is not
    # finite and one too large to split
    rng = np.random.default_rng(12)
    x = rng.integers(-1, 2, size=(9000, 16)).astype(np.float32)
    c = rng.integers(-1, 2, size=(4000, 16)).astype(np.float32)
    for bad in (None, np.nan, 1e30):
        if bad is not None:
            c[17, 2] = bad
        a, dist = api.kmeans_assign(dev(x), dev(c))
        a2, d2 = api.kmeans_assign(dev(x[:300]), dev(c))
        assert torch.equal(a[:300], a2) and torch.equal(dist[:300], d2)
    a, dist = a.cpu().numpy(), dist.cpu().numpy()
    c64 = np.delete(c.astype(np.float64), 17, axis=0)
    keep = np.delete(np.arange(4000), 17)
    for i in range(0, 9000, 301):
        d64 = ((x[i].astype(np.float64) - c64) ** 2).sum(1)
        assert dist[i] == d64.min() and a[i] == keep[d64.argmin()]


# few queries over any database (16 queries a block, 64 from 17 on), group and
# tile remainders, short and long result lists
@pytest.mark.parametrize("metric", ["l2", "ip"])
@pytest.mark.parametrize("nq,nb,d,k", [(1, 2048, 128, 64), (1, 100_003, 128, 10), (16, 70_001, 33, 5),
                                       (17, 65_537, 64, 100), (63, 40_001, 96, 1000), (40, 33_000, 200, 7),
                                       (5, 300_000, 256, 1024), (200, 2049, 32, 63), (700, 5003, 100, 150)])
def test_dense_shapes(api, nq, nb, d, k, metric):
    rng = np.random.default_rng(nq + nb + d + k)
    xb, xq = mixture(rng, nb, d), mixture(rng, nq, d)
    xb[nb // 2], xq[0] = xb[3], xb[3]
    yn = api.norms(dev(xb)) if nq % 2 else None
    check(api, xq, xb, k, metric, yn)


def test_dense_rows_without_score(api):
    # rows whose supplied norm is infinite, and rows with a NaN, are left out
    rng = np.random.default_rng(21)
    xb, xq = mixture(rng, 20_000, 24), mixture(rng, 9, 24)
    yn = api.norms(dev(xb))
    yn[1::2] = float("inf")
    xb[4::8, 5] = np.nan
    keep = np.array([i for i in range(0, 20_000, 2) if i % 8 != 4])
    D, I = api.knn_search(dev(xq), dev(xb), 12, "l2", yn)
    fails = check_rows(D.cpu().numpy(), np.searchsorted(keep, I.cpu().numpy()), xq,
                       np.ascontiguousarray(xb[keep]), np.arange(9), 12, "l2")
    assert not fails and np.isin(I.cpu().numpy(), keep).all(), fails[:10]


# both sides of the dense search's selection rules: a wave or a workgroup per query
# (1,024 queries; 48 results), whole rows of minima or segments of them; ties and
# rows without a score among the candidates, the same answers on both sides
@pytest.mark.parametrize("nq,nb,d,k", [(1023, 2049, 20, 48), (1024, 2049, 20, 48), (1025, 4096, 32, 1),
                                       (1030, 2500, 33, 49), (3, 40_000, 16, 48), (3, 140_001, 16, 49),
                                       (9, 500_000, 8, 500), (2, 131_072, 24, 1000)])
def test_dense_selection(api, nq, nb, d, k):
    rng = np.random.default_rng(nq + nb + k)
    xb = rng.integers(-2, 3, size=(nb, d)).astype(np.float32)  # many equal distances
    xq = rng.integers(-2, 3, size=(nq, d)).astype(np.float32)
    yn = api.norms(dev(xb))
    yn[5::7] = float("inf")
    D, I = api.knn_search(dev(xq), dev(xb), k, "l2", yn)
    D, I = D.cpu().numpy(), I.cpu().numpy()
    live = np.ones(nb, bool)
    live[5::7] = False
    rows = np.flatnonzero(live)
    for i in range(0, nq, max(1, nq // 12)):
        d64 = ((xq[i].astype(np.float64) - xb[rows]) ** 2).sum(1)
        order = np.argsort(d64, kind="stable")[:k]  # integers: exact, ties by row
        assert (I[i] == rows[order]).all() and (D[i] == d64[order]).all(), i


# few queries go through the small-side search, many through the threshold-first
# one: the same rows and distances, whatever the granules of a row and the norms
@pytest.mark.parametrize("metric", ["l2", "ip"])
@pytest.mark.parametrize("d", [8, 30, 64, 100, 128, 132])
@pytest.mark.parametrize("given", [False, True])
def test_dense_equals_sieve(api, d, given, metric):
    rng = np.random.default_rng(d)
    nb, k = 70_003, 30
    xb, xq = mixture(rng, nb, d), mixture(rng, 2000, d)
    if metric == "l2":  # (no distance; a NaN inner product has no place in the order)
        xb[5, 0], xb[nb - 2, d - 1] = np.nan, np.nan
    xb_d, xq_d = dev(xb), dev(xq)
    yn = api.norms(xb_d) if given and metric == "l2" else None
    D, I = api.knn_search(xq_d, xb_d, k, metric, yn)
    for nq in (1, 15, 17, 65):
        D2, I2 = api.knn_search(xq_d[:nq].contiguous(), xb_d, k, metric, yn)
        assert torch.equal(torch.nan_to_num(D2, 0, 1e38, -1e38), torch.nan_to_num(D[:nq], 0, 1e38, -1e38))
        assert torch.equal(I2, I[:nq])


# both sides of the host-resident search's choice for a chunk
@pytest.mark.parametrize("nq", [3500, 3501])
@pytest.mark.parametrize("metric", ["l2", "ip"])
def test_host_chunks_alike(api, nq, metric):
    rng = np.random.default_rng(nq)
    xb = torch.from_numpy(mixture(rng, 60_000, 40)).pin_memory()
    xq = dev(mixture(rng, nq, 40))
    D, I = api.knn_search_host(xq, xb, 12, metric, 25_000)
    D2, I2 = api.knn_search(xq, xb.cuda(), 12, metric)
    assert torch.equal(D, D2) and torch.equal(I, I2)


@pytest.mark.parametrize("nq", [257, 300, 512])
@pytest.mark.parametrize("d,k", [(40, 12), (128, 100), (200, 300)])
def test_sieve_norms_of_minus_infinity(api, nq, d, k):
    # such rows pass every threshold and no more: the k nearest are the oracle's, also
    # where the last block of queries is not full
    rng = np.random.default_rng(d + nq)
    xb, xq = mixture(rng, 70_000, d), mixture(rng, nq, d)
    yn = api.norms(dev(xb))
    yn[5::14_001] = float("-inf")
    print(f"norms of -inf nq={nq} d={d} k={k}", flush=True)
    D, I = api.knn_search(dev(xq), dev(xb), k, "l2", yn)
    rows = np.arange(0, nq, 17)
    fails = check_rows(D.cpu().numpy()[rows], I.cpu().numpy()[rows], xq, xb, rows, k, "l2")
    assert not fails, fails[:10]
    # calls of 32 queries, which need no thresholds
    for r in (0, nq - 32):
        Ds, Is = api.knn_search(dev(xq[r:r + 32]), dev(xb), k, "l2", yn)
        assert torch.equal(D[r:r + 32], Ds) and torch.equal(I[r:r + 32], Is)
