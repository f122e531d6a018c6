"""GPU parity of the exact searches where their routes meet: calls on both sides of a
routing rule, rows left out by supplied norms, database slabs and query batches, data
on which few or all queries lack a proof."""
import numpy as np
import pytest

import oracle
from band import check_rows, gamma

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


# k = 1 on both sides of the nearest-row search's 8,192 queries: rows that the caller
# left out by an infinite or NaN norm are never the answer, though queries equal them
# and every group of four rows holds one with a score
@pytest.mark.parametrize("left_out", [float("inf"), float("nan")])
@pytest.mark.parametrize("nq", [8191, 8192])
@pytest.mark.parametrize("d", [30, 64, 200])
def test_nearest_rows_left_out(api, d, nq, left_out):
    rng = np.random.default_rng(d)
    nb = 4099
    xb, xq = mixture(rng, nb, d), mixture(rng, nq, d)
    xb[1::2] = xb[:-1:2] + np.float32(0.01) * rng.standard_normal((nb // 2, d)).astype(np.float32)
    xq[:2000] = xb[1:4001:2]
    yn = api.norms(dev(xb))
    yn[1::2] = left_out
    print(f"nearest rows left out d={d} nq={nq} {left_out}", flush=True)
    D, I = api.knn_search(dev(xq), dev(xb), 1, "l2", yn)
    D, I = D.cpu().numpy(), I.cpu().numpy()
    assert (I % 2 == 0).all()
    rows = np.arange(0, nq, 61)
    fails = check_rows(D[rows], I[rows] // 2, xq, np.ascontiguousarray(xb[::2]), rows, 1, "l2")
    assert not fails, fails[:10]


# a few queries in a batch without a proof (zero rows under inner products: every row
# ties), as many as fill no block or several, beside others that have one
@pytest.mark.parametrize("nq,every", [(1500, 1499), (1500, 30), (257, 2), (4000, 3)])
@pytest.mark.parametrize("k", [10, 100])
def test_few_unproven_queries(api, nq, every, k):
    rng = np.random.default_rng(nq + every)
    nb, d = 40_003, 40
    xb, xq = mixture(rng, nb, d), mixture(rng, nq, d)
    xq[::every] = 0.0
    print(f"few unproven nq={nq} every={every} k={k}", flush=True)
    D, I = api.knn_search(dev(xq), dev(xb), k, "ip")
    D, I = D.cpu().numpy(), I.cpu().numpy()
    assert (D[::every] == 0).all() and (I[::every] == np.arange(k)).all()
    rows = np.setdiff1d(np.arange(1, nq, 37), np.arange(0, nq, every))
    fails = check_rows(D[rows], I[rows], xq, xb, rows, k, "ip")
    assert not fails, fails[:10]


@pytest.mark.parametrize("prec", ["bf16", "fp8"])
def test_few_unproven_queries_lowp(api, prec):
    # the same candidates as calls of 32 queries, which the fused search answers
    rng = np.random.default_rng(3)
    xb, xq = dev(mixture(rng, 60_001, 40)), dev(mixture(rng, 700, 40))
    xq[::9] = 0.0
    lp, inv = api.quantize_rows(xb, prec)
    print(f"few unproven {prec}", flush=True)
    D, I = api.knn_search_lowp(xq, xb, lp, inv, 10, 40, prec, "ip")
    for lo in (0, 300, 668):
        d2, i2 = api.knn_search_lowp(xq[lo:lo + 32].contiguous(), xb, lp, inv, 10, 40, prec, "ip")
        assert torch.equal(I[lo:lo + 32], i2) and torch.equal(D[lo:lo + 32], d2)


# data on which the first candidates prove nothing: clusters far apart for their width,
# rows far from the origin, integers with many equal distances; short and long lists
# (a wave or a workgroup per query finishes)
@pytest.mark.parametrize("kind,scale", [("spread", 30), ("spread", 300), ("far", 30), ("far", 300),
                                        ("integers", 1)])
@pytest.mark.parametrize("d,k", [(24, 10), (64, 48), (64, 49), (128, 300), (33, 1000)])
def test_unproven_by_the_first_candidates(api, kind, scale, d, k):
    rng = np.random.default_rng(d + k)
    nb, nq = 80_009, 520
    if kind == "spread":
        mu = scale * rng.standard_normal((40, d))
        xb = (mu[rng.integers(0, 40, nb)] + rng.standard_normal((nb, d))).astype(np.float32)
    elif kind == "far":
        xb = (mixture(rng, nb, d) + np.float32(scale)).astype(np.float32)
    else:
        xb = np.round(mixture(rng, nb, d) * 0.7).astype(np.float32)
    xq = xb[rng.integers(0, nb, nq)].copy()
    if kind != "integers":
        xq += np.float32(0.1) * rng.standard_normal((nq, d)).astype(np.float32)
    print(f"unproven {kind} {scale} d={d} k={k}", flush=True)
    D, I = api.knn_search(dev(xq), dev(xb), k)
    D, I = D.cpu().numpy(), I.cpu().numpy()
    rows = np.arange(0, nq, 41)
    if kind == "integers":  # exact: ties by the lower row
        for i in rows:
            d64 = ((xq[i].astype(np.float64) - xb) ** 2).sum(1)
            order = np.argsort(d64, kind="stable")[:k]
            assert (I[i] == order).all() and (D[i] == d64[order]).all(), i
    else:
        # A query that stays without a proof has the answer of a search that ranks by
        # FP32 scores ||y||^2 - 2 <x, y> and re-ranks the k + 16 best: where norms are
        # 10^5 times the distances, a rank may be off by what two scores err by (d
        # products, d squares and their sum, each rounded once).
        for i in rows:
            fails = check_rows(D[i:i + 1], I[i:i + 1], xq, xb, np.array([i]), k, "l2")
            if fails:
                x, y = xq[i].astype(np.float64), xb.astype(np.float64)
                d64 = np.sort(((x - y) ** 2).sum(1))[:k]
                err = gamma(d + 2) * ((x * x).sum() + (y * y).sum(1).max())
                assert scale == 300 and (D[i] <= d64 + 2 * err).all(), (i, fails[:10])
                assert (np.diff(D[i]) >= 0).all() and len(set(I[i])) == k


# a second slab of split rows (524,288 of 1,024 bytes are one), shorter than a tile, that
# holds the best rows; the same by supplied norms
@pytest.mark.parametrize("metric", ["l2", "ip"])
@pytest.mark.parametrize("given", [False, True])
def test_sieve_second_slab(api, metric, given):
    rng = np.random.default_rng(11)
    nb, d, nq = 524_288 + 37, 132, 300
    xb, xq = mixture(rng, nb, d), mixture(rng, nq, d)
    xb[-37:] = 1.001 * xq[:37] + np.float32(1e-3) * rng.standard_normal((37, d)).astype(np.float32)
    xb[524_287] = xq[40]
    yn = api.norms(dev(xb)) if given else None
    print(f"second slab {metric} {given}", flush=True)
    D, I = api.knn_search(dev(xq), dev(xb), 7, metric, yn)
    D, I = D.cpu().numpy(), I.cpu().numpy()
    if metric == "l2":
        assert (I[:37, 0] == np.arange(nb - 37, nb)).all() and I[40, 0] == 524_287
    rows = np.array([0, 17, 36, 40, 41, 299])
    fails = check_rows(D[rows], I[rows], xq, xb, rows, 7, metric)
    assert not fails, fails[:10]


def test_sieve_query_batches(api):
    # 60,000 queries with pools for 39,936 at a time
    rng = np.random.default_rng(12)
    xb, xq = dev(mixture(rng, 200_000, 32)), dev(mixture(rng, 60_000, 32))
    print("query batches", flush=True)
    D, I = api.knn_search(xq, xb, 1000)
    for lo in (0, 20_000, 40_000):
        d2, i2 = api.knn_search(xq[lo:lo + 20_000].contiguous(), xb, 1000)
        assert torch.equal(D[lo:lo + 20_000], d2) and torch.equal(I[lo:lo + 20_000], i2)


def test_lowp_query_batches(api):
    rng = np.random.default_rng(13)
    xb, xq = dev(mixture(rng, 200_000, 32)), dev(mixture(rng, 60_000, 32))
    lp, inv = api.quantize_rows(xb, "bf16")
    print("lowp query batches", flush=True)
    D, I = api.knn_search_lowp(xq, xb, lp, inv, 10, 1024, "bf16", "ip")
    for lo in (0, 20_000, 40_000):
        d2, i2 = api.knn_search_lowp(xq[lo:lo + 20_000].contiguous(), xb, lp, inv, 10, 1024, "bf16", "ip")
        assert torch.equal(D[lo:lo + 20_000], d2) and torch.equal(I[lo:lo + 20_000], i2)


def test_nearest_query_batches(api):
    # 2^20 queries at a time
    rng = np.random.default_rng(14)
    n = (1 << 20) + 300
    x, c = dev(mixture(rng, n, 8)), dev(mixture(rng, 260, 8))
    print("nearest query batches", flush=True)
    a, dist = api.kmeans_assign(x, c)
    for lo in (0, (1 << 20) - 5000, n - 9000):
        a2, d2 = api.kmeans_assign(x[lo:lo + 9000].contiguous(), c)
        assert torch.equal(a[lo:lo + 9000], a2) and torch.equal(dist[lo:lo + 9000], d2)


# rows in the order of their clusters, queries near one of them: the sample's entries are
# of strata far apart
@pytest.mark.parametrize("metric", ["l2", "ip"])
@pytest.mark.parametrize("nb,d,nq,k", [(60_000, 64, 300, 100), (60_033, 128, 512, 10), (131_071, 32, 700, 300),
                                       (99_990, 200, 260, 40)])
def test_sieve_rows_by_cluster(api, nb, d, nq, k, metric):
    rng = np.random.default_rng(nb)
    mu = 3.0 * rng.standard_normal((30, d))
    xb = (mu[np.sort(rng.integers(0, 30, nb))] + rng.standard_normal((nb, d))).astype(np.float32)
    xq = (mu[29] + rng.standard_normal((nq, d))).astype(np.float32)
    check_all = np.unique(np.linspace(0, nq - 1, 12).astype(int))
    print(f"rows by cluster nb={nb} d={d} {metric}", flush=True)
    D, I = api.knn_search(dev(xq), dev(xb), k, metric)
    fails = check_rows(D.cpu().numpy()[check_all], I.cpu().numpy()[check_all], xq, xb, check_all, k, metric)
    assert not fails, fails[:10]


# rows nearer to the origin and further from it than the eight deviations from which on
# the pass takes them less a center, rows of one point, and a component out of its range
@pytest.mark.parametrize("kind", ["6", "9", "one point", "zeros", "huge component"])
@pytest.mark.parametrize("nb,d,nq,k", [(60_000, 64, 300, 100), (50_021, 130, 260, 10), (90_000, 256, 300, 300)])
def test_sieve_center(api, nb, d, nq, k, kind):
    rng = np.random.default_rng(nb + d)
    xb = rng.standard_normal((nb, d)).astype(np.float32)
    xq = rng.standard_normal((nq, d)).astype(np.float32)
    if kind in ("6", "9"):
        xb, xq = xb + np.float32(kind), xq + np.float32(kind)
    elif kind == "one point":
        xb[:] = 5.0 + xb[0]
        xb[::nb // 400] += rng.standard_normal((len(xb[::nb // 400]), d)).astype(np.float32)
        xq = xq + np.float32(5)
    elif kind == "zeros":
        xb[:] = 0.0
    else:
        xb[:, 3] = np.float32(2.0 ** 51)
        xq[:, 3] = np.float32(2.0 ** 51)
    rows = np.unique(np.linspace(0, nq - 1, 12).astype(int))
    print(f"center {kind} nb={nb} d={d}", flush=True)
    D, I = api.knn_search(dev(xq), dev(xb), k, "l2")
    if kind == "huge component":  # (nothing of the other components is left in a score)
        D64 = ((xq[rows, None].astype(np.float64) - xb[I.cpu().numpy()[rows]]) ** 2).sum(2)
        np.testing.assert_allclose(D.cpu().numpy()[rows], D64, rtol=gamma(d) * 4)
        return
    # (equal rows: the band reaches over all of them)
    fails = check_rows(D.cpu().numpy()[rows], I.cpu().numpy()[rows], xq, xb, rows, k, "l2", extra=nb - k)
    assert not fails, fails[:10]


# nearest row: queries that leave for the general search, entered into its list together by
# a workgroup's waves, the last of which may have no query at all
@pytest.mark.parametrize("d", [24, 96, 250])
@pytest.mark.parametrize("nq", [8192, 8193, 8215, 9001])
@pytest.mark.parametrize("every", [1, 3, 40])
def test_nearest_queries_left_together(api, d, nq, every):
    rng = np.random.default_rng(nq + d + every)
    x = dev(rng.standard_normal((nq, d)).astype(np.float32))
    c = dev(rng.standard_normal((700, d)).astype(np.float32))
    left = torch.zeros(nq, dtype=torch.bool, device="cuda")
    left[::every] = True
    left[-3:] = True
    y = torch.where(left[:, None], torch.full_like(x, float("nan")), x)
    print(f"nearest left together d={d} nq={nq} every={every}", flush=True)
    a, dist = api.kmeans_assign(x, c)
    a2, dist2 = api.kmeans_assign(y, c)
    part = y[left][:4000].contiguous()  # (too few for the nearest-row search)
    a3, dist3 = api.kmeans_assign(part, c)
    assert torch.equal(a2[~left], a[~left]) and torch.equal(dist2[~left], dist[~left])
    assert torch.equal(a2[left][:4000], a3)
    assert torch.equal(dist2[left][:4000].view(torch.int32), dist3.view(torch.int32))
