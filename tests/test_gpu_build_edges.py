"""GPU checks of the index-building kernels at the ends of their ranges."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def api():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1702_08734_amd import api as a
    a.lib()
    return a


def test_update_more_clusters_than_a_grid(api):
    # 2^24 clusters of one point each (every cluster's mean is its point): a
    # workgroup per cluster would be more than 2^32 work items
    K, d = 1 << 24, 32
    print(f"kmeans_update K={K} d={d}", flush=True)
    x = torch.rand((K, d), device="cuda")
    assign = (torch.arange(K, device="cuda") * 2654435761) % K  # odd factor: a permutation
    c, counts = api.kmeans_update(x, assign, torch.zeros((K, d), device="cuda"))
    assert (counts == 1).all()
    assert torch.equal(c[assign], x)


# points in the order of their clusters, all in one, half in one, and points that are
# ignored: the sums by cluster put waves of them in order at once
@pytest.mark.parametrize("kind", ["sorted", "one", "half", "even", "ignored"])
@pytest.mark.parametrize("n,K,d", [(4099, 5, 32), (100_003, 700, 64), (70_000, 16, 36)])
def test_update_orders(api, kind, n, K, d):
    rng = np.random.default_rng(n + K)
    x = rng.integers(-8, 9, size=(n, d)).astype(np.float32)
    a = rng.integers(0, K, n)
    if kind == "sorted":
        a = np.sort(a)
    elif kind == "one":
        a[:] = K // 2
    elif kind == "half":
        a[rng.random(n) < 0.5] = 1
    elif kind == "ignored":
        a[::3] = -1
        a[1::7] = K
    print(f"update {kind} n={n} K={K} d={d}", flush=True)
    c, counts = api.kmeans_update(torch.from_numpy(x).cuda(), torch.from_numpy(a).cuda(),
                                  torch.zeros((K, d), device="cuda"))
    live = (a >= 0) & (a < K)
    want = np.bincount(a[live], minlength=K)
    sums = np.zeros((K, d))
    np.add.at(sums, a[live], x[live].astype(np.float64))
    if kind != "one":  # (an empty cluster splits another)
        assert (want > 0).all() and (counts.cpu().numpy() == want).all()
        np.testing.assert_array_equal(c.cpu().numpy(), (sums / want[:, None]).astype(np.float32))
    else:
        assert counts.sum().item() == n
        np.testing.assert_allclose(c.cpu().numpy()[K // 2], sums[K // 2] / n, rtol=0.02, atol=1e-6)


# rows and code words whose nearest word the products cannot tell (ties, repeated words,
# components out of the split's range, rows of NaN, rows far from the origin): the codes of
# the plain kernel, which calls of fewer than 2,048 rows take
@pytest.mark.parametrize("kind", ["integers", "repeated", "tiny", "tiny rows", "nan rows", "far", "mixed"])
@pytest.mark.parametrize("M,ds", [(4, 2), (4, 3), (8, 4), (4, 5), (8, 8), (4, 12), (4, 16)])
def test_encode_without_proof(api, kind, M, ds):
    rng = np.random.default_rng(M * ds)
    n = 20_003
    r = rng.standard_normal((n, M * ds)).astype(np.float32)
    books = rng.standard_normal((M, 256, ds)).astype(np.float32)
    if kind == "integers":
        r, books = np.round(r), np.round(books)
    elif kind == "repeated":
        books[:, 128:] = books[:, :128]
        books[:, 3] = books[:, 200]
    elif kind == "tiny":
        r, books = r * np.float32(1e-20), books * np.float32(1e-20)
    elif kind == "tiny rows":
        r *= np.float32(1e-20)
    elif kind == "nan rows":
        r[::9, 1] = np.nan
    elif kind == "far":
        r, books = r + np.float32(300), books + np.float32(300)
    else:  # stretches of rows with and without
        r[4000:9000] = np.round(r[4000:9000])
        books[:, ::2] = np.round(books[:, ::2])
        r[12_000:12_100] = np.inf
    print(f"encode {kind} M={M} ds={ds}", flush=True)
    rd, bd = torch.from_numpy(r).cuda(), torch.from_numpy(books).cuda()
    codes = api.pq_encode(rd, bd)
    part = torch.cat([api.pq_encode(rd[i:i + 2000].contiguous(), bd) for i in range(0, n, 2000)])
    assert torch.equal(codes, part)


# both sides of the cluster count up to which workgroups count in LDS, of its chunk, and of
# the sizes from which sums go by cluster at all
@pytest.mark.parametrize("kind", ["even", "sorted", "half"])
@pytest.mark.parametrize("n,K", [(4096, 1), (4097, 2), (4097, 1024), (22_001, 30), (21_000, 30), (32_768, 1024),
                                 (32_769, 1024), (40_000, 1025), (300_007, 256)])
def test_update_counts(api, n, K, kind):
    rng = np.random.default_rng(n)
    d = 32
    x = rng.integers(-8, 9, size=(n, d)).astype(np.float32)
    a = rng.integers(0, K, n)
    if kind == "half":
        a[rng.random(n) < 0.5] = K - 1
    a[:K] = rng.permutation(K)
    if kind == "sorted":
        a = np.sort(a)
    a[K + 5:K + 50:9] = -1
    a[K + 60] = K
    print(f"update counts {kind} n={n} K={K}", flush=True)
    c, counts = api.kmeans_update(torch.from_numpy(x).cuda(), torch.from_numpy(a).cuda(),
                                  torch.zeros((K, d), device="cuda"))
    live = (a >= 0) & (a < K)
    want = np.bincount(a[live], minlength=K)
    assert (want > 0).all()  # (an empty cluster splits another)
    sums = np.zeros((K, d))
    np.add.at(sums, a[live], x[live].astype(np.float64))
    assert (counts.cpu().numpy() == want).all()
    np.testing.assert_array_equal(c.cpu().numpy(), (sums / want[:, None]).astype(np.float32))
