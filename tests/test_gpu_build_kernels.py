"""GPU parity of the index-building kernels that large inputs take: encoding on
the matrix cores against the plain kernel (calls of few rows), sums by cluster
against float64, and the empty-cluster rule against the oracle."""
import numpy as np
import pytest

import oracle

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


@pytest.mark.parametrize("n,M,ds", [(2048, 4, 2), (2049, 8, 3), (5000, 16, 8), (4099, 20, 5),
                                    (70_001, 4, 8), (3001, 8, 12), (9000, 4, 16), (2100, 128, 4)])
def test_encode_equals_plain_kernel(api, n, M, ds):
    print(f"encode n={n} M={M} ds={ds}", flush=True)
    rng = np.random.default_rng(n + M + ds)
    r = rng.standard_normal((n, M * ds)).astype(np.float32)
    books = rng.standard_normal((M, 256, ds)).astype(np.float32)
    books[:, 200] = books[:, 3]               # equal code words: the lower index
    books[1] = np.round(books[1])             # exact ties
    r[:, ds:2 * ds] = np.round(r[:, ds:2 * ds])
    books[2] *= np.float32(1e-3) ** rng.integers(0, 9, (256, 1))  # norms 1e-24 apart
    r[7] = 0.0
    r[8, 0], r[9, 0], r[10, 0] = np.nan, np.inf, 1e30
    r[11] *= np.float32(1e-25)
    r[12, :ds] = books[0, 77]
    codes = api.pq_encode(dev(r), dev(books)).cpu().numpy()
    part = [api.pq_encode(dev(r[i:i + 1500]), dev(books)).cpu().numpy() for i in (0, n - 1500)]
    np.testing.assert_array_equal(codes[:1500], part[0])
    np.testing.assert_array_equal(codes[n - 1500:], part[1])
    rows = np.arange(13, n, 397)
    np.testing.assert_array_equal(codes[rows][:, 0], oracle.pq_encode(r[rows], books)[:, 0])


def test_encode_code_words_not_finite(api):
    rng = np.random.default_rng(3)
    r = rng.standard_normal((4000, 32)).astype(np.float32)
    books = rng.standard_normal((4, 256, 8)).astype(np.float32)
    books[0, 5, 1], books[1, 6, 2], books[2, 7, 3] = np.nan, np.inf, 3e38
    codes = api.pq_encode(dev(r), dev(books)).cpu().numpy()
    for lo in (0, 2500):
        part = api.pq_encode(dev(r[lo:lo + 1500]), dev(books)).cpu().numpy()
        np.testing.assert_array_equal(codes[lo:lo + 1500], part)


@pytest.mark.parametrize("n,d,K", [(4096, 32, 1), (20_001, 64, 7), (30_000, 36, 2000),
                                   (5000, 1024, 3), (9000, 128, 9000)])
def test_update_by_cluster(api, n, d, K):
    print(f"update n={n} d={d} K={K}", flush=True)
    rng = np.random.default_rng(n + K)
    x = rng.standard_normal((n, d)).astype(np.float32)
    # most points in one cluster (many stretches), some ignored, some clusters empty
    a = np.where(rng.random(n) < 0.7, 0, rng.integers(0, K, n)).astype(np.int64)
    a[::50] = -1
    a[1::50] = K
    c0 = rng.standard_normal((K, d)).astype(np.float32)
    c, counts = api.kmeans_update(dev(x), dev(a), dev(c0))
    valid = (a >= 0) & (a < K)
    co, no = oracle.kmeans_update(x[valid], a[valid], c0)
    np.testing.assert_array_equal(counts.cpu().numpy(), no)
    # FP64 sums in another order: at most one unit of the last FP32 place
    np.testing.assert_allclose(c.cpu().numpy(), co, rtol=2.0 ** -22, atol=1e-12)
