"""GPU parity of the row rotation on BF16 triples (many rows, d <= 128)."""
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


def dev(x):
    return torch.from_numpy(np.ascontiguousarray(x)).cuda()


def errors(out, x, rot):
    """Largest and mean |out - exact| / sum |rot x| (0 where that is 0)."""
    x, rot = x.astype(np.float64), rot.astype(np.float64)
    mag = np.abs(x) @ np.abs(rot).T
    e = np.abs(out.astype(np.float64) - x @ rot.T) / np.where(mag > 0, mag, 1.0)
    return e.max(), e.mean()


@pytest.mark.parametrize("n,d,dout", [(16_384, 128, 128), (20_001, 33, 65), (16_385, 100, 40),
                                      (30_003, 96, 600), (40_000, 64, 64), (16_400, 1, 1),
                                      (17_000, 31, 17), (17_000, 24, 16)])
def test_rotate_split(api, n, d, dout):
    print(f"rotate n={n} d={d} dout={dout}", flush=True)
    rng = np.random.default_rng(n + d + dout)
    x = (rng.standard_normal((n, d)) * np.exp(3 * rng.standard_normal((n, 1)))).astype(np.float32)
    rot = rng.standard_normal((dout, d)).astype(np.float32)
    out = api.rotate_rows(dev(x), dev(rot)).cpu().numpy()
    worst, mean = errors(out, x, rot)
    # the bound of an FP32 sum of d products
    assert worst <= (d + 2) * 2.0 ** -24
    # no further off than the FP32 products of smaller calls
    part = np.concatenate([api.rotate_rows(dev(x[i:i + 8000]), dev(rot)).cpu().numpy()
                           for i in range(0, n, 8000)])
    pw, pm = errors(part, x, rot)
    assert worst <= pw * 1.5 and mean <= pm * 1.01, (worst, pw, mean, pm)


def test_rotate_split_permutation_is_exact(api):
    rng = np.random.default_rng(1)
    x = rng.standard_normal((17_000, 96)).astype(np.float32)
    p = rng.permutation(96)
    rot = np.zeros((96, 96), np.float32)
    rot[np.arange(96), p] = 1.0
    np.testing.assert_array_equal(api.rotate_rows(dev(x), dev(rot)).cpu().numpy(), x[:, p])


def test_rotate_split_special_rows(api):
    # rows that triples cannot hold: as the FP32 products of smaller calls
    rng = np.random.default_rng(2)
    x = rng.standard_normal((16_500, 40)).astype(np.float32)
    rot = rng.standard_normal((24, 40)).astype(np.float32)
    x[5, 3], x[100, 0], x[200, 1], x[16_499, 7] = np.nan, np.inf, 1e30, -np.inf
    x[300] *= np.float32(1e-30)
    x[301, :20] = 0.0
    for bad in (None, 1e-25, 1e25, np.inf):
        if bad is not None:
            rot[3, 9] = bad
        out = api.rotate_rows(dev(x), dev(rot)).cpu().numpy()
        for lo in (0, 16_000):
            part = api.rotate_rows(dev(x[lo:lo + 500]), dev(rot)).cpu().numpy()
            np.testing.assert_allclose(out[lo:lo + 500], part, rtol=1e-5,
                                       atol=1e-5 * (bad if bad == 1e25 else 1.0))
        np.testing.assert_allclose(out[300], part_of(api, x[300:301], rot)[0], rtol=1e-4, atol=1e-36)


def part_of(api, x, rot):
    return api.rotate_rows(dev(x), dev(rot)).cpu().numpy()
