"""GPU k-selection by pools on rows of few different values: every value equal to the
threshold's comes after the kept ones, so the lowest columns win."""
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


@pytest.mark.parametrize("largest", [False, True])
@pytest.mark.parametrize("k", [65, 512, 513, 1000])
@pytest.mark.parametrize("nrows,length", [(5, 2047), (40, 5000), (7, 70_001), (1200, 3333)])
@pytest.mark.parametrize("kind", ["few", "constant", "infinite", "ascending", "zeros", "offset"])
def test_pool_ties(api, kind, nrows, length, k, largest):
    rng = np.random.default_rng(length + k)
    a = rng.random((nrows, length)).astype(np.float32)
    if kind == "few":
        a = np.round(a * 4)
    elif kind == "constant":
        a[:] = 3.5
    elif kind == "infinite":
        a[a < 0.7] = np.inf
        a[a < 0.75] = -np.inf
    elif kind == "ascending":
        a = np.sort(np.round(a * 300), axis=1)
    elif kind == "zeros":
        a = np.where(a < 0.5, np.float32(0.0), np.float32(-0.0))
    else:
        a = np.float32(1e6) + a
    v, i = api.kselect(torch.from_numpy(a).cuda(), k, largest)
    want = np.argsort(-a if largest else a, axis=1, kind="stable")[:, :k]
    np.testing.assert_array_equal(i.cpu().numpy(), want)
    np.testing.assert_array_equal(v.cpu().numpy(), np.take_along_axis(a, want, 1))


# rows on both sides of the length up to which a wave's queue takes k = 65 to 128, shorter
# than k, empty, and off the 16-byte grid
@pytest.mark.parametrize("largest", [False, True])
@pytest.mark.parametrize("k", [65, 100, 128, 129])
@pytest.mark.parametrize("nrows,length", [(3, 0), (5, 40), (9, 127), (301, 128), (2, 511), (70, 512), (70, 513)])
@pytest.mark.parametrize("kind", ["random", "few", "signed"])
def test_short_rows(api, kind, nrows, length, k, largest):
    rng = np.random.default_rng(length + k)
    a = rng.random((nrows, length)).astype(np.float32)
    if kind == "few":
        a = np.round(a * 4)
    elif kind == "signed":
        a = np.exp(20 * a) * np.where(a < 0.4, np.float32(-1), np.float32(1))
    v, i = api.kselect(torch.from_numpy(a).cuda(), k, largest)
    n = min(k, length)
    want = np.argsort(-a if largest else a, axis=1, kind="stable")[:, :n]
    v, i = v.cpu().numpy(), i.cpu().numpy()
    np.testing.assert_array_equal(i[:, :n], want)
    np.testing.assert_array_equal(v[:, :n], np.take_along_axis(a, want, 1))
    assert (i[:, n:] == -1).all() and (v[:, n:] == (-np.inf if largest else np.inf)).all()
