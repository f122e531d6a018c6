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
