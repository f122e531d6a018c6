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
