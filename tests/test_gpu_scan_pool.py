"""GPU parity of the list scan's shared candidate pool against the float64
oracle: pool sizes, cuts, ties, odd numbers of sub-quantizers, short lists."""
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


def index(api, rng, n, d, nlist, M, copies=1):
    x = rng.standard_normal((n // copies, d)).astype(np.float32)
    x = np.ascontiguousarray(np.repeat(x, copies, axis=0))
    ix = api.IVFPQ(d, nlist, M)
    books = rng.standard_normal((M, 256, d // M)).astype(np.float32)
    ix.set_quantizers(x[rng.permutation(len(x))[:nlist]], books)
    ix.add(torch.from_numpy(x).cuda())
    return ix, x


# k at the pools' sizes and the cuts' steps; every vector of the second index
# stored 40 times (equal distances, ids break the ties)
@pytest.mark.parametrize("copies", [1, 40])
@pytest.mark.parametrize("M,k", [(16, 1), (16, 64), (16, 512), (16, 513), (16, 1024), (4, 100),
                                 (20, 256), (32, 700)])
def test_scan_pool(api, M, k, copies):
    print(f"scan pool M={M} k={k} copies={copies}", flush=True)
    rng = np.random.default_rng(M + k + copies)
    d = 2 * M
    ix, x = index(api, rng, 40_000, d, 13, M, copies)
    xq = rng.standard_normal((30, d)).astype(np.float32)
    coarse, books = ix.get_quantizers()
    offs, codes, ids = ix.get_lists()
    for nprobe in (1, 5):
        D, I = ix.search(torch.from_numpy(xq).cuda(), k, nprobe)
        Do, Io = oracle.ivfpq_search(xq, coarse, books, offs, codes, ids, k, nprobe)
        D, I = D.cpu().numpy().astype(np.float64), I.cpu().numpy()
        # sums of M + 2 terms in FP32 (term 1 holds M more), distances of a few d
        tol = (2 * M + 4) * 2.0 ** -24 * 8 * np.maximum(np.abs(Do), d)
        got = np.isfinite(Do)
        assert (np.abs(D[got] - Do[got]) <= tol[got]).all()
        assert ((I < 0) == (Io < 0)).all()
        if copies > 1:  # equal codes and lists: equal distances, ids in order
            full = I[:, :k // copies * copies].reshape(30, -1, copies)
            assert (np.diff(full, axis=2) == 1)[full[:, :, 1:] >= 0].all()
        # the same entries whatever the grouping
        ix.set_scan_options(lists_per_group=2)
        D2, I2 = ix.search(torch.from_numpy(xq).cuda(), k, nprobe)
        ix.set_scan_options()
        assert (I2.cpu().numpy() == I).all()


def test_scan_pool_rerank_from_scan(api):
    # one list of candidates per query goes straight to the re-rank
    rng = np.random.default_rng(5)
    ix, x = index(api, rng, 30_000, 32, 8, 8)
    xb = torch.from_numpy(x).cuda()
    xq = torch.from_numpy(rng.standard_normal((40, 32)).astype(np.float32)).cuda()
    for k, R in ((1, 1), (10, 100), (300, 300), (64, 1024)):
        out = []
        for g in (-1, 1):
            ix.set_scan_options(lists_per_group=g)
            out.append(ix.search_rerank(xq, k, 3, R, xb))
        assert torch.equal(out[0][0], out[1][0]) and torch.equal(out[0][1], out[1][1])


# lists of a group as one range of entries: more lists than one range takes (64),
# empty lists at its ends, ranges of less and more than a step of 1,024 entries
@pytest.mark.parametrize("M", [4, 16, 32])
@pytest.mark.parametrize("n,nlist", [(40, 150), (900, 150), (20_000, 150), (20_000, 64)])
def test_scan_ranges(api, M, n, nlist):
    print(f"scan ranges M={M} n={n} nlist={nlist}", flush=True)
    rng = np.random.default_rng(n + nlist + M)
    d = 2 * M
    x = rng.standard_normal((max(n, nlist), d)).astype(np.float32)
    ix = api.IVFPQ(d, nlist, M)
    ix.set_quantizers(x[:nlist], rng.standard_normal((M, 256, 2)).astype(np.float32))
    ix.add(torch.from_numpy(x[:n]).cuda())
    coarse, books = ix.get_quantizers()
    offs, codes, ids = ix.get_lists()
    xq = rng.standard_normal((9, d)).astype(np.float32)
    for nprobe, k in ((64, 20), (65, 300), (140, 100), (nlist, 600)):
        nprobe = min(nprobe, nlist)
        ix.set_scan_options(lists_per_group=-1)
        D, I = ix.search(torch.from_numpy(xq).cuda(), k, nprobe)
        ix.set_scan_options(lists_per_group=1)
        D1, I1 = ix.search(torch.from_numpy(xq).cuda(), k, nprobe)
        ix.set_scan_options()
        assert torch.equal(I, I1) and torch.equal(D, D1)
        Do, Io = oracle.ivfpq_search(xq, coarse, books, offs, codes, ids, k, nprobe)
        D, I = D.cpu().numpy().astype(np.float64), I.cpu().numpy()
        got = np.isfinite(Do)
        assert ((I < 0) == (Io < 0)).all()
        # sums of M + 2 terms in FP32 (term 1 holds M more), distances of a few d
        tol = (2 * M + 4) * 2.0 ** -24 * 8 * np.maximum(np.abs(Do), d)
        assert (np.abs(D[got] - Do[got]) <= tol[got]).all()
