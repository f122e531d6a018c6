"""Performance cases: the calls that a program built on this library spends its time in.

Every case goes through the public entry points of ``paper_1702_08734_amd.api`` with device-resident inputs.
Inputs follow the library's own synthetic workloads (``synth.py``): Gaussian mixtures with centres
N(0, 4 I) and per-component scales U[0.5, 1.5], unit-norm mixtures for the low-precision search, U[0, 1)
rows for the k-selection.  They are drawn on the GPU from the seed alone.
"""
from __future__ import annotations

import math

import torch

from paper_1702_08734_amd import api as mk

DEV = "cuda:0"
LARGEST = 10_000 * 1_000_000 * 128  # nq * nb * d of the largest exact search


def listed():
    return [
        # Online use, a small resident database: launches and latency count
        # (the 50,000 x 64 workload with 500 queries, k = 10).
        dict(name="exact_small", kind="exact", nq=500, nb=50_000, d=64, k=10, metric="l2",
             prenorm=False),
        # One query at a time against a million resident rows whose norms the
        # program keeps: one pass over the database.
        dict(name="exact_one", kind="exact", nq=1, nb=1_000_000, d=128, k=10, metric="l2",
             prenorm=True),
        # The headline batch: 10,000 queries against 1,000,000 x 128 (ground
        # truth, k-NN graphs), short result lists.
        dict(name="exact_batch", kind="exact", nq=10_000, nb=1_000_000, d=128, k=32, metric="l2",
             prenorm=False),
        # The same database with long result lists (candidate generation for
        # a later re-ranking stage).
        dict(name="exact_deep", kind="exact", nq=2_000, nb=1_000_000, d=128, k=1000, metric="l2",
             prenorm=False),
        # Inner products, a reduced dimension, and sizes that fill no tile.
        dict(name="exact_ragged_ip", kind="exact", nq=1_777, nb=300_007, d=100, k=100,
             metric="ip", prenorm=False),
        # Low-precision brute force with exact re-rank of 4 k candidates on a
        # database quantised once.
        dict(name="lowp_bf16", kind="lowp", nq=10_000, nb=2_000_000, d=96, k=100, R=400,
             prec="bf16", metric="ip"),
        dict(name="lowp_fp8", kind="lowp", nq=3_000, nb=2_000_000, d=96, k=100, R=400,
             prec="fp8", metric="l2"),
        # k-selection on a resident matrix (distances computed elsewhere).
        dict(name="kselect", kind="kselect", nrows=10_000, length=128_000, k=100, largest=False),
        # Index building: one k-means step over the training sample and the
        # product-quantizer encoding of its residuals.
        dict(name="index_build", kind="build", n=500_000, d=128, nlist=4096, M=16),
        # OPQ-style pre-processing of database rows.
        dict(name="rotate", kind="rotate", n=2_000_000, d=128, dout=128),
        # IVFADC: a large batch with exact re-rank, the setting that reaches
        # R@10 >= 0.9 on the 4,096-list workload.
        dict(name="ivf_rerank", kind="ivf", nq=10_000, nb=4_000_000, d=128, nlist=4096, M=16,
             k=10, nprobe=8, R=256),
        # IVFADC: a small online batch, ADC distances only.
        dict(name="ivf_online", kind="ivf", nq=64, nb=4_000_000, d=128, nlist=4096, M=16,
             k=100, nprobe=32, R=0),
    ]


def _log_int(rng, lo: int, hi: int) -> int:
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    kind = rng.choice(["exact", "exact", "exact", "lowp", "kselect", "build", "rotate", "ivf"])
    if kind == "exact":
        c = dict(kind=kind, nq=_log_int(rng, 1, 10_000), nb=_log_int(rng, 20_000, 1_000_000),
                 d=rng.choice([rng.randint(33, 128), 4 * rng.randint(16, 64), 64, 128]),
                 k=_log_int(rng, 1, 1000), metric=rng.choice(["l2", "ip"]),
                 prenorm=rng.random() < 0.5)
        while c["nq"] * c["nb"] * c["d"] > LARGEST:
            c["nq"] //= 2
        return c
    if kind == "lowp":
        k = _log_int(rng, 10, 200)
        return dict(kind=kind, nq=_log_int(rng, 500, 10_000), nb=_log_int(rng, 100_000, 2_000_000),
                    d=rng.choice([64, 96, rng.randint(48, 96)]), k=k, R=4 * k,
                    prec=rng.choice(["bf16", "fp8"]), metric=rng.choice(["l2", "ip"]))
    if kind == "kselect":
        length = _log_int(rng, 1_000, 128_000)
        return dict(kind=kind, nrows=_log_int(rng, 500, 10_000), length=length,
                    k=_log_int(rng, 1, min(1000, length)), largest=rng.random() < 0.5)
    if kind == "build":
        return dict(kind=kind, n=_log_int(rng, 50_000, 500_000), d=rng.choice([64, 96, 128]),
                    nlist=_log_int(rng, 256, 4096), M=rng.choice([8, 16, 32]))
    if kind == "rotate":
        d = rng.choice([64, 96, 128, rng.randint(48, 128)])
        return dict(kind=kind, n=_log_int(rng, 100_000, 2_000_000), d=d,
                    dout=rng.choice([d, max(16, d // 2), max(16, d - rng.randint(1, 31))]))
    k = _log_int(rng, 1, 100)
    R = rng.choice([0, 256])
    return dict(kind=kind, nq=_log_int(rng, 16, 10_000), nb=_log_int(rng, 500_000, 4_000_000),
                d=rng.choice([64, 96, 128]), nlist=rng.choice([1024, 2048, 4096]),
                M=rng.choice([8, 16, 32]), k=k, nprobe=_log_int(rng, 1, 32), R=R)


# ------------------------------------------------------------------ inputs
def _gen(seed: int) -> torch.Generator:
    return torch.Generator(device=DEV).manual_seed(seed)


class _Mixture:
    """1,000-component Gaussian mixture on the device (see synth.Mixture)."""

    def __init__(self, d: int, g: torch.Generator, ncomp: int = 1000):
        self.g = g
        self.mu = 2.0 * torch.randn((ncomp, d), device=DEV, generator=g)
        self.sigma = 0.5 + torch.rand((ncomp, 1), device=DEV, generator=g)

    def sample(self, n: int, unit_norm: bool = False) -> torch.Tensor:
        out = torch.empty((n, self.mu.shape[1]), device=DEV)
        for lo in range(0, n, 1 << 20):
            m = min(1 << 20, n - lo)
            comp = torch.randint(0, self.mu.shape[0], (m,), device=DEV, generator=self.g)
            v = torch.randn((m, self.mu.shape[1]), device=DEV, generator=self.g)
            v = v.mul_(self.sigma[comp]).add_(self.mu[comp])
            out[lo:lo + m] = v / v.norm(dim=1, keepdim=True) if unit_norm else v
        return out


def _inputs(case, seed: int):
    """The arrays of a case, from the seed alone."""
    g = _gen(seed)
    kind = case["kind"]
    if kind == "kselect":
        a = torch.rand((case["nrows"], case["length"]), device=DEV, generator=g)
        return {"a": a}
    mix = _Mixture(case["d"], g)
    if kind in ("exact", "lowp"):
        unit = kind == "lowp"
        return {"xb": mix.sample(case["nb"], unit), "xq": mix.sample(case["nq"], unit)}
    if kind == "rotate":
        # rows of a random orthogonal matrix, the first dout of them
        a = torch.randn((case["d"], case["d"]), generator=torch.Generator().manual_seed(seed),
                        dtype=torch.float64)
        q = torch.linalg.qr(a)[0][:case["dout"]]
        return {"x": mix.sample(case["n"]), "rot": q.float().contiguous().to(DEV)}
    n = case["n"] if kind == "build" else case["nb"]
    d, M = case["d"], case["M"]
    x = mix.sample(n)
    # quantizers drawn as k-means initialisations are: database rows for the
    # coarse ones, residual sub-vectors of other rows for the codebooks
    pick = torch.randperm(min(n, 200_000), device=DEV, generator=g)
    coarse = x[pick[:case["nlist"]]].contiguous()
    rows = x[pick[case["nlist"]:case["nlist"] + 4096]]
    near = torch.cdist(rows.double(), coarse.double()).argmin(1)
    res = (rows - coarse[near]).view(-1, M, d // M)
    books = torch.stack([res[torch.randperm(res.shape[0], device=DEV, generator=g)[:256], m]
                         for m in range(M)]).contiguous()
    out = {"x": x, "coarse": coarse, "books": books}
    if kind == "ivf":
        out["xq"] = mix.sample(case["nq"])
    return out


def prepare(case, seed: int):
    s = dict(_inputs(case, seed), case=case)
    if case["kind"] == "exact":
        s["yn"] = mk.norms(s["xb"]) if case["prenorm"] else None
    elif case["kind"] == "lowp":
        s["lp"], s["inv"] = mk.quantize_rows(s["xb"], case["prec"])
        s["yn"] = mk.norms(s["xb"])
    elif case["kind"] == "ivf":
        s["index"] = mk.IVFPQ(case["d"], case["nlist"], case["M"])
        s["index"].set_quantizers(s["coarse"].cpu().numpy(), s["books"].cpu().numpy())
        s["index"].add(s["x"])
    return s


def run(s):
    c = s["case"]
    kind = c["kind"]
    if kind == "exact":
        return mk.knn_search(s["xq"], s["xb"], c["k"], c["metric"], s["yn"])
    if kind == "lowp":
        return mk.knn_search_lowp(s["xq"], s["xb"], s["lp"], s["inv"], c["k"], c["R"], c["prec"],
                                  c["metric"], s["yn"])
    if kind == "kselect":
        return mk.kselect(s["a"], c["k"], c["largest"])
    if kind == "rotate":
        return mk.rotate_rows(s["x"], s["rot"])
    if kind == "build":
        assign, dist = mk.kmeans_assign(s["x"], s["coarse"])
        centroids, counts = mk.kmeans_update(s["x"], assign, s["coarse"])
        codes = mk.pq_encode(s["x"] - s["coarse"][assign], s["books"])
        return assign, dist, centroids, counts, codes
    if c["R"]:
        return s["index"].search_rerank(s["xq"], c["k"], c["nprobe"], c["R"], s["x"])
    return s["index"].search(s["xq"], c["k"], c["nprobe"])


def work(case):
    c, kind = case, case["kind"]
    if kind in ("exact", "lowp"):
        size = {"bf16": 2, "fp8": 1}.get(c.get("prec"), 4)
        return {"bytes": c["nb"] * c["d"] * size + c["nq"] * c["d"] * 4 + c["nq"] * c["k"] * 12,
                "flops": 2 * c["nq"] * c["nb"] * c["d"]}
    if kind == "kselect":
        return {"bytes": 4 * c["nrows"] * c["length"] + 12 * c["nrows"] * c["k"],
                "flops": c["nrows"] * c["length"]}
    if kind == "rotate":
        return {"bytes": 4 * c["n"] * (c["d"] + c["dout"]),
                "flops": 2 * c["n"] * c["d"] * c["dout"]}
    if kind == "build":
        # the rows are needed again once the assignment is known
        return {"bytes": 2 * 4 * c["n"] * c["d"] + 4 * c["nlist"] * c["d"] * 2
                + c["n"] * (12 + c["M"]),
                "flops": 2 * c["n"] * c["d"] * (c["nlist"] + 256 + 1)}
    scanned = c["nq"] * c["nprobe"] * c["nb"] / c["nlist"]
    return {"bytes": int(min(scanned, c["nb"]) * (c["M"] + 4) + 4 * c["nlist"] * c["d"]
                         + c["nq"] * (4 * c["d"] + 12 * c["k"]) + 4 * c["nq"] * c["R"] * c["d"]),
            "flops": int(2 * c["nq"] * c["d"] * (c["nlist"] + 256 + c["R"]) + scanned * c["M"])}


# ------------------------------------------------- 64-bit reference results
def _nearest64(xq, xb, k: int, metric: str):
    """Sorted squared L2 distances (or inner products) of the k best rows."""
    out = []
    xb = xb.double()
    yn = (xb * xb).sum(1)
    step = max(1, (1 << 28) // xb.shape[0])
    for lo in range(0, xq.shape[0], step):
        q = xq[lo:lo + step].double()
        p = q @ xb.T
        if metric == "ip":
            out.append(p.topk(k, dim=1).values)
        else:
            i = (yn - 2 * p).topk(k, dim=1, largest=False).indices
            for j in range(0, q.shape[0], 256):
                diff = xb[i[j:j + 256]] - q[j:j + 256, None]
                out.append((diff * diff).sum(2).sort(dim=1).values)
    return torch.cat(out)


def _assign64(x, coarse):
    c = coarse.double()
    cn = (c * c).sum(1)
    return torch.cat([(cn - 2 * (v.double() @ c.T)).argmin(1) for v in x.split(1 << 16)])


def _encode64(r, books):
    M, _, ds = books.shape
    b = books.double()
    bn = (b * b).sum(2)
    codes = torch.empty((r.shape[0], M), dtype=torch.int64, device=r.device)
    for lo in range(0, r.shape[0], 1 << 18):
        v = r[lo:lo + (1 << 18)].double().view(-1, M, ds)
        for m in range(M):
            codes[lo:lo + v.shape[0], m] = (bn[m] - 2 * (v[:, m] @ b[m].T)).argmin(1)
    return codes


def _ivf64(case, s):
    x, coarse, books, xq = s["x"], s["coarse"], s["books"], s["xq"]
    d, M, nlist, k = case["d"], case["M"], case["nlist"], case["k"]
    assign = _assign64(x, coarse)
    codes = torch.cat([_encode64(x[i:i + (1 << 19)] - coarse[assign[i:i + (1 << 19)]], books)
                       for i in range(0, x.shape[0], 1 << 19)])
    order = assign.argsort(stable=True)
    counts = torch.bincount(assign, minlength=nlist)
    start = counts.cumsum(0) - counts
    c64, b64 = coarse.double(), books.double()
    cn = (c64 * c64).sum(1)
    sub = torch.arange(M, device=x.device)
    out = torch.full((xq.shape[0], k), math.inf, dtype=torch.float64, device=x.device)
    lo = 0
    while lo < xq.shape[0]:
        q = xq[lo:lo + 512].double()
        probes = (cn - 2 * (q @ c64.T)).topk(case["nprobe"], dim=1, largest=False).indices
        # as many queries as keep 2^21 gathered entries
        total = counts[probes].sum(1).cumsum(0)
        n = max(1, int((total <= (1 << 21)).sum()))
        q, probes = q[:n], probes[:n]
        ln = counts[probes].flatten()
        owner = torch.arange(ln.numel(), device=x.device).repeat_interleave(ln)
        pos = torch.arange(owner.numel(), device=x.device) - (ln.cumsum(0) - ln)[owner]
        lists = probes.flatten()[owner]
        ids = order[start[lists] + pos]
        row = owner // case["nprobe"]
        rec = b64[sub, codes[ids]].reshape(ids.numel(), d) + c64[lists]
        adc = ((q[row] - rec) ** 2).sum(1)
        # the best R (or k) of each query by ADC distance, in sorted order
        keep = case["R"] or k
        by = adc.argsort()
        by = by[row[by].argsort(stable=True)]
        per = torch.bincount(row, minlength=n)
        rank = torch.arange(by.numel(), device=x.device) - (per.cumsum(0) - per)[row[by]]
        by, rank = by[rank < keep], rank[rank < keep]
        best = torch.full((n, keep), math.inf, dtype=torch.float64, device=x.device)
        if case["R"]:
            adc = ((x[ids[by]].double() - q[row[by]]) ** 2).sum(1)
            best[row[by], rank] = adc
        else:
            best[row[by], rank] = adc[by]
        out[lo:lo + n] = best.sort(dim=1).values[:, :k]
        lo += n
    return out


def exact(case, seed: int):
    s = _inputs(case, seed)
    kind = case["kind"]
    if kind in ("exact", "lowp"):
        # (indices of rows at equal rounded distances have no 64-bit value)
        return _nearest64(s["xq"], s["xb"], case["k"], case["metric"]), None
    if kind == "kselect":
        # values are copied, not computed
        v = torch.cat([r.topk(case["k"], dim=1, largest=case["largest"]).values.double()
                       for r in s["a"].split(1000)])
        return v, None
    if kind == "rotate":
        rot = s["rot"].double().T.contiguous()
        return torch.cat([v.double() @ rot for v in s["x"].split(1 << 18)])
    if kind == "build":
        x, coarse = s["x"], s["coarse"]
        assign = _assign64(x, coarse)
        dist = torch.cat([((v.double() - coarse[a].double()) ** 2).sum(1)
                          for v, a in zip(x.split(1 << 18), assign.split(1 << 18))])
        # (the centroids of clusters at a near-tie depend on which side a
        # point falls, so only the distances are compared)
        return None, dist, None, None, None
    return _ivf64(case, s), None
