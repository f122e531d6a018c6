// Threshold-first exact search of FP32 rows (sieve.hpp): host side.
#include <algorithm>

#include "dense.hpp"
#include "knn_classes.hpp"
#include "sieve.hpp"

namespace mk {

namespace {

template <int DP>
mk_status split_rows(const float* x, int64_t n, int32_t d, bool vec, int kind,
                     const float* yn, const float* center, int64_t sample_of, void* out,
                     float* scale, float* off, float* raw, uint32_t* bad, hipStream_t s) {
    const int64_t rows_per_block = 4 * (DP >= 96 ? 4 : 64 / (DP / 8));
    const int64_t blocks = ceil_div(n, rows_per_block);
    hipLaunchKernelGGL((split_rows_kernel<DP>), dim3((unsigned)(blocks < 16384 ? blocks : 16384)),
                       dim3(256), 0, s, x, n, d, (int32_t)vec, (int32_t)kind, yn, center, sample_of,
                       static_cast<unsigned char*>(out), scale, off, raw, bad);
    MK_LAUNCHED();
    return MK_OK;
}

}  // namespace

mk_status sieve_finish_any(const SieveScratch& w, const float* xq, int64_t nq, const float* xb,
                           int32_t d, bool vec, bool l2, int32_t k, int32_t keff, bool cert,
                           float* D, int64_t* I, hipStream_t s) {
    ProfScope prof("sieve_finish", s);
    if (keff <= 64) {
        hipLaunchKernelGGL(sieve_finish_wave, dim3((unsigned)ceil_div(nq, kMergeWaves)),
                           dim3(64 * kMergeWaves), 0, s, w.pool, w.cnt, w.cap, w.thr, w.thr_ld, xq, nq, xb, d,
                           (int32_t)vec, (int32_t)l2, k, keff, (int32_t)cert, w.err, w.qnorm, w.bad_db,
                           w.flags, w.rest, w.nrest, D, I);
        MK_LAUNCHED();
        return MK_OK;
    }
    auto kern = keff <= 256    ? sieve_finish<1024>
                : keff <= 1024 ? sieve_finish<2048>
                               : sieve_finish<4096>;
    hipLaunchKernelGGL(kern, dim3((unsigned)nq), dim3(kPoolThreads), 0, s, w.pool, w.cnt, w.cap, w.thr,
                       w.thr_ld, xq, xb, d, (int32_t)vec, (int32_t)l2, k, keff, (int32_t)cert, w.err, w.qnorm, w.bad_db,
                       w.flags, w.rest, w.nrest, D, I);
    MK_LAUNCHED();
    return MK_OK;
}

// The queries that are left (none, as a rule): few by the small-side search, more by
// the fused one.  Each has the caller's memory (256-byte aligned) as scratch, as far as
// it goes (an allocation between the launches costs some 10 us).
template <int DP>
static mk_status search_rest(const float* xq, int64_t nq, const float* xb, const float* yn, int64_t nb,
                             int32_t d, int32_t k, bool l2, bool vec, float* D, int64_t* I,
                             RestQueries rest, unsigned char* scratch, size_t bytes, hipStream_t s) {
    Arena first, second;
    first.base = second.base = scratch;
    first.size = second.size = bytes;
    {
        ArenaScope scope(&first);
        MK_TRY(dense_rest(xq, nq, xb, yn, nb, d, k, l2, vec, D, I, &rest, s));
    }
    if (rest.done >= nq) return MK_OK;
    ArenaScope scope(&second);
    return knn_dispatch_k<DP>(xq, nq, xb, yn, nb, d, k, l2, vec, D, I, s, nullptr, &rest);
}

// Exact search by thresholds (sieve.hpp); yn may be null (norms of the rows
// are then taken where the rows are split).
template <int DP>
mk_status sieve_dispatch(const float* xq, int64_t nq, const float* xb, const float* yn, int64_t nb,
                         int32_t d, int32_t k, bool l2, bool vec, float* D, int64_t* I,
                         hipStream_t s) {
    using S = SieveShape<SieveSplit, DP>;
    constexpr int64_t RB = DP * 4;  // bytes of a split row
    const int32_t keff = k + kSlack;
    const SievePlan plan = plan_sieve(nb, keff);
    // rows per launch: at most 512 MiB of split rows at a time
    const int64_t slab = std::min<int64_t>(nb, (512ll << 20) / RB / S::BN * S::BN);

    // one allocation, carved (each part 256-byte aligned): first what the search of the
    // queries that are left needs too; that search has the rest of it
    size_t used = 0;
    auto part = [&](size_t bytes) {
        const size_t at = used;
        used += (bytes + 255) & ~(size_t)255;
        return at;
    };
    const bool own_norms = l2 && !yn;
    const size_t o_w = part(sizeof(uint32_t) * (size_t)(3 * nq + 2));
    const size_t o_n = part(own_norms ? sizeof(float) * (size_t)nb : 0);
    const size_t kept = used;
    Scratch mem;
    const size_t o_q = part((size_t)(nq * RB)), o_s = part((size_t)(plan.sample * RB));
    const size_t o_y = part((size_t)(slab * RB)), o_qs = part(sizeof(float) * (size_t)nq);
    const size_t o_qn = part(sizeof(float) * (size_t)nq);
    const size_t o_ss = part(sizeof(float) * (size_t)plan.sample);
    const size_t o_so = part(sizeof(float) * (size_t)plan.sample);
    const size_t o_ys = part(sizeof(float) * (size_t)slab), o_yo = part(sizeof(float) * (size_t)slab);
    const size_t o_p = part(sizeof(uint64_t) * (size_t)(nq * plan.cap));
    const size_t o_sc = part(sizeof(float) * (size_t)(nq * (plan.sample / S::PER)));
    const size_t o_c = part(sizeof(float) * (kCenterOn + 1));
    const size_t o_t = part(sizeof(float) * (size_t)(nq * plan.rank));
    const size_t o_ti = part(sizeof(int64_t) * (size_t)(nq * plan.rank));
    used = std::max(used, kept + dense_rest_bytes(nq, nb, k));
    MK_TRY(mem.alloc(used, s));
    unsigned char* base = mem.as<unsigned char>();
    auto floats = [&](size_t at) { return reinterpret_cast<float*>(base + at); };
    void *qrows = base + o_q, *srows = base + o_s, *rows = base + o_y;
    float *qscale = floats(o_qs), *qnorm = floats(o_qn), *sscale = floats(o_ss);
    float *soff = floats(o_so), *yscale = floats(o_ys), *yoff = floats(o_yo);
    float *scores = floats(o_sc), *top = floats(o_t);
    float* norms = own_norms ? reinterpret_cast<float*>(base + o_n) : nullptr;
    uint32_t* words = reinterpret_cast<uint32_t*>(base + o_w);
    SieveScratch w;
    w.pool = reinterpret_cast<uint64_t*>(base + o_p);
    w.cap = (uint32_t)plan.cap;
    w.cnt = words;
    w.flags = w.cnt + nq;
    w.bad_db = w.flags + nq;
    w.nrest = w.bad_db + 1;
    w.rest = w.nrest + 1;
    w.qnorm = qnorm;
    float* center = l2 ? floats(o_c) : nullptr;
    MK_TRY(sieve_clear(words, 2 * nq + 2, xb, nb, d, center, s));
    const int kind = l2 ? kSplitDbL2 : kSplitDbIp;
    MK_TRY(split_rows<DP>(xq, nq, d, vec, kSplitQuery, nullptr, center, 0, qrows, qscale, qnorm, nullptr, w.flags, s));
    MK_TRY(split_rows<DP>(xb, plan.sample, d, vec, kind, yn, center, nb, srows, sscale, soff, nullptr, w.bad_db, s));

    SieveArgs a{};
    a.xq = qrows;
    a.qscale = qscale;
    a.qnorm = qnorm;
    a.nq = nq;
    a.nqb = (int32_t)ceil_div(nq, S::BQ);
    a.stride = (int32_t)RB;
    a.cnt = w.cnt;
    a.pool = w.pool;
    a.cap = w.cap;
    a.thr = top + (plan.rank - 1);
    a.thr_ld = plan.rank;
    a.flags = w.flags;
    a.bad_db = w.bad_db;
    w.thr = a.thr;
    w.thr_ld = a.thr_ld;
    w.err = split_err(DP);
    const double fk = (double)plan.sample / (double)nb * k;  // of the k best, in the sample
    a.tail = (float)(std::log(plan.rank / fk) / std::log((double)plan.rank));
    a.scores = scores;
    a.ld = plan.sample / S::PER;
    auto launch = [&](bool sample, const void* r, const float* ya, const float* yb, int64_t n,
                      int64_t row0) -> mk_status {
        a.xb = r;
        a.ya = ya;
        a.yb = yb;
        a.nb = n;
        a.row0 = (uint32_t)row0;
        int64_t nchunks;
        plan_sieve_chunks(a.nqb, n, S::BN, &nchunks, &a.chunk_len);
        a.nchunks = (int32_t)nchunks;
        ProfScope prof(sample ? "sieve_sample" : "sieve_tiles", s);
        auto kern = sample ? (l2 ? sieve_tiles<SieveSplit, DP, true, kSample> : sieve_tiles<SieveSplit, DP, false, kSample>)
                          : (l2 ? sieve_tiles<SieveSplit, DP, true, kFilter> : sieve_tiles<SieveSplit, DP, false, kFilter>);
        hipLaunchKernelGGL(kern, dim3((unsigned)(a.nqb * nchunks)), dim3(64 * S::WAVES), 0, s, a);
        MK_LAUNCHED();
        return MK_OK;
    };
    MK_TRY(launch(true, srows, sscale, soff, plan.sample, 0));
    MK_TRY(mk_kselect(scores, nq, a.ld, plan.rank, 0, top,
                      reinterpret_cast<int64_t*>(base + o_ti), s));
    for (int64_t r0 = 0; r0 < nb; r0 += slab) {
        const int64_t n = std::min(slab, nb - r0);
        MK_TRY(split_rows<DP>(xb + r0 * d, n, d, vec, kind, yn ? yn + r0 : nullptr, center, 0, rows,
                              yscale, yoff, norms ? norms + r0 : nullptr, w.bad_db, s));
        MK_TRY(launch(false, rows, yscale, yoff, n, r0));
    }
    MK_TRY(sieve_finish_any(w, xq, nq, xb, d, vec, l2, k, keff, true, D, I, s));
    return search_rest<DP>(xq, nq, xb, yn ? yn : norms, nb, d, k, l2, vec, D, I,
                           RestQueries{w.rest, w.nrest, 0}, base + kept, used - kept, s);
}


// Nearest row (k = 1, squared L2) of each query among few rows.
template <int DP>
mk_status nearest_dispatch(const float* xq, int64_t nq, const float* xb, const float* yn,
                           int64_t nb, int32_t d, bool vec, float* D, int64_t* I, hipStream_t s) {
    using S = SieveShape<SieveSplit, DP>;
    constexpr int64_t RB = DP * 4;
    size_t used = 0;
    auto part = [&](size_t bytes) {
        const size_t at = used;
        used += (bytes + 255) & ~(size_t)255;
        return at;
    };
    const size_t o_n = part(yn ? 0 : sizeof(float) * (size_t)nb);
    const size_t o_w = part(sizeof(uint32_t) * (size_t)(2 * nq + 2));
    const size_t kept = used;
    Scratch mem;
    const size_t o_q = part((size_t)(nq * RB)), o_y = part((size_t)(nb * RB));
    const size_t o_qs = part(sizeof(float) * (size_t)nq), o_qn = part(sizeof(float) * (size_t)nq);
    const size_t o_ys = part(sizeof(float) * (size_t)nb), o_yo = part(sizeof(float) * (size_t)nb);
    const size_t o_r = part(sizeof(uint4) * (size_t)nq), o_c = part(sizeof(float) * (kCenterOn + 1));
    used = std::max(used, kept + dense_rest_bytes(nq, nb, 1));
    MK_TRY(mem.alloc(used, s));
    unsigned char* base = mem.as<unsigned char>();
    auto floats = [&](size_t at) { return reinterpret_cast<float*>(base + at); };
    uint32_t* flags = reinterpret_cast<uint32_t*>(base + o_w);
    uint32_t *bad_db = flags + nq, *nrest = bad_db + 1;
    float* norms = yn ? nullptr : reinterpret_cast<float*>(base + o_n);
    MK_TRY(sieve_clear(flags, nq + 2, xb, nb, d, floats(o_c), s));
    MK_TRY(split_rows<DP>(xq, nq, d, vec, kSplitQuery, nullptr, floats(o_c), 0, base + o_q, floats(o_qs),
                          floats(o_qn), nullptr, flags, s));
    MK_TRY(split_rows<DP>(xb, nb, d, vec, kSplitDbL2, yn, floats(o_c), 0, base + o_y, floats(o_ys),
                          floats(o_yo), norms, bad_db, s));
    SieveArgs a{};
    a.xq = base + o_q;
    a.qscale = floats(o_qs);
    a.qnorm = floats(o_qn);
    a.xb = base + o_y;
    a.ya = floats(o_ys);
    a.yb = floats(o_yo);
    a.nq = nq;
    a.nb = nb;
    a.stride = (int32_t)RB;
    a.chunk_len = ceil_div(nb, S::BN) * S::BN;
    a.nchunks = 1;
    a.nqb = (int32_t)ceil_div(nq, S::BQ);
    a.near = reinterpret_cast<uint4*>(base + o_r);
    a.bad_db = bad_db;
    {
        ProfScope prof("sieve_nearest", s);
        hipLaunchKernelGGL((sieve_tiles<SieveSplit, DP, true, kNearest>), dim3((unsigned)a.nqb),
                           dim3(64 * S::WAVES), 0, s, a);
        MK_LAUNCHED();
    }
    hipLaunchKernelGGL(nearest_finish, dim3((unsigned)ceil_div(nq, 16)), dim3(256), 0, s, a.near,
                       xq, nq, xb, yn, (int32_t)nb, d, (int32_t)vec, split_err(DP), floats(o_qn), bad_db, flags, nrest + 1, nrest, D, I);
    MK_LAUNCHED();
    return search_rest<DP>(xq, nq, xb, yn ? yn : norms, nb, d, 1, true, vec, D, I,
                           RestQueries{nrest + 1, nrest, 0}, base + kept, used - kept, s);
}

#define MK_SIEVE_CLASS(DP)                                                                        \
    template mk_status sieve_dispatch<DP>(const float*, int64_t, const float*, const float*,      \
                                          int64_t, int32_t, int32_t, bool, bool, float*,          \
                                          int64_t*, hipStream_t);                                 \
    template mk_status nearest_dispatch<DP>(const float*, int64_t, const float*, const float*,    \
                                            int64_t, int32_t, bool, float*, int64_t*, hipStream_t);
MK_SIEVE_CLASS(32)
MK_SIEVE_CLASS(64)
MK_SIEVE_CLASS(96)
MK_SIEVE_CLASS(128)
MK_SIEVE_CLASS(256)
#undef MK_SIEVE_CLASS

}  // namespace mk
