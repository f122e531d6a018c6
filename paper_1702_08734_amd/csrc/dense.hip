// Exact search where either side is small: few queries over any database, or
// any number over a few thousand rows (the coarse search of an IVF index).
//
//   1. quad_min_kernel: FP32 products (v_mfma_f32_16x16x4f32, the fused kernel's
//      products in its order) of every query with every row, straight from
//      memory to the matrix operands; of every four rows the least score is
//      stored.  One read of the database, nq * nb bytes written.
//   2. The k + 16 best groups of four.  A row of the k best has at most k - 1 groups
//      before its own, so these groups hold every candidate that the fused search
//      would keep.
//   3. Direct-form FP32 distances of the groups' rows, the k best written.
// 2 and 3 are one kernel (a wave or a workgroup per query); where few queries have
// long rows of minima, workgroups first select in segments of them.
//
// Bound by memory for few queries: one query over 10^6 x 128 rows, k = 10: 130 us
// (the rows' read 96 us, 5.3 TB/s; selections and finish in two kernels 24 us less
// than in three) against 2,422 us by the fused search, which has 16 workgroups for
// it (one per chunk).  By the FP32 matrix products for many: 10^4 queries over
// 4,096 x 128 centroids, k = 8: products 135 us, selection and finish 93 us (by a
// workgroup per query 150 us) against 450 us by the fused search.
#include <algorithm>
#include <cmath>
#include <type_traits>

#include "dense.hpp"
#include "fused.hpp"
#include "kselect.hpp"
#include "pool.hpp"

namespace mk {

namespace {

// Queries list[first .. min(*count, first + most)) of those left by another search;
// none where there are more than limit.
struct RestSpan {
    const uint32_t* list;
    const uint32_t* count;
    int64_t first, most, limit;
    __device__ __forceinline__ int64_t size() const {
        const int64_t n = *count;
        if (n > limit || n <= first) return 0;
        return n - first < most ? n - first : most;
    }
    __device__ __forceinline__ int64_t at(int64_t i) const { return list[first + i]; }
};

struct QuadArgs {
    const float* xq;
    const float* xb;
    const float* yn;  // ||y||^2 (L2; null: computed from the rows read)
    int64_t nq, nb;
    int32_t d;
    int64_t groups;           // of 64 rows
    int64_t groups_per_wave;
    int32_t nqb;              // query blocks of 16 QB
    float* out;               // [nq][ld] least score of four rows
    int64_t ld;
    RestSpan rest;            // REST: these queries in the place of 0 .. nq - 1
};

// Groups of 64 rows per wave for more than 16 queries: four waves per SIMD's worth,
// for an even end (fewer than 8,192 + nqb waves).
__host__ __device__ inline int64_t quad_groups(int64_t groups, int64_t nqb) {
    const int64_t n = groups * nqb / 4096;
    return n > 1 ? n : 1;
}

enum class QuadNorms { kNone, kGiven, kOwn };  // inner products; L2 with and without yn
// A wave takes 16 QB queries (B operands, in registers) and streams its rows 64
// at a time: block b of four, A row m is row 16 (m / 4) + 4 b + m % 4 of them, so
// that lane (query li, quarter lh) ends up with groups 4 lh .. 4 lh + 3 of four
// consecutive rows: one 16-byte store.  The next block's rows are loaded while
// this block's products run.  No load is under a branch (rows and granules beyond
// the end are clamped, and made zero or given no score), so that the waits before
// the products are for this block's rows alone: with branches the compiler waited
// for everything in flight, and kept twice the registers (500 queries, 50,000 x 64
// rows: 69 -> 47 us; 10^4 queries, 4,096 x 128 rows 175 -> 135 us, half of the
// matrix cores' rate).
// REST: the queries of a list (by itself: asked at run time, the searches without one
// took 80.6 us, 77.6 so: 500 queries, 50,000 x 64 rows).
template <int DP, int QB, bool VEC, QuadNorms NORMS, bool REST>
__global__ __launch_bounds__(256)
__attribute__((amdgpu_waves_per_eu(DP <= 32 || (DP <= 64 && QB == 1) ? 3 : DP <= 128 ? 2 : 1))) void
quad_min_kernel(QuadArgs a) {
    constexpr bool L2 = NORMS != QuadNorms::kNone;
    constexpr int S4 = DP / 16;  // granule steps of four floats per lane
    const int lane = lane_id(), li = lane & 15, lh = lane >> 4;
    if constexpr (REST) {
        a.nq = a.rest.size();
        if (a.nq == 0) return;
        a.nqb = (int32_t)((a.nq + 16 * QB - 1) / (16 * QB));
        a.groups_per_wave = quad_groups(a.groups, a.nqb);
    }
    const int64_t w = (int64_t)blockIdx.x * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    // neighbouring waves: the query blocks of one stretch of rows
    const int64_t q0 = (w % a.nqb) * (16 * QB);
    const int64_t g0 = (w / a.nqb) * a.groups_per_wave;
    const int64_t g1 = g0 + a.groups_per_wave < a.groups ? g0 + a.groups_per_wave : a.groups;
    if (g0 >= g1) return;

    uint4 q[QB][S4];
#pragma unroll
    for (int qb = 0; qb < QB; ++qb) {
        const int64_t i = q0 + qb * 16 + li;
        const bool ok = i < a.nq;
        const float* row = a.xq + (!ok ? 0 : REST ? a.rest.at(i) : i) * a.d;
#pragma unroll
        for (int s = 0; s < S4; ++s) q[qb][s] = load_granule<OpF32, VEC>(row, 4 * s + lh, a.d, ok);
    }
    // (d > DP - 32, or more than 128 for DP = 256: the first granules always exist)
    constexpr int WHOLE = DP > 128 ? 8 : S4 - 2;
    auto load = [&](int64_t g, int b, uint4 (&y)[S4]) __attribute__((always_inline)) {
        int64_t r = g * 64 + 16 * (li >> 2) + 4 * b + (li & 3);
        r = r < a.nb ? r : a.nb - 1;
        const float* row = a.xb + r * a.d;
#pragma unroll
        for (int s = 0; s < S4; ++s) {
            if constexpr (VEC) {
                const int e = 16 * s + 4 * lh;
                y[s] = *reinterpret_cast<const uint4*>(row + (s < WHOLE || e < a.d ? e : a.d - 4));
            } else {
                y[s] = load_granule<OpF32, false>(row, 4 * s + lh, a.d, true);
            }
        }
    };
    uint4 y[2][S4];
    load(g0, 0, y[0]);
#pragma unroll 1
    for (int64_t g = g0; g < g1; ++g) {
        float least[QB][4];
#pragma unroll
        for (int b = 0; b < 4; ++b) {
            uint4 (&now)[S4] = y[b & 1];
            __builtin_amdgcn_sched_barrier(0);  // (loads further ahead cost registers)
            const int64_t r = g * 64 + 16 * lh + 4 * b;  // first of this lane's four rows
            float add[4] = {0.f, 0.f, 0.f, 0.f};
            if constexpr (NORMS == QuadNorms::kGiven)
#pragma unroll
                for (int i = 0; i < 4; ++i) add[i] = a.yn[r + i < a.nb ? r + i : a.nb - 1];
            // (the last group's last block loads its own rows again)
            load(b < 3 || g + 1 == g1 ? g : g + 1, (b + 1) & 3, y[(b + 1) & 1]);
            if constexpr (VEC)
#pragma unroll
                for (int s = WHOLE; s < S4; ++s)
                    if (16 * s + 4 * lh >= a.d) now[s] = make_uint4(0, 0, 0, 0);
            if constexpr (NORMS == QuadNorms::kOwn) {
                float s2 = 0.f;
#pragma unroll
                for (int s = 0; s < S4; ++s) {
                    const float e0 = __uint_as_float(now[s].x), e1 = __uint_as_float(now[s].y);
                    const float e2 = __uint_as_float(now[s].z), e3 = __uint_as_float(now[s].w);
                    s2 = fmaf(e0, e0, s2);
                    s2 = fmaf(e1, e1, s2);
                    s2 = fmaf(e2, e2, s2);
                    s2 = fmaf(e3, e3, s2);
                }
                s2 += __shfl_xor(s2, 16);
                s2 += __shfl_xor(s2, 32);
#pragma unroll
                for (int i = 0; i < 4; ++i) add[i] = __shfl(s2, 4 * lh + i);
            }
            floatx4 acc[QB];
#pragma unroll
            for (int qb = 0; qb < QB; ++qb) acc[qb] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int s = 0; s < S4; ++s)
#pragma unroll
                for (int qb = 0; qb < QB; ++qb) acc[qb] = OpF32::mma(acc[qb], now[s], q[qb][s]);
#pragma unroll
            for (int i = 0; i < 4; ++i) add[i] = r + i < a.nb ? add[i] : INFINITY;
#pragma unroll
            for (int qb = 0; qb < QB; ++qb) {
                float m = INFINITY;
                bool first = false;
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const float sc = fmaf(L2 ? -2.f : -1.f, acc[qb][i], add[i]);
                    // A NaN is left out, as by the fused search, but for two kinds:
                    // rows whose norm and product overflow (their direct distance
                    // may not), and, beside rows with a score, inner products whose
                    // NaN has a key before all numbers.
                    first |= sc != sc && r + i < a.nb &&
                             (L2 ? add[i] == INFINITY : !(__float_as_uint(acc[qb][i]) >> 31));
                    m = fminf(m, sc);
                }
                if (first && (L2 || m < INFINITY)) m = -INFINITY;
                least[qb][b] = m;
            }
        }
#pragma unroll
        for (int qb = 0; qb < QB; ++qb) {
            const int64_t i = q0 + qb * 16 + li;
            if (i < a.nq)
                *reinterpret_cast<float4*>(&a.out[i * a.ld + g * 16 + 4 * lh]) =
                    make_float4(least[qb][0], least[qb][1], least[qb][2], least[qb][3]);
        }
    }
}

// Row r in the place of its group's key; whether its direct value counts: a NaN only
// where it made its group the first of the inner products.
__device__ __forceinline__ uint64_t row_key(uint64_t group, int64_t r) {
    return (group & ~0xFFFFFFFFull) | (uint64_t)r;
}
__device__ __forceinline__ bool is_distance(float v, uint64_t key, int32_t l2) {
    return v == v || (!l2 && key_score(key) == -INFINITY);
}

// Steps 2 and 3 by a workgroup per query: the kq best groups, from the row of group minima itself
// (lists null) or from the nlists lists of kq keys of a first pass over its
// segments; exact distances of the groups' rows (16 rows per wave and step, as in
// the fused search's re-rank); the k best of them by (distance, row).
template <int P, int U, int N, bool REST>  // kq <= P - 1024 U, kq <= P / 2, 4 kq <= N <= P
__global__ __launch_bounds__(kPoolThreads) void quad_finish_kernel(
    const float* __restrict__ least, int64_t ld, const uint64_t* __restrict__ lists,
    int32_t nlists, int32_t kq, const float* __restrict__ xq, const float* __restrict__ xb,
    const float* __restrict__ yn, int64_t nb, int32_t d, int32_t vec, int32_t l2, int32_t k,
    RestSpan rest, float* __restrict__ D, int64_t* __restrict__ I) {
    __shared__ __align__(16) float xs[kMaxDim];
    __shared__ uint64_t pool[P];
    __shared__ float dist[N];
    __shared__ uint32_t bins[kCutBins];
    __shared__ PoolState st;
    __shared__ uint32_t ws[2][kPoolWaves];
    const int tid = threadIdx.x;
    const int64_t i = blockIdx.x;
    int64_t q = i;
    if constexpr (REST) {
        if (i >= rest.size()) return;
        q = rest.at(i);
    }
    for (int t = tid; t < d; t += kPoolThreads) xs[t] = xq[q * d + t];
    uint32_t found;
    if (lists) {
        uint64_t limit;
        found = pool_stream<P>(lists + i * (int64_t)nlists * kq, (int64_t)nlists * kq, pool, bins,
                               &st, kq, limit);
    } else {
        found = pool_values<P, U, false>(least + i * ld, (uint32_t)ld, 0u, kq, pool, bins, &st, ws);
        if (found > (uint32_t)kq) {
            pool_cut<P>(pool, bins, &st, found, kq);
            found = (uint32_t)kq;
        }
    }
    __syncthreads();
    // the groups' rows in the groups' place
    const int n = 4 * (int)found;
    uint64_t row[N / kPoolThreads];
#pragma unroll
    for (int j = 0; j < N / kPoolThreads; ++j) {
        const int e = j * kPoolThreads + tid;
        row[j] = kSentinel;
        if (e >= n || pool[e >> 2] == kSentinel) continue;
        const int64_t r = 4 * (int64_t)key_index(pool[e >> 2]) + (e & 3);
        if (r < nb && has_score(yn, xb, r, d)) row[j] = row_key(pool[e >> 2], r);
    }
    __syncthreads();
#pragma unroll
    for (int j = 0; j < N / kPoolThreads; ++j) {
        const int e = j * kPoolThreads + tid;
        if (e < n) pool[e] = row[j];
    }
    if (tid == 0) st.count = 0u;
    __syncthreads();
#pragma unroll 1
    for (int e0 = 16 * (tid >> 6); e0 < n; e0 += 16 * kPoolWaves)
        rerank_rows16(xs, pool, e0, n, xb, d, vec, l2, dist);
    __syncthreads();
    // live rows to the front
    uint64_t key[N / kPoolThreads];
#pragma unroll
    for (int j = 0; j < N / kPoolThreads; ++j) {
        const int e = j * kPoolThreads + tid;
        key[j] = kSentinel;
        if (e < n && pool[e] != kSentinel && is_distance(dist[e], pool[e], l2))
            key[j] = make_key(l2 ? dist[e] : -dist[e], (uint32_t)pool[e]);
    }
    __syncthreads();
#pragma unroll
    for (int j = 0; j < N / kPoolThreads; ++j)
        if (key[j] != kSentinel) pool[atomicAdd(&st.count, 1u)] = key[j];
    __syncthreads();
    const uint32_t have = st.count;
    float* Dq = D + q * k;
    int64_t* Iq = I + q * k;
    pool_emit<P>(pool, bins, &st, have, (uint32_t)k, [&](uint32_t r, uint64_t key) {
        const float s = key_score(key);
        Dq[r] = l2 ? s : -s;
        Iq[r] = (int64_t)key_index(key);
    });
    for (int e = tid; e < k; e += kPoolThreads)
        if (e >= (int)have) {
            Dq[e] = l2 ? INFINITY : -INFINITY;
            Iq[e] = -1;
        }
}

// The same with one wave per query and sorted register queues, for kq <= 64 and
// whole rows: no barriers, so it is the better one where there are more queries
// than the chip takes workgroups at a time.
__global__ __launch_bounds__(64 * kMergeWaves) void quad_finish_wave(
    const float* __restrict__ least, int64_t ld, int64_t nq, int32_t kq,
    const float* __restrict__ xq, const float* __restrict__ xb, const float* __restrict__ yn,
    int64_t nb, int32_t d, int32_t vec, int32_t l2, int32_t k, float* __restrict__ D,
    int64_t* __restrict__ I) {
    constexpr int T = SelParams<1>::T;
    __shared__ __align__(16) float xs[kMergeWaves][kMaxDim];
    __shared__ uint64_t kl[kMergeWaves][256];
    __shared__ float dist[kMergeWaves][256];
    const int wave = threadIdx.x >> 6, lane = lane_id();
    const int64_t q = (int64_t)blockIdx.x * kMergeWaves + wave;
    if (q >= nq) return;
    for (int t = lane; t < d; t += 64) xs[wave][t] = xq[q * d + t];
    const float* row = least + q * ld;
    WaveSelect<1, T> ws;
    ws.init(kq);
    constexpr int AHEAD = 4;  // values in flight per lane
    auto value = [&](int64_t e) { return e + lane < ld ? row[e + lane] : INFINITY; };
    float v[AHEAD];
#pragma unroll
    for (int j = 0; j < AHEAD; ++j) v[j] = value(64 * j);
#pragma unroll 1
    for (int64_t e = 0; e < ld; e += 64) {
        const float now = v[0];
#pragma unroll
        for (int j = 0; j + 1 < AHEAD; ++j) v[j] = v[j + 1];
        v[AHEAD - 1] = value(e + 64 * AHEAD);
        const uint64_t key = e + lane < ld ? make_key(now, (uint32_t)(e + lane)) : kSentinel;
        if (ws.push(key)) ws.merge();
    }
    ws.finish();
    // the groups' rows
    const uint64_t group = ws.w[0];
    const int n = 4 * kq;
    if (lane < kq) {
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int64_t r = 4 * (int64_t)key_index(group) + j;
            kl[wave][4 * lane + j] =
                group != kSentinel && r < nb && has_score(yn, xb, r, d) ? row_key(group, r) : kSentinel;
        }
    }
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "workgroup");
#pragma unroll 1
    for (int e0 = 0; e0 < n; e0 += 16) rerank_rows16(xs[wave], kl[wave], e0, n, xb, d, vec, l2, dist[wave]);
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "workgroup");
    ws.init(k);
#pragma unroll 1
    for (int e0 = 0; e0 < n; e0 += 64) {
        const int e = e0 + lane;
        uint64_t key = kSentinel;
        if (e < n && kl[wave][e] != kSentinel && is_distance(dist[wave][e], kl[wave][e], l2))
            key = make_key(l2 ? dist[wave][e] : -dist[wave][e], (uint32_t)kl[wave][e]);
        if (ws.push(key)) ws.merge();
    }
    ws.finish();
    emit_reranked<1>(ws.w, k, l2, D + q * k, I + q * k);
}

template <int DP, int QB, bool REST = false>
mk_status launch_quads(const QuadArgs& a, bool vec, bool l2, int64_t waves, hipStream_t s) {
    ProfScope prof("dense_quads", s);
    auto of = [&](auto v) {
        constexpr bool V = decltype(v)::value;
        return !l2    ? quad_min_kernel<DP, QB, V, QuadNorms::kNone, REST>
               : a.yn ? quad_min_kernel<DP, QB, V, QuadNorms::kGiven, REST>
                      : quad_min_kernel<DP, QB, V, QuadNorms::kOwn, REST>;
    };
    auto kern = vec ? of(std::true_type{}) : of(std::false_type{});
    hipLaunchKernelGGL(kern, dim3((unsigned)ceil_div(waves, 4)), dim3(256), 0, s, a);
    MK_LAUNCHED();
    return MK_OK;
}

template <int DP>
mk_status quads(QuadArgs a, bool vec, bool l2, hipStream_t s) {
    // query blocks of 64 (32 for wide rows), or 16 when that is all there is
    constexpr int WIDE = DP > 96 ? 2 : 4;
    const int qb = a.nq <= 16 ? 1 : WIDE;
    a.nqb = (int32_t)ceil_div(a.nq, 16 * qb);
    if (a.rest.list) {  // (how many there are is known on the device)
        const int64_t waves = std::min<int64_t>(8192, a.groups * ceil_div(a.nq, 16 * WIDE)) + ceil_div(a.nq, 16 * WIDE);
        return launch_quads<DP, WIDE, true>(a, vec, l2, waves, s);
    }
    // few queries: long runs of rows per wave (one query, 10^6 x 64 rows, 2 waves per
    // SIMD's worth 68 us, 8 waves 82)
    a.groups_per_wave = qb == 1 ? ceil_div(a.groups, 2048) : quad_groups(a.groups, a.nqb);
    const int64_t waves = ceil_div(a.groups, a.groups_per_wave) * a.nqb;
    return qb == 1 ? launch_quads<DP, 1>(a, vec, l2, waves, s)
                   : launch_quads<DP, WIDE>(a, vec, l2, waves, s);
}

mk_status quads_any(const QuadArgs& a, bool vec, bool l2, hipStream_t s) {
    if (a.d <= 32) return quads<32>(a, vec, l2, s);
    if (a.d <= 64) return quads<64>(a, vec, l2, s);
    if (a.d <= 96) return quads<96>(a, vec, l2, s);
    if (a.d <= 128) return quads<128>(a, vec, l2, s);
    return quads<256>(a, vec, l2, s);
}

// Selection and finish by a workgroup per query.
mk_status finish_any(const QuadArgs& a, int64_t nq, const uint64_t* lists, int32_t nseg, int32_t kq,
                     bool l2, bool vec, int32_t k, float* D, int64_t* I, hipStream_t s) {
    auto of = [&](auto with_list) {
        constexpr bool R = decltype(with_list)::value;
        return kq <= 64    ? quad_finish_kernel<1280, 1, 256, R>
               : kq <= 512 ? quad_finish_kernel<2560, 2, 2048, R>
                           : quad_finish_kernel<4096, 2, 4096, R>;
    };
    auto kern = a.rest.list ? of(std::true_type{}) : of(std::false_type{});
    hipLaunchKernelGGL(kern, dim3((unsigned)nq), dim3(kPoolThreads), 0, s, a.out, a.ld, lists, nseg,
                       kq, a.xq, a.xb, l2 ? a.yn : nullptr, a.nb, a.d, (int32_t)vec, (int32_t)l2, k,
                       a.rest, D, I);
    MK_LAUNCHED();
    return MK_OK;
}

int32_t groups_kept(int32_t k) { return std::min(k + kSlack, kMaxK); }

// Segments that a row of ld minima is selected in: a workgroup takes a segment of
// it and leaves kq keys to the finish, so their number is best where a segment is
// about as long as the keys of all segments; with enough queries to fill the chip
// the finish takes whole rows.
int64_t segments(int64_t ld, int32_t kq, int64_t nq) {
    const int64_t even = (int64_t)std::sqrt((double)ld / kq);
    const int64_t n = std::min({even, ld / 2048, ceil_div(1024, nq)});
    return n < 4 ? 1 : n;
}

}  // namespace

int64_t dense_query_bytes(int64_t nb, int32_t k) {
    const int64_t ld = ceil_div(nb, 64) * 16;
    const int32_t kq = groups_kept(k);
    const int64_t n = segments(ld, kq, 1);
    return 4 * ld + (n > 1 ? 8 * n * kq : 0);
}

mk_status dense_search(const float* xq, int64_t nq, const float* xb, const float* yn, int64_t nb,
                       int32_t d, int32_t k, bool l2, bool vec, float* D, int64_t* I,
                       void* scratch, hipStream_t s) {
    const int32_t kq = groups_kept(k);
    const int64_t ld = ceil_div(nb, 64) * 16;
    Scratch mem;
    if (!scratch) {
        MK_TRY(mem.alloc((size_t)(nq * dense_query_bytes(nb, k) + 256), s));
        scratch = mem.ptr;
    }
    float* least = static_cast<float*>(scratch);
    QuadArgs a{xq, xb, yn, nq, nb, d, ceil_div(nb, 64), 1, 1, least, ld, RestSpan{}};
    MK_TRY(quads_any(a, vec, l2, s));
    uint64_t* lists = nullptr;
    int64_t nseg = segments(ld, kq, nq);
    if (nseg > 1) {
        const int64_t seg_len = ceil_div(ceil_div(ld, nseg), 256) * 256;
        nseg = ceil_div(ld, seg_len);
        lists = reinterpret_cast<uint64_t*>(
            (reinterpret_cast<uintptr_t>(least + nq * ld) + 255) & ~(uintptr_t)255);
        MK_TRY(kselect_segments(least, nq, ld, kq, seg_len, lists, s));
    }
    ProfScope prof("dense_finish", s);
    // (a wave takes 64 minima in the time that a workgroup takes 1,024: 1,024 queries,
    // 8,192 minima 55 us more, 10^4 queries, 1,024 minima 57 us less)
    if (kq <= 64 && nseg == 1 && nq >= 1024 && 2 * nq >= ld) {
        hipLaunchKernelGGL(quad_finish_wave, dim3((unsigned)ceil_div(nq, kMergeWaves)),
                           dim3(64 * kMergeWaves), 0, s, least, ld, nq, kq, xq, xb,
                           l2 ? yn : nullptr, nb, d, (int32_t)vec, (int32_t)l2, k, D, I);
        MK_LAUNCHED();
        return MK_OK;
    }
    return finish_any(a, nq, lists, (int32_t)nseg, kq, l2, vec, k, D, I, s);
}

// The fused search has one workgroup for 64 queries and a sixteenth of the rows, and
// needs as long for one query as for a batch that fills the chip: 34 of 1,000 queries
// left, 10^6 x 128 rows: 3.4 ms of the call, here 0.5.
mk_status dense_rest(const float* xq, int64_t nq, const float* xb, const float* yn, int64_t nb,
                     int32_t d, int32_t k, bool l2, bool vec, float* D, int64_t* I, RestQueries* rest,
                     hipStream_t s) {
    rest->done = 0;
    const int64_t most = dense_rest_most(nq, nb);
    if (most == 0 || !dense_pays(nq, nb, k)) return MK_OK;
    const int64_t rounds = ceil_div(nq, most), ld = ceil_div(nb, 64) * 16;
    Scratch mem;
    const mk_status st = mem.alloc(dense_rest_bytes(nq, nb, k), s);
    if (st == MK_ERR_OOM) {
        (void)hipGetLastError();
        return MK_OK;
    }
    MK_TRY(st);
    const bool all = rounds <= 2;
    for (int64_t r = 0; r < (all ? rounds : 1); ++r) {
        QuadArgs a{xq, xb, yn, most, nb, d, ceil_div(nb, 64), 1, 1, mem.as<float>(), ld,
                   RestSpan{rest->list, rest->count, r * most, most, all ? nq : most}};
        MK_TRY(quads_any(a, vec, l2, s));
        ProfScope prof("dense_finish", s);
        MK_TRY(finish_any(a, most, nullptr, 1, groups_kept(k), l2, vec, k, D, I, s));
    }
    rest->done = all ? nq : most;
    return MK_OK;
}

}  // namespace mk
