// Exact search where either side is small: few queries over any database, or
// any number over a few thousand rows (the coarse search of an IVF index).
//
//   1. quad_min_kernel: FP32 products (v_mfma_f32_16x16x4f32, the fused kernel's
//      products in its order) of every query with every row, straight from
//      memory to the matrix operands; of every four rows the least score is
//      stored.  One read of the database, nq * nb bytes written.
//   2. k-selection of the k + 16 best groups of four.  A row of the k best has
//      at most k - 1 groups before its own, so these groups hold every candidate
//      that the fused search would keep.
//   3. quad_finish_kernel: direct-form FP32 distances of the groups' rows, the k
//      best written.
//
// Bound by memory for few queries: one query over 10^6 x 128 rows, k = 10: 154 us
// (the rows' read 96 us, 5.3 TB/s) against 2,422 us by the fused search, which has
// 16 workgroups for it (one per chunk).  By the FP32 matrix products for many:
// 10^4 queries over 4,096 x 128 centroids, k = 8: 270 us against 450 us.
#include <algorithm>

#include "dense.hpp"
#include "fused.hpp"
#include "kselect.hpp"

namespace mk {

namespace {

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
};

// A wave takes 16 QB queries (B operands, in registers) and streams its rows 64
// at a time: block b of four, A row m is row 16 (m / 4) + 4 b + m % 4 of them, so
// that lane (query li, quarter lh) ends up with groups 4 lh .. 4 lh + 3 of four
// consecutive rows: one 16-byte store.  The next block's rows are loaded while
// this block's products run; enough waves per CU keep the memory busy.
template <int DP, int QB, bool VEC, bool L2>
__global__ __launch_bounds__(256) void quad_min_kernel(QuadArgs a) {
    constexpr int S4 = DP / 16;  // granule steps of four floats per lane
    const int lane = lane_id(), li = lane & 15, lh = lane >> 4;
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
        const float* row = a.xq + (ok ? i : 0) * a.d;
#pragma unroll
        for (int s = 0; s < S4; ++s) q[qb][s] = load_granule<OpF32, VEC>(row, 4 * s + lh, a.d, ok);
    }
    auto load = [&](int64_t g, int b, uint4 (&y)[S4]) __attribute__((always_inline)) {
        int64_t r = g * 64 + 16 * (li >> 2) + 4 * b + (li & 3);
        r = r < a.nb ? r : a.nb - 1;
        const float* row = a.xb + r * a.d;
#pragma unroll
        for (int s = 0; s < S4; ++s) y[s] = load_granule<OpF32, VEC>(row, 4 * s + lh, a.d, true);
    };
    uint4 y[S4], next[S4];
    load(g0, 0, next);
#pragma unroll 1
    for (int64_t g = g0; g < g1; ++g) {
        float least[QB][4];
#pragma unroll
        for (int b = 0; b < 4; ++b) {
#pragma unroll
            for (int s = 0; s < S4; ++s) y[s] = next[s];
            if (b < 3)
                load(g, b + 1, next);
            else if (g + 1 < g1)
                load(g + 1, 0, next);
            const int64_t r = g * 64 + 16 * lh + 4 * b;  // first of this lane's four rows
            float yn[4] = {0.f, 0.f, 0.f, 0.f};
            if constexpr (L2) {
                if (a.yn) {
#pragma unroll
                    for (int i = 0; i < 4; ++i) yn[i] = a.yn[r + i < a.nb ? r + i : a.nb - 1];
                } else {
                    float s2 = 0.f;
#pragma unroll
                    for (int s = 0; s < S4; ++s) {
                        const float e0 = __uint_as_float(y[s].x), e1 = __uint_as_float(y[s].y);
                        const float e2 = __uint_as_float(y[s].z), e3 = __uint_as_float(y[s].w);
                        s2 = fmaf(e0, e0, s2);
                        s2 = fmaf(e1, e1, s2);
                        s2 = fmaf(e2, e2, s2);
                        s2 = fmaf(e3, e3, s2);
                    }
                    s2 += __shfl_xor(s2, 16);
                    s2 += __shfl_xor(s2, 32);
#pragma unroll
                    for (int i = 0; i < 4; ++i) yn[i] = __shfl(s2, 4 * lh + i);
                }
            }
            floatx4 acc[QB];
#pragma unroll
            for (int qb = 0; qb < QB; ++qb) acc[qb] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int s = 0; s < S4; ++s)
#pragma unroll
                for (int qb = 0; qb < QB; ++qb) acc[qb] = OpF32::mma(acc[qb], y[s], q[qb][s]);
#pragma unroll
            for (int qb = 0; qb < QB; ++qb) {
                float m = INFINITY;
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const float sc = L2 ? fmaf(-2.f, acc[qb][i], yn[i]) : -acc[qb][i];
                    m = fminf(m, r + i < a.nb ? sc : INFINITY);
                }
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

// A workgroup per query: exact distances of the rows of its kq groups (16 rows
// per wave and step, as in the fused search's re-rank), then wave 0 selects the
// k best by (distance, row).
template <int KR>
__global__ __launch_bounds__(64 * kMergeWaves) void quad_finish_kernel(
    const int64_t* __restrict__ groups, int32_t kq, const float* __restrict__ xq,
    const float* __restrict__ xb, const float* __restrict__ yn, int64_t nb, int32_t d, int32_t vec,
    int32_t l2, int32_t k, float* __restrict__ D, int64_t* __restrict__ I) {
    constexpr int T = SelParams<KR>::T;
    extern __shared__ __align__(16) unsigned char smem[];
    float* xs = reinterpret_cast<float*>(smem);
    uint64_t* kl = reinterpret_cast<uint64_t*>(smem + sizeof(float) * kMaxDim);
    float* dist = reinterpret_cast<float*>(kl + 4 * kq);
    const int wave = threadIdx.x >> 6, lane = lane_id();
    const int64_t q = blockIdx.x;
    const int n = 4 * kq;
    for (int e = threadIdx.x; e < n; e += 64 * kMergeWaves) {
        const int64_t g = groups[q * kq + (e >> 2)];
        const int64_t row = 4 * g + (e & 3);
        // (a row without a finite norm has no score: it was no candidate)
        kl[e] = g >= 0 && row < nb && (!yn || yn[row] < INFINITY) ? (uint64_t)row : kSentinel;
    }
    for (int t = threadIdx.x; t < d; t += 64 * kMergeWaves) xs[t] = xq[q * d + t];
    __syncthreads();
#pragma unroll 1
    for (int e0 = 16 * wave; e0 < n; e0 += 16 * kMergeWaves)
        rerank_rows16(xs, kl, e0, n, xb, d, vec, l2, dist);
    __syncthreads();
    if (wave != 0) return;
    WaveSelect<KR, T> ws;
    ws.init(k);
#pragma unroll 1
    for (int e0 = 0; e0 < n; e0 += 64) {
        const int e = e0 + lane;
        uint64_t key = kSentinel;
        // (a NaN is no distance)
        if (e < n && kl[e] != kSentinel && dist[e] == dist[e])
            key = make_key(l2 ? dist[e] : -dist[e], (uint32_t)kl[e]);
        if (ws.push(key)) ws.merge();
    }
    ws.finish();
    emit_reranked<KR>(ws.w, k, l2, D + q * k, I + q * k);
}

template <int DP, int QB>
mk_status launch_quads(const QuadArgs& a, bool vec, bool l2, int64_t waves, hipStream_t s) {
    ProfScope prof("dense_quads", s);
    auto kern = vec ? (l2 ? quad_min_kernel<DP, QB, true, true> : quad_min_kernel<DP, QB, true, false>)
                    : (l2 ? quad_min_kernel<DP, QB, false, true> : quad_min_kernel<DP, QB, false, false>);
    hipLaunchKernelGGL(kern, dim3((unsigned)ceil_div(waves, 4)), dim3(256), 0, s, a);
    MK_LAUNCHED();
    return MK_OK;
}

template <int DP>
mk_status quads(QuadArgs a, bool vec, bool l2, hipStream_t s) {
    // query blocks of 64 (32 for wide rows), or 16 when that is all there is
    constexpr int WIDE = DP > 128 ? 2 : 4;
    const int qb = a.nq <= 16 ? 1 : WIDE;
    a.nqb = (int32_t)ceil_div(a.nq, 16 * qb);
    // about 8 waves per SIMD's worth, of at least one group each
    a.groups_per_wave = std::max<int64_t>(1, a.groups * a.nqb / 8192);
    const int64_t waves = ceil_div(a.groups, a.groups_per_wave) * a.nqb;
    return qb == 1 ? launch_quads<DP, 1>(a, vec, l2, waves, s)
                   : launch_quads<DP, WIDE>(a, vec, l2, waves, s);
}

template <int KR>
mk_status finish(const int64_t* groups, int32_t kq, const float* xq, int64_t nq, const float* xb,
                 const float* yn, int64_t nb, int32_t d, bool vec, bool l2, int32_t k, float* D,
                 int64_t* I, hipStream_t s) {
    ProfScope prof("dense_finish", s);
    const size_t lds = sizeof(float) * kMaxDim + 12 * 4 * (size_t)kq;
    hipLaunchKernelGGL((quad_finish_kernel<KR>), dim3((unsigned)nq), dim3(64 * kMergeWaves), lds, s,
                       groups, kq, xq, xb, l2 ? yn : nullptr, nb, d, (int32_t)vec, (int32_t)l2, k, D, I);
    MK_LAUNCHED();
    return MK_OK;
}

int32_t groups_kept(int32_t k) { return std::min(k + kSlack, kMaxK); }

}  // namespace

int64_t dense_query_bytes(int64_t nb, int32_t k) {
    return ceil_div(nb, 64) * 64 + 12 * (int64_t)groups_kept(k);
}

mk_status dense_search(const float* xq, int64_t nq, const float* xb, const float* yn, int64_t nb,
                       int32_t d, int32_t k, bool l2, bool vec, float* D, int64_t* I,
                       void* scratch, hipStream_t s) {
    const int32_t kq = groups_kept(k);
    const int64_t ld = ceil_div(nb, 64) * 16;
    Scratch mem;
    const size_t b_out = ((size_t)(nq * ld) * sizeof(float) + 255) & ~(size_t)255;
    const size_t b_val = ((size_t)nq * kq * sizeof(float) + 255) & ~(size_t)255;
    if (!scratch) {
        MK_TRY(mem.alloc(b_out + b_val + (size_t)nq * kq * sizeof(int64_t), s));
        scratch = mem.ptr;
    }
    unsigned char* base = static_cast<unsigned char*>(scratch);
    float* vals = reinterpret_cast<float*>(base + b_out);
    int64_t* groups = reinterpret_cast<int64_t*>(base + b_out + b_val);
    QuadArgs a{xq, xb, yn, nq, nb, d, ceil_div(nb, 64), 1, 1, reinterpret_cast<float*>(base), ld};
    if (d <= 32) MK_TRY(quads<32>(a, vec, l2, s));
    else if (d <= 64) MK_TRY(quads<64>(a, vec, l2, s));
    else if (d <= 96) MK_TRY(quads<96>(a, vec, l2, s));
    else if (d <= 128) MK_TRY(quads<128>(a, vec, l2, s));
    else MK_TRY(quads<256>(a, vec, l2, s));
    MK_TRY(mk_kselect(a.out, nq, ld, kq, 0, vals, groups, s));
    switch (queue_regs(k)) {
        case 1: return finish<1>(groups, kq, xq, nq, xb, yn, nb, d, vec, l2, k, D, I, s);
        case 2: return finish<2>(groups, kq, xq, nq, xb, yn, nb, d, vec, l2, k, D, I, s);
        case 4: return finish<4>(groups, kq, xq, nq, xb, yn, nb, d, vec, l2, k, D, I, s);
        case 8: return finish<8>(groups, kq, xq, nq, xb, yn, nb, d, vec, l2, k, D, I, s);
        default: return finish<16>(groups, kq, xq, nq, xb, yn, nb, d, vec, l2, k, D, I, s);
    }
}

}  // namespace mk
