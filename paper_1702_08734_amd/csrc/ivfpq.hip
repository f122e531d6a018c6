// IVFADC index (Section 2 Eq. 3-6, Section 5.2-5.3): k-means training of the
// coarse quantizer and of the product quantizer, encoding and list building,
// and the search: coarse exact search (Eq. 5), query tables of term 3, the
// list scan with per-(query, list) lookup tables in LDS feeding WaveSelect,
// and the merge of the per-list partial results (Eq. 6).
#include <hip/hip_fp16.h>

#include <algorithm>
#include <cstring>
#include <type_traits>
#include <vector>

#include "common.hpp"
#include "fileio.hpp"
#include "kselect.hpp"
#include "sieve.hpp"
#include "mlp.hpp"
#include "pool.hpp"
#include "profile.hpp"
#include "wave_select.hpp"

struct mk_ivfpq {
    int32_t d = 0, nlist = 0, M = 0, dsub = 0;
    bool trained = false;
    float* coarse = nullptr;        // [nlist, d]
    float* coarse_norms = nullptr;  // [nlist]
    float* books = nullptr;         // [M, 256, dsub]
    float* term1 = nullptr;         // [nlist, M, 256]
    int64_t ntotal = 0;
    int64_t capacity = 0;
    uint8_t* codes = nullptr;       // [capacity, M], grouped by list
    int64_t* ids = nullptr;         // [capacity]
    float* t1e = nullptr;           // [capacity] term 1 of Eq. 11 per entry
    int64_t* offsets_dev = nullptr; // [nlist + 1]
    std::vector<int64_t> offsets;   // host copy
    // scan options: 16-bit lookup tables; probed lists per scan workgroup
    // (0: chosen from the launch size, -1: all of a query's lists)
    bool lut16 = false;
    int32_t lists_per_group = 0;
};

namespace mk {

namespace {

constexpr int kBlock = 256;
// Element-wise kernels walk their items with a grid-stride loop; grids are
// capped at kMaxBlocks so that no launch exceeds the 32-bit work-item count
// of a grid dimension (a 50,000,000 x 128 array has 6.4e9 elements).
constexpr int64_t kMaxBlocks = 1 << 20;
#define kStride ((int64_t)gridDim.x * kBlock)

unsigned grid_of(int64_t n) {
    const int64_t b = ceil_div(n > 0 ? n : 1, kBlock);
    return (unsigned)(b < kMaxBlocks ? b : kMaxBlocks);
}

void free_dev(void*& p) {
    if (p) (void)hipFree(p);
    p = nullptr;
}

template <class T>
mk_status alloc_dev(T*& p, size_t count) {
    void* v = nullptr;
    MK_HIP(hipMalloc(&v, sizeof(T) * (count ? count : 1)));
    p = static_cast<T*>(v);
    return MK_OK;
}

// ---------------------------------------------------------------- k-means
__global__ void gather_rows_kernel(const float* __restrict__ src, int32_t d,
                                   const int64_t* __restrict__ rows, int64_t n,
                                   float* __restrict__ dst) {
    for (int64_t g = (int64_t)blockIdx.x * kBlock + threadIdx.x; g < n * d; g += kStride) {
        const int64_t i = g / d, t = g % d;
        dst[g] = src[rows[i] * d + t];
    }
}

// Sum points into their centroid's FP64 accumulator (one thread per
// coordinate, so neighbouring lanes add to neighbouring addresses).
__global__ void km_accumulate(const float* __restrict__ x, int64_t n, int32_t d,
                              const int64_t* __restrict__ assign, int32_t K,
                              double* __restrict__ sums, unsigned long long* __restrict__ counts) {
    for (int64_t g = (int64_t)blockIdx.x * kBlock + threadIdx.x; g < n * d; g += kStride) {
        const int64_t i = g / d, t = g % d;
        const int64_t a = assign[i];
        if (a < 0 || a >= K) continue;  // invalid assignments are ignored
        if (t == 0) atomicAdd(&counts[a], 1ull);
        atomicAdd(&sums[a * d + t], (double)x[g]);
    }
}

__global__ void km_finalize(const double* __restrict__ sums,
                            const unsigned long long* __restrict__ counts, int32_t K, int32_t d,
                            float* __restrict__ c, int64_t* __restrict__ counts_out) {
    for (int64_t g = (int64_t)blockIdx.x * kBlock + threadIdx.x; g < (int64_t)K * d;
         g += kStride) {
        const int64_t j = g / d, t = g % d;
        const unsigned long long n = counts[j];
        if (n > 0) c[g] = (float)(sums[g] / (double)n);
        if (t == 0) counts_out[j] = (int64_t)n;
    }
}

__global__ void fill_u32_kernel(unsigned int* __restrict__ a, int64_t n);

// Sums by cluster without an atomic per coordinate: the points' indices are put
// in cluster order (a count and a cursor per cluster), and a workgroup adds up
// each stretch of at most kSegRows points of one cluster, 16-byte loads, FP64
// sums in registers, one FP64 atomic per coordinate and stretch.  500,000 x 128
// points, 4,096 clusters: 156 us in all; 64 million FP64 atomics took 437 us.
constexpr int kSegRows = 256;

// One to at[a] for every lane with 0 <= a < K, and the lane's place among them: of the
// clusters of four lanes, those that eight lanes share or more are added once for all of
// these (500,000 points in the order of 16 clusters: 11.4 ms with an atomic each, 0.24), the
// others' by themselves.  Whole waves.
__device__ __forceinline__ uint32_t wave_counts(int32_t a, int32_t K, uint32_t* __restrict__ at) {
    const bool live = a >= 0 && a < K;
    const int lane = lane_id();
    uint64_t todo = __ballot(live), single = 0;
    uint32_t place = 0;
#pragma unroll 1
    for (int r = 0; r < 4 && todo; ++r) {
        const int src = __builtin_ctzll(todo);
        const int32_t v = __builtin_amdgcn_readlane(a, src);
        const uint64_t same = __ballot(live && a == v);
        todo &= ~same;
        if (__popcll(same) < 8) {
            single |= same;
            continue;
        }
        uint32_t base = 0;
        if (lane == src) base = atomicAdd(&at[v], (uint32_t)__popcll(same));
        base = (uint32_t)__builtin_amdgcn_readlane((int)base, src);
        if (live && a == v)
            place = base + __builtin_amdgcn_mbcnt_hi((uint32_t)(same >> 32),
                                                     __builtin_amdgcn_mbcnt_lo((uint32_t)same, 0u));
    }
    if ((todo | single) >> lane & 1) place = atomicAdd(&at[a], 1u);
    return place;
}

__global__ void km_count(const int64_t* __restrict__ assign, int64_t n, int32_t K,
                         uint32_t* __restrict__ counts) {
    for (int64_t i0 = (int64_t)blockIdx.x * kBlock; i0 < n; i0 += kStride) {
        const int64_t a = i0 + threadIdx.x < n ? assign[i0 + threadIdx.x] : -1;
        (void)wave_counts(a >= 0 && a < K ? (int32_t)a : -1, K, counts);  // others are ignored
    }
}

// Few clusters: a workgroup counts kCountPoints points in LDS and adds up once per
// cluster.  One word per cluster takes the atomics of n / K points one by one: 500,000
// points of 32 components in 256 clusters 506 us with wave_counts alone, 97.  From a
// quarter of kCountPoints clusters on there are about as many additions as points.
constexpr int kCountPoints = 4096, kCountClusters = kCountPoints / 4;
struct FewCounts {
    uint32_t bins[kCountClusters];
    // the clusters of this thread's points of the chunk at i0 (-1: none) and, in bins,
    // the chunk's counts; the points' places in them
    __device__ __forceinline__ void take(const int64_t* __restrict__ assign, int64_t i0, int64_t n,
                                         int32_t K, int32_t (&a)[kCountPoints / kBlock],
                                         uint32_t (&place)[kCountPoints / kBlock]) {
        __syncthreads();
        for (int j = threadIdx.x; j < K; j += kBlock) bins[j] = 0u;
        __syncthreads();
#pragma unroll
        for (int e = 0; e < kCountPoints / kBlock; ++e) {
            const int64_t i = i0 + e * kBlock + threadIdx.x;
            const int64_t v = i < n ? assign[i] : -1;
            a[e] = v >= 0 && v < K ? (int32_t)v : -1;  // others are ignored
        }
#pragma unroll
        for (int e = 0; e < kCountPoints / kBlock; ++e)
            place[e] = a[e] >= 0 ? atomicAdd(&bins[a[e]], 1u) : 0u;
        __syncthreads();
    }
};

__global__ __launch_bounds__(kBlock) void km_count_few(const int64_t* __restrict__ assign, int64_t n,
                                                       int32_t K, uint32_t* __restrict__ counts) {
    __shared__ FewCounts few;
    int32_t a[kCountPoints / kBlock];
    uint32_t place[kCountPoints / kBlock];
    for (int64_t i0 = (int64_t)blockIdx.x * kCountPoints; i0 < n; i0 += (int64_t)gridDim.x * kCountPoints) {
        few.take(assign, i0, n, K, a, place);
        for (int j = threadIdx.x; j < K; j += kBlock)
            if (few.bins[j]) atomicAdd(&counts[j], few.bins[j]);
    }
}

// Exclusive prefix of the counts (first[K]: their sum) and of the stretches, the
// cursors, and the counts as 64-bit words.  One workgroup.
__global__ __launch_bounds__(1024) void km_prefix(const uint32_t* __restrict__ counts, int32_t K,
                                                  uint32_t* __restrict__ first,
                                                  uint32_t* __restrict__ cursor,
                                                  uint32_t* __restrict__ seg,
                                                  unsigned long long* __restrict__ counts64) {
    __shared__ uint32_t w1[16], w2[16], c1, c2;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    if (threadIdx.x == 0) c1 = c2 = 0u;
    __syncthreads();
    for (int32_t base = 0; base < K; base += 1024) {
        const int32_t j = base + threadIdx.x;
        const uint32_t n = j < K ? counts[j] : 0u;
        const uint32_t s = (n + kSegRows - 1) / kSegRows;
        const uint32_t i1 = (uint32_t)wave_inclusive_sum((int)n);
        const uint32_t i2 = (uint32_t)wave_inclusive_sum((int)s);
        if (lane == 63) {
            w1[wave] = i1;
            w2[wave] = i2;
        }
        __syncthreads();
        uint32_t b1 = c1, b2 = c2;
        for (int w = 0; w < wave; ++w) {
            b1 += w1[w];
            b2 += w2[w];
        }
        if (j < K) {
            first[j] = cursor[j] = b1 + i1 - n;
            seg[j] = b2 + i2 - s;
            counts64[j] = n;
        }
        __syncthreads();
        if (threadIdx.x == 1023) {
            c1 = b1 + i1;
            c2 = b2 + i2;
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        first[K] = c1;
        seg[K] = c2;
    }
}

// Points in cluster order, and the cluster of each stretch.
__global__ void km_order(const int64_t* __restrict__ assign, int64_t n, int32_t K,
                         uint32_t* __restrict__ cursor, uint32_t* __restrict__ order,
                         const uint32_t* __restrict__ seg, uint32_t* __restrict__ seg_cluster) {
    for (int64_t i0 = (int64_t)blockIdx.x * kBlock; i0 < n; i0 += kStride) {
        const int64_t i = i0 + threadIdx.x;
        const int64_t a = i < n ? assign[i] : -1;
        const bool live = a >= 0 && a < K;
        const uint32_t place = wave_counts(live ? (int32_t)a : -1, K, cursor);
        if (live) order[place] = (uint32_t)i;
    }
    for (int64_t j = (int64_t)blockIdx.x * kBlock + threadIdx.x; j < K; j += kStride)
        for (uint32_t t = seg[j]; t < seg[j + 1]; ++t) seg_cluster[t] = (uint32_t)j;
}

__global__ __launch_bounds__(kBlock) void km_order_few(
    const int64_t* __restrict__ assign, int64_t n, int32_t K, uint32_t* __restrict__ cursor,
    uint32_t* __restrict__ order, const uint32_t* __restrict__ seg, uint32_t* __restrict__ seg_cluster) {
    __shared__ FewCounts few;
    int32_t a[kCountPoints / kBlock];
    uint32_t place[kCountPoints / kBlock];
    for (int64_t i0 = (int64_t)blockIdx.x * kCountPoints; i0 < n; i0 += (int64_t)gridDim.x * kCountPoints) {
        few.take(assign, i0, n, K, a, place);
        for (int j = threadIdx.x; j < K; j += kBlock)
            if (few.bins[j]) few.bins[j] = atomicAdd(&cursor[j], few.bins[j]);
        __syncthreads();
#pragma unroll
        for (int e = 0; e < kCountPoints / kBlock; ++e)
            if (a[e] >= 0)
                order[few.bins[a[e]] + place[e]] = (uint32_t)(i0 + e * kBlock + threadIdx.x);
    }
    for (int64_t j = (int64_t)blockIdx.x * kBlock + threadIdx.x; j < K; j += kStride)
        for (uint32_t t = seg[j]; t < seg[j + 1]; ++t) seg_cluster[t] = (uint32_t)j;
}

// d % 4 == 0, d <= 4 kBlock, 16-byte aligned rows.  Workgroups walk the stretches
// (nlist may be 2^24 and more: a workgroup each would pass what a grid can hold).
__global__ __launch_bounds__(kBlock) void km_segment_sums(
    const float* __restrict__ x, int32_t d, int32_t K, const uint32_t* __restrict__ first,
    const uint32_t* __restrict__ seg, const uint32_t* __restrict__ seg_cluster,
    const uint32_t* __restrict__ order, double* __restrict__ sums) {
    __shared__ double red[kBlock][4];
    const uint32_t segs = seg[K];
    const int gpr = d / 4, rows = kBlock / gpr;  // granules per row, rows at a time
    const int r = threadIdx.x / gpr, c = threadIdx.x % gpr;
#pragma unroll 1
    for (uint32_t t = blockIdx.x; t < segs; t += gridDim.x) {
        const uint32_t j = seg_cluster[t];
        const uint32_t lo = first[j] + (t - seg[j]) * kSegRows;
        const uint32_t hi = lo + kSegRows < first[j + 1] ? lo + kSegRows : first[j + 1];
        double s[4] = {0.0, 0.0, 0.0, 0.0};
        if (r < rows) {
#pragma unroll 4
            for (uint32_t i = lo + r; i < hi; i += rows) {
                const float4 v = *reinterpret_cast<const float4*>(x + (int64_t)order[i] * d + 4 * c);
                s[0] += (double)v.x;
                s[1] += (double)v.y;
                s[2] += (double)v.z;
                s[3] += (double)v.w;
            }
        }
#pragma unroll
        for (int e = 0; e < 4; ++e) red[threadIdx.x][e] = s[e];
        __syncthreads();
        for (int g = threadIdx.x; g < d; g += kBlock) {
            double v = 0.0;
            for (int q = 0; q < rows; ++q) v += red[q * gpr + g / 4][g % 4];
            atomicAdd(&sums[(int64_t)j * d + g], v);
        }
        __syncthreads();
    }
}

// Empty clusters, in increasing index order, split the currently largest
// cluster (ties to the lower index): multiplicative offsets 1 +- 2^-10 with
// alternating sign per coordinate, products in FP64 rounded to FP32, and the
// empty cluster takes floor(count / 2).  One workgroup; each round finds the next
// empty cluster and the largest one together (a single thread's walk over 4,096
// counts took 420 us).
__global__ __launch_bounds__(kBlock) void km_split_empty(float* __restrict__ c,
                                                         int64_t* __restrict__ counts, int32_t K,
                                                         int32_t d) {
    __shared__ int64_t s_cnt[kBlock];
    __shared__ int32_t s_idx[kBlock], s_zero[kBlock];
    const int tid = threadIdx.x;
    int32_t next = 0;  // first cluster not yet looked at
    for (;;) {
        int64_t best = -1;
        int32_t bi = 0, zero = K;
        for (int32_t q = tid; q < K; q += kBlock) {
            const int64_t v = counts[q];
            if (v > best) {
                best = v;
                bi = q;
            }
            if (v == 0 && q >= next && q < zero) zero = q;
        }
        s_cnt[tid] = best;
        s_idx[tid] = bi;
        s_zero[tid] = zero;
        __syncthreads();
        for (int w = kBlock / 2; w > 0; w >>= 1) {
            if (tid < w) {
                const int64_t o = s_cnt[tid + w];
                const int32_t oi = s_idx[tid + w];
                if (o > s_cnt[tid] || (o == s_cnt[tid] && oi < s_idx[tid])) {
                    s_cnt[tid] = o;
                    s_idx[tid] = oi;
                }
                s_zero[tid] = min(s_zero[tid], s_zero[tid + w]);
            }
            __syncthreads();
        }
        const int32_t b = s_idx[0], j = s_zero[0];
        __syncthreads();  // read before the next round writes
        if (j >= K) break;
        const double eps = 1.0 / 1024.0;
        for (int32_t t = tid; t < d; t += kBlock) {
            const double s = (t % 2 == 0) ? 1.0 : -1.0;
            const double v = (double)c[(int64_t)b * d + t];
            c[(int64_t)j * d + t] = (float)(v * (1.0 + s * eps));
            c[(int64_t)b * d + t] = (float)(v * (1.0 - s * eps));
        }
        if (tid == 0) {
            const int64_t half = counts[b] / 2;
            counts[j] = half;
            counts[b] -= half;
        }
        __syncthreads();
        next = j + 1;
    }
}

mk_status kmeans_update(const float* x, int64_t n, int32_t d, const int64_t* assign, int32_t K,
                        float* c, int64_t* counts_out, hipStream_t s) {
    Scratch sums, cnt, cnt64;
    MK_TRY(sums.alloc(sizeof(double) * (size_t)K * d, s));
    MK_TRY(cnt.alloc(sizeof(unsigned long long) * (size_t)K, s));
    int64_t* counts = counts_out;
    if (!counts) {
        MK_TRY(cnt64.alloc(sizeof(int64_t) * (size_t)K, s));
        counts = cnt64.as<int64_t>();
    }
    MK_HIP(hipMemsetAsync(sums.ptr, 0, sizeof(double) * (size_t)K * d, s));
    MK_HIP(hipMemsetAsync(cnt.ptr, 0, sizeof(unsigned long long) * (size_t)K, s));
    // By cluster, except for few points in clusters enough that the atomics of the plain
    // sums do not wait for each other: there the launches set the time.  Plain / by
    // cluster, us: 4,096 x 128 points in 64 clusters 56 / 81; in 4, 8,192 x 64 141 / 100; in
    // 64, 16,384 74 / 97, 32,768 124 / 99; in 256, 32,768 59 / 97, 65,536 93 / 97; 100,000 x
    // 32 in 1,000, all alike 60 / 97, half of them in one 1,363 / 167.  Rows of less than
    // 32 components are cheaper to add where they belong than to gather (500,000 x 8: 330
    // us in 256 clusters, 73 in 4,096).
    bool by_cluster = d >= 32 && d % 4 == 0 && d <= 4 * kBlock && n >= 4096 && n < (1ll << 31) &&
                      (n > 32768 || n * n >= 16000000ll * K) &&
                      reinterpret_cast<uintptr_t>(x) % 16 == 0;
    const int64_t segs = ceil_div(n, kSegRows) + K;
    Scratch words;
    if (by_cluster) {
        // (without room for the points' order the plain sums, which need none)
        const mk_status st = words.alloc(sizeof(uint32_t) * (size_t)(4 * (int64_t)K + 2 + n + segs), s);
        if (st != MK_OK && st != MK_ERR_OOM) return st;
        if (st == MK_ERR_OOM) (void)hipGetLastError();
        by_cluster = st == MK_OK;
    }
    if (by_cluster) {
        uint32_t* count = words.as<uint32_t>();
        uint32_t *cursor = count + K, *first = cursor + K, *seg = first + K + 1;
        uint32_t *order = seg + K + 1, *seg_cluster = order + n;
        hipLaunchKernelGGL(fill_u32_kernel, dim3(grid_of(K)), dim3(kBlock), 0, s, count, (int64_t)K);
        MK_LAUNCHED();
        const bool few = K <= kCountClusters;
        const dim3 chunks((unsigned)std::min<int64_t>(ceil_div(n, kCountPoints), 1 << 16));
        hipLaunchKernelGGL(few ? km_count_few : km_count, few ? chunks : dim3(grid_of(n)),
                           dim3(kBlock), 0, s, assign, n, K, count);
        MK_LAUNCHED();
        hipLaunchKernelGGL(km_prefix, dim3(1), dim3(1024), 0, s, count, K, first, cursor, seg,
                           cnt.as<unsigned long long>());
        MK_LAUNCHED();
        hipLaunchKernelGGL(few ? km_order_few : km_order,
                           few ? chunks : dim3(grid_of(std::max<int64_t>(n, K))), dim3(kBlock), 0, s,
                           assign, n, K, cursor, order, seg, seg_cluster);
        MK_LAUNCHED();
        hipLaunchKernelGGL(km_segment_sums, dim3((unsigned)std::min<int64_t>(segs, 1 << 16)), dim3(kBlock), 0, s, x, d, K, first,
                           seg, seg_cluster, order, sums.as<double>());
        MK_LAUNCHED();
    } else if (n > 0) {
        hipLaunchKernelGGL(km_accumulate, dim3(grid_of(n * d)), dim3(kBlock), 0,
                           s, x, n, d, assign, K, sums.as<double>(), cnt.as<unsigned long long>());
        MK_LAUNCHED();
    }
    hipLaunchKernelGGL(km_finalize, dim3(grid_of((int64_t)K * d)), dim3(kBlock),
                       0, s, sums.as<double>(), cnt.as<unsigned long long>(), K, d, c, counts);
    MK_LAUNCHED();
    hipLaunchKernelGGL(km_split_empty, dim3(1), dim3(kBlock), 0, s, c, counts, K, d);
    MK_LAUNCHED();
    return MK_OK;
}

mk_status kmeans_assign(const float* x, int64_t n, int32_t d, const float* c, int32_t K,
                        int64_t* assign, float* dist, hipStream_t s) {
    Scratch dtmp;
    float* D = dist;
    if (!D) {
        MK_TRY(dtmp.alloc(sizeof(float) * (size_t)(n > 0 ? n : 1), s));
        D = dtmp.as<float>();
    }
    return knn_search(x, n, c, nullptr, K, d, 1, MK_METRIC_L2, D, assign, s);
}

// Lloyd iterations on c [K, d], initialised by the caller.
mk_status kmeans_run(const float* x, int64_t n, int32_t d, float* c, int32_t K, int32_t niter,
                     hipStream_t s) {
    Scratch a;
    MK_TRY(a.alloc(sizeof(int64_t) * (size_t)n, s));
    for (int32_t it = 0; it < niter; ++it) {
        MK_TRY(kmeans_assign(x, n, d, c, K, a.as<int64_t>(), nullptr, s));
        MK_TRY(kmeans_update(x, n, d, a.as<int64_t>(), K, c, nullptr, s));
    }
    return MK_OK;
}

// ---------------------------------------------------------------- PQ encode
template <int DS>
__global__ __launch_bounds__(kBlock) void pq_encode_fixed(const float* __restrict__ r, int64_t n,
                                                          int32_t d, int32_t M,
                                                          const float* __restrict__ books,
                                                          uint8_t* __restrict__ codes) {
    __shared__ float cb[256 * DS];
    const int m = blockIdx.y;
    for (int e = threadIdx.x; e < 256 * DS; e += kBlock) cb[e] = books[(int64_t)m * 256 * DS + e];
    __syncthreads();
    const int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (i >= n) return;
    float rv[DS];
#pragma unroll
    for (int t = 0; t < DS; ++t) rv[t] = r[i * d + (int64_t)m * DS + t];
    float best = INFINITY;
    int arg = 0;
    for (int j = 0; j < 256; ++j) {
        float s = 0.f;
#pragma unroll
        for (int t = 0; t < DS; ++t) {
            const float df = rv[t] - cb[j * DS + t];
            s = fmaf(df, df, s);
        }
        if (s < best) {  // strict: ties keep the lower index
            best = s;
            arg = j;
        }
    }
    codes[i * M + m] = (uint8_t)arg;
}

__global__ __launch_bounds__(kBlock) void pq_encode_any(const float* __restrict__ r, int64_t n,
                                                        int32_t d, int32_t M, int32_t ds,
                                                        const float* __restrict__ books,
                                                        uint8_t* __restrict__ codes) {
    extern __shared__ float cbs[];
    const int m = blockIdx.y;
    for (int e = threadIdx.x; e < 256 * ds; e += kBlock) cbs[e] = books[(int64_t)m * 256 * ds + e];
    __syncthreads();
    const int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (i >= n) return;
    const float* rv = r + i * d + (int64_t)m * ds;
    float best = INFINITY;
    int arg = 0;
    for (int j = 0; j < 256; ++j) {
        float s = 0.f;
        for (int t = 0; t < ds; ++t) {
            const float df = rv[t] - cbs[j * ds + t];
            s = fmaf(df, df, s);
        }
        if (s < best) {
            best = s;
            arg = j;
        }
    }
    codes[i * M + m] = (uint8_t)arg;
}

// Encoding on the matrix cores, for sub-vectors of up to 16 components: FP16
// pairs (h + l, scaled by a power of two) laid side by side along the 32 products
// of one v_mfma_f32_16x16x32_f16,
//   up to 8 components:  code [ h | h | l | 0 ] . row [ h | l | h | h ],
//   up to 16: code [ h h | h h ] . row [ h h | l l ], then code [ l l | - ] .
//   row [ h h | 0 ],
// so a 16 x 16 block of code words and rows costs one or two products.  The code
// words (A, all 256 of one sub-quantizer) stay in registers while a wave walks
// its rows 16 at a time (B: lane = row); each lane keeps the two best groups of
// four code words and a bound of the rest (LowKeys).  The best group is then
// evaluated as the plain kernel does, the second where the bound asks for it, and
// every code word where that proves nothing either, so codes are the plain
// kernel's.  Scores are lowered by kSplitErr (|r|^2 + |c|^2) as by split_err for sieve.hpp
// (in units of 2^-24: 10 for the product, 16 for a norm, 4 for the last sums, of 32), and
// by what the code words' common scale can lose.
// Bound by vector operations (11 per lane and block of 4 x 16 scores, and as many
// again per row for the split and the exact distances): 500,000 x 128, M = 16: 427
// us; the plain kernel's 16 operations per row and code word took 764 us.
constexpr float kSplitErr = 0x1p-19f;
struct PqGroup {
    float score;
    int32_t code;
};

// Lowest three of a stream of 32-bit keys; a key is a distance, its low 6 bits
// replaced by the number of its group of four code words (rounding it towards
// zero), compared as an integer.
struct LowKeys {
    int32_t k1, k2, k3;
    __device__ __forceinline__ void init() { k1 = k2 = k3 = 0x7F800000; }
    __device__ __forceinline__ void offer(int32_t k) {
        k3 = med3(k, k2, k3);
        k2 = med3(k, k1, k2);
        k1 = min(k, k1);
    }
    // k1 <= k2 <= k3
    static __device__ __forceinline__ int32_t med3(int32_t a, int32_t b, int32_t c) {
        int32_t r;
        asm("v_med3_i32 %0, %1, %2, %3" : "=v"(r) : "v"(a), "v"(b), "v"(c));
        return r;
    }
};

template <int DS, bool VEC>
__global__ __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(DS > 8 ? 2 : 3))) void pq_encode_mfma(const float* __restrict__ r, int64_t n,
                                                         int32_t d, int32_t M, int32_t ds,
                                                         const float* __restrict__ books,
                                                         uint8_t* __restrict__ codes) {
    constexpr int C = DS > 8 ? 2 : 1;   // products per block
    constexpr int NB = DS > 8 ? 1 : 2;  // blocks of 16 rows in flight
    __shared__ __align__(16) float cb[256 * DS];  // the code words, zero padded
    __shared__ __align__(16) float cn[256];       // |c|^2 (1 - kSplitErr)
    const int m = blockIdx.x % M;
    const int64_t wg = blockIdx.x / M, nwg = gridDim.x / M;
    const int lane = lane_id(), li = lane & 15, lh = lane >> 4, wave = threadIdx.x >> 6;
    for (int e = threadIdx.x; e < 256 * DS; e += kBlock) {
        const int j = e / DS, t = e % DS;
        cb[e] = t < ds ? books[((int64_t)m * 256 + j) * ds + t] : 0.f;
    }
    __syncthreads();
    // largest component and norm, each wave for itself (256 words, 4 per lane)
    float big = 0.f;
    bool fine = true;
#pragma unroll
    for (int w = 0; w < 4; ++w) {
        const int j = w * 64 + lane;
        float ss = 0.f;
        for (int t = 0; t < DS; ++t) {
            const float v = cb[j * DS + t];
            big = fmaxf(big, fabsf(v));
            ss = fmaf(v, v, ss);
        }
        fine = fine && ss < 0x1p100f;  // (false for a NaN)
        if (wave == 0) cn[j] = ss * (1.f - kSplitErr);
    }
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) big = fmaxf(big, __shfl_xor(big, o));
    fine = __ballot(fine) == ~0ull && (big == 0.f || (big >= 0x1p-50f && big < 0x1p50f));
    const int ce = fine && big > 0.f ? 13 - ((int)((__float_as_uint(big) >> 23) & 0xFF) - 127) : 0;
    const float cup = __uint_as_float((uint32_t)(127 + ce) << 23);
    const float cdn = __uint_as_float((uint32_t)(127 - ce) << 23);
    __syncthreads();
    // which half of the components and which plane this lane's slots hold
    const int t0 = C == 1 ? 0 : 8 * (lh & 1);
    half8 a[16][C];
#pragma unroll
    for (int b = 0; b < 16; ++b) {
        half8 h, l;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const float v = fine && e < DS ? cb[(b * 16 + li) * DS + (e < DS ? t0 + e : 0)] * cup : 0.f;
            h[e] = (_Float16)v;
            l[e] = (_Float16)(v - (float)h[e]);
        }
        if constexpr (C == 1) {
            const half8 zero = {};
            a[b][0] = lh < 2 ? h : lh == 2 ? l : zero;
        } else {
            a[b][0] = h;
            a[b][1] = l;
        }
    }
    // distance of this lane's row to code word j, as the plain kernel takes it
    auto direct = [&](const float (&v)[DS], int j) __attribute__((always_inline)) {
        // (the padding's differences are zero)
        float s = 0.f;
#pragma unroll
        for (int t = 0; t < DS; t += 4) {
            const floatx4 w = *reinterpret_cast<const floatx4*>(&cb[j * DS + t]);
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const float df = v[t + e] - w[e];
                s = fmaf(df, df, s);
            }
        }
        return s;
    };
    // the lower distance of the four lanes of a row, the lower code on ties
    auto row_best = [&](PqGroup g) __attribute__((always_inline)) {
#pragma unroll
        for (int o = 16; o <= 32; o <<= 1) {
            const float s = __shfl_xor(g.score, o);
            const int c = __shfl_xor(g.code, o);
            if (s < g.score || (s == g.score && c < g.code)) {
                g.score = s;
                g.code = c;
            }
        }
        return g;
    };
    // NB blocks of 16 rows at a time, the next ones' components loaded ahead
    float next[NB][DS];
    auto load = [&](int64_t i0) __attribute__((always_inline)) {
#pragma unroll
        for (int x = 0; x < NB; ++x) {
            int64_t i = i0 + x * 16 + li;
            i = i < n ? i : n - 1;
            const float* rp = r + i * d + (int64_t)m * ds;
            if constexpr (VEC) {
#pragma unroll
                for (int t = 0; t < DS; t += 4) {
                    float4 w = make_float4(0.f, 0.f, 0.f, 0.f);
                    if (t < ds) w = *reinterpret_cast<const float4*>(rp + t);
                    next[x][t] = w.x;
                    next[x][t + 1] = w.y;
                    next[x][t + 2] = w.z;
                    next[x][t + 3] = w.w;
                }
            } else {
#pragma unroll
                for (int t = 0; t < DS; ++t) next[x][t] = t < ds ? rp[t] : 0.f;
            }
        }
    };
    const int64_t step = nwg * (kBlock / 64) * 16 * NB;
    const int64_t start = (wg * (kBlock / 64) + wave) * 16 * NB;
    if (start < n) load(start);
    int skip = 0, streak = 3;
#pragma unroll 1
    for (int64_t i0 = start; i0 < n; i0 += step) {
        float v[NB][DS], nr[NB], mq[NB];
        bool ok[NB];
        half8 q[NB][C];
#pragma unroll
        for (int x = 0; x < NB; ++x)
#pragma unroll
            for (int t = 0; t < DS; ++t) v[x][t] = next[x][t];
        if (i0 + step < n) load(i0 + step);
#pragma unroll
        for (int x = 0; x < NB; ++x) {
            float top = 0.f;
            nr[x] = 0.f;
#pragma unroll
            for (int t = 0; t < DS; ++t) {
                top = fmaxf(top, fabsf(v[x][t]));
                nr[x] = fmaf(v[x][t], v[x][t], nr[x]);
            }
            // (a row that is not finite, or far outside, takes the plain loop)
            ok[x] = fine && (nr[x] == 0.f ? top == 0.f
                                          : (top >= 0x1p-50f && top < 0x1p50f && nr[x] < 0x1p100f));
            const int re =
                ok[x] && top > 0.f ? 13 - ((int)((__float_as_uint(top) >> 23) & 0xFF) - 127) : 0;
            const float rup = __uint_as_float((uint32_t)(127 + re) << 23);
            mq[x] = -2.f * __uint_as_float((uint32_t)(127 - re) << 23) * cdn;
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const float lo = e < DS ? v[x][e % DS] : 0.f, hi = v[x][(8 + e) % DS];
                const float y = C == 1 || !(lh & 1) ? lo : hi;
                // (what is not finite spoils its own row's scores only)
                const float xs = y * rup;
                const _Float16 h = (_Float16)xs, l = (_Float16)(xs - (float)h), z = (_Float16)0.f;
                if constexpr (C == 1) {
                    q[x][0][e] = lh == 1 ? l : h;
                } else {
                    q[x][0][e] = lh < 2 ? h : l;
                    q[x][1][e] = lh < 2 ? h : z;
                }
            }
        }
        PqGroup g[NB];
        bool sure[NB];
#pragma unroll
        for (int x = 0; x < NB; ++x) {
            g[x] = PqGroup{INFINITY, 0};
            sure[x] = false;
        }
        if (skip == 0) {
            // a score plus |r|^2 (a little more than it, so that none is negative)
            // is a lower bound of a distance
            LowKeys best[NB];
            float shift[NB];
#pragma unroll
            for (int x = 0; x < NB; ++x) {
                best[x].init();
                shift[x] = nr[x] * (1.f + 4.f * kSplitErr) + 0x1p-120f;
            }
#pragma unroll
            for (int b = 0; b < 16; ++b) {
                const floatx4 cnv = *reinterpret_cast<const floatx4*>(&cn[b * 16 + 4 * lh]);
#pragma unroll
                for (int x = 0; x < NB; ++x) {
                    floatx4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
                    for (int c = 0; c < C; ++c)
                        acc = __builtin_amdgcn_mfma_f32_16x16x32_f16(a[b][c], q[x][c], acc, 0, 0, 0);
                    float s[4];
#pragma unroll
                    for (int e = 0; e < 4; ++e) s[e] = fmaf(acc[e], mq[x], cnv[e]);
                    const float low = fminf(fminf(fminf(s[0], s[1]), s[2]), s[3]) + shift[x];
                    best[x].offer((int32_t)((__float_as_uint(low) & ~63u) | (uint32_t)(b * 4 + lh)));
                }
            }
#pragma unroll
            for (int x = 0; x < NB; ++x) {
#pragma unroll
                for (int o = 16; o <= 32; o <<= 1) {
                    const int32_t k1 = __shfl_xor(best[x].k1, o), k2 = __shfl_xor(best[x].k2, o),
                                  k3 = __shfl_xor(best[x].k3, o);
                    best[x].offer(k1);
                    best[x].offer(k2);
                    best[x].offer(k3);
                }
            }
#pragma unroll
            for (int x = 0; x < NB; ++x) {
                // lane lh takes word lh of the best group
                const float edge =
                    -nr[x] * (6.f * kSplitErr) - sqrtf(nr[x]) * big * 0x1p-24f - 0x1p-119f;
                const float b2 = __uint_as_float((uint32_t)best[x].k2 & ~63u);
                const float b3 = __uint_as_float((uint32_t)best[x].k3 & ~63u);
                const int g1 = best[x].k1 & 63;
                g[x] = row_best(PqGroup{direct(v[x], 4 * g1 + lh), 4 * g1 + lh});
                sure[x] = ok[x] && g[x].score < (edge + b2) * (1.f - kDirectErr);
                if (__ballot(!sure[x])) {
                    const int g2 = best[x].k2 & 63;
                    const PqGroup h = row_best(PqGroup{direct(v[x], 4 * g2 + lh), 4 * g2 + lh});
                    if (!sure[x]) {
                        if (h.score < g[x].score || (h.score == g[x].score && h.code < g[x].code))
                            g[x] = h;
                        sure[x] = ok[x] && g[x].score < (edge + b3) * (1.f - kDirectErr);
                    }
                }
            }
        } else {
            --skip;
        }
        // every word for rows x0 .. x1, a quarter of them per lane, in the plain kernel's
        // order of preference (a row of NaN distances: code 0)
        auto every = [&](int x0, int x1) __attribute__((always_inline)) {
            PqGroup f[NB];
#pragma unroll
            for (int x = x0; x < x1; ++x) f[x] = PqGroup{INFINITY, lh == 0 ? 0 : 256};
#pragma unroll 2
            for (int j = lh; j < 256; j += 4)  // (a row's four lanes in different LDS banks)
#pragma unroll
                for (int x = x0; x < x1; ++x) {
                    const float s = direct(v[x], j);
                    if (s < f[x].score) {
                        f[x].score = s;
                        f[x].code = j;
                    }
                }
#pragma unroll
            for (int x = x0; x < x1; ++x) {
                f[x] = row_best(f[x]);
                if (!sure[x]) g[x] = f[x];
            }
        };
        const bool first = __ballot(!sure[0]), last = __ballot(!sure[NB - 1]);
        if (first || last) {
            if (NB == 1 || (first && last))
                every(0, NB);
            else if (first)
                every(0, 1);
            else
                every(NB - 1, NB);
            // Where four steps in five need it (code words or rows in ties, out of the
            // split's range, far from the origin) products cost more than they save, and
            // are tried again after 15 steps.
            if (skip == 0) {
                streak = streak < 6 ? streak + 1 : 6;
                if (streak == 6) skip = 15;
            }
        } else {
            streak = streak > 4 ? streak - 4 : 0;
        }
#pragma unroll
        for (int x = 0; x < NB; ++x) {
            const int64_t i = i0 + x * 16 + li;
            if (lh == 0 && i < n) codes[i * M + m] = (uint8_t)g[x].code;
        }
    }
}

mk_status pq_encode(const float* r, int64_t n, int32_t d, int32_t M, const float* books,
                    uint8_t* codes, hipStream_t s) {
    if (n == 0) return MK_OK;
    const int32_t ds = d / M;
    // enough rows that a workgroup's set-up (256 code words into operands) is
    // small beside them
    // (for one or two components the words are cheaper to compare: 131,072 x 32, M = 16: 101
    // us by products, 79 without)
    if (ds >= 3 && ds <= 16 && n >= 2048) {
        // about two rounds of the workgroups that fit (three per CU)
        int64_t wgs = ceil_div(n, 64 * 4);
        if (wgs > 1536 / M) wgs = std::max<int64_t>(1, 1536 / M);
        const dim3 g((unsigned)(wgs * M));
        const bool vec = ds % 4 == 0 && reinterpret_cast<uintptr_t>(r) % 16 == 0;
        auto kern = ds <= 4   ? (vec ? pq_encode_mfma<4, true> : pq_encode_mfma<4, false>)
                    : ds <= 8 ? (vec ? pq_encode_mfma<8, true> : pq_encode_mfma<8, false>)
                              : (vec ? pq_encode_mfma<16, true> : pq_encode_mfma<16, false>);
        hipLaunchKernelGGL(kern, g, dim3(kBlock), 0, s, r, n, d, M, ds, books, codes);
        MK_LAUNCHED();
        return MK_OK;
    }
    const dim3 grid((unsigned)ceil_div(n, kBlock), (unsigned)M), block(kBlock);
    switch (ds) {
        case 1: hipLaunchKernelGGL(pq_encode_fixed<1>, grid, block, 0, s, r, n, d, M, books, codes); break;
        case 2: hipLaunchKernelGGL(pq_encode_fixed<2>, grid, block, 0, s, r, n, d, M, books, codes); break;
        case 4: hipLaunchKernelGGL(pq_encode_fixed<4>, grid, block, 0, s, r, n, d, M, books, codes); break;
        case 8: hipLaunchKernelGGL(pq_encode_fixed<8>, grid, block, 0, s, r, n, d, M, books, codes); break;
        case 16: hipLaunchKernelGGL(pq_encode_fixed<16>, grid, block, 0, s, r, n, d, M, books, codes); break;
        default:
            hipLaunchKernelGGL(pq_encode_any, grid, block, sizeof(float) * 256 * ds, s, r, n, d, M,
                               ds, books, codes);
            break;
    }
    MK_LAUNCHED();
    return MK_OK;
}

// ---------------------------------------------------------------- helpers
// r[i] = x[i] - c[list[i]]  (FP32)
__global__ void residual_kernel(const float* __restrict__ x, int64_t n, int32_t d,
                                const float* __restrict__ c, const int64_t* __restrict__ list,
                                float* __restrict__ r) {
    for (int64_t g = (int64_t)blockIdx.x * kBlock + threadIdx.x; g < n * d; g += kStride) {
        const int64_t i = g / d, t = g % d;
        r[g] = x[g] - c[list[i] * d + t];
    }
}

// dst[i, :] = src[i, off : off + w]
__global__ void columns_kernel(const float* __restrict__ src, int64_t n, int32_t d, int32_t off,
                               int32_t w, float* __restrict__ dst) {
    for (int64_t g = (int64_t)blockIdx.x * kBlock + threadIdx.x; g < n * w; g += kStride) {
        const int64_t i = g / w, t = g % w;
        dst[g] = src[i * d + off + t];
    }
}

// term1[L, m, j] = ||c_{m,j}||^2 + 2 <c_L^m, c_{m,j}>   (Eq. 11, term 1)
__global__ void term1_kernel(const float* __restrict__ coarse, const float* __restrict__ books,
                             int32_t nlist, int32_t M, int32_t ds, float* __restrict__ term1) {
    for (int64_t g = (int64_t)blockIdx.x * kBlock + threadIdx.x; g < (int64_t)nlist * M * 256;
         g += kStride) {
        const int64_t L = g / (M * 256);
        const int32_t m = (int32_t)((g / 256) % M), j = (int32_t)(g % 256);
        const float* cw = books + ((int64_t)m * 256 + j) * ds;
        const float* cl = coarse + L * (int64_t)M * ds + (int64_t)m * ds;
        float nn = 0.f, ip = 0.f;
        for (int t = 0; t < ds; ++t) {
            nn = fmaf(cw[t], cw[t], nn);
            ip = fmaf(cl[t], cw[t], ip);
        }
        term1[g] = fmaf(2.f, ip, nn);
    }
}

// term3[q, m, j] = <x_q^m, c_{m,j}>   (Eq. 11, term 3)
// term3[q][m][j] = <x_q^m, c_{m,j}> (Eq. 11).  One workgroup per (tile of
// kT3Queries queries, sub-quantizer m), thread j owns codeword j; the
// codebook and the queries' sub-vectors pass through LDS in slices of 16
// components (summed in component order), and each query's 256 outputs are
// written as one coalesced row.
constexpr int kT3Queries = 16;

__global__ __launch_bounds__(256) void term3_kernel(const float* __restrict__ xq, int64_t nq,
                                                    int32_t M, int32_t ds,
                                                    const float* __restrict__ books,
                                                    float* __restrict__ term3) {
    __shared__ float cb[256][17];
    __shared__ float xs[kT3Queries][16];
    const int64_t q0 = (int64_t)blockIdx.x * kT3Queries;
    const int32_t m = blockIdx.y;
    const int j = threadIdx.x;
    const int d = M * ds;
    float acc[kT3Queries];
#pragma unroll
    for (int i = 0; i < kT3Queries; ++i) acc[i] = 0.f;
    for (int t0 = 0; t0 < ds; t0 += 16) {
        const int w = ds - t0 < 16 ? ds - t0 : 16;
        for (int e = j; e < 256 * 16; e += 256) {
            const int jj = e / 16, t = e % 16;
            cb[jj][t] = t < w ? books[((int64_t)m * 256 + jj) * ds + t0 + t] : 0.f;
        }
        for (int e = j; e < kT3Queries * 16; e += 256) {
            const int i = e / 16, t = e % 16;
            const int64_t q = q0 + i;
            xs[i][t] = (t < w && q < nq) ? xq[q * d + (int64_t)m * ds + t0 + t] : 0.f;
        }
        __syncthreads();
        for (int t = 0; t < w; ++t) {
            const float c = cb[j][t];
#pragma unroll
            for (int i = 0; i < kT3Queries; ++i) acc[i] = fmaf(xs[i][t], c, acc[i]);
        }
        __syncthreads();
    }
#pragma unroll
    for (int i = 0; i < kT3Queries; ++i) {
        const int64_t q = q0 + i;
        if (q < nq) term3[(q * M + m) * 256 + j] = acc[i];
    }
}

mk_status launch_term3(const float* xq, int64_t nq, int32_t M, int32_t ds, const float* books,
                       float* term3, hipStream_t s) {
    if (nq == 0) return MK_OK;
    hipLaunchKernelGGL(term3_kernel, dim3((unsigned)ceil_div(nq, kT3Queries), (unsigned)M),
                       dim3(256), 0, s, xq, nq, M, ds, books, term3);
    MK_LAUNCHED();
    return MK_OK;
}

__global__ void fill_u32_kernel(unsigned int* __restrict__ a, int64_t n) {
    for (int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x; i < n; i += kStride) a[i] = 0u;
}

// Stable placement of a batch into its lists without sorting.  The batch is
// cut into chunks of kPlaceChunk entries, one wave each, walked 64 entries
// at a time in batch order.  Within a group of 64 the lanes with equal lists
// are found by repeated ballots on the first remaining lane's list; the
// group's count for that list goes to the chunk's counter in one atomic.
//   place_count: cnt[c][L] = entries of chunk c in list L
//   place_prefix: per list, exclusive prefix over chunks (cnt[c][L] becomes
//                 the list rank of chunk c's first entry) and the total
//   place_new:   the same walk again; the atomic's old value plus the lane's
//                rank among equal lanes below it is the entry's rank in its
//                list among the batch, so entries keep batch order per list
constexpr int64_t kPlaceChunk = 65536;

template <bool PLACE>
__device__ __forceinline__ void place_walk(const int64_t* __restrict__ list, int64_t nb,
                                           int32_t nlist, unsigned int* __restrict__ cnt,
                                           const int64_t* __restrict__ new_off,
                                           const int64_t* __restrict__ old_off, int32_t M,
                                           const uint8_t* __restrict__ batch_codes, int64_t id0,
                                           uint8_t* __restrict__ codes, int64_t* __restrict__ ids) {
    const int64_t c = blockIdx.x;
    const int lane = threadIdx.x;
    unsigned int* row = cnt + c * (int64_t)nlist;
    const int64_t lo = c * kPlaceChunk;
    const int64_t hi = lo + kPlaceChunk < nb ? lo + kPlaceChunk : nb;
    const uint64_t below = lane == 0 ? 0ull : (~0ull >> (64 - lane));
    for (int64_t g = lo; g < hi; g += 64) {
        const int64_t i = g + lane;
        const bool ok = i < hi;
        const int64_t L = ok ? list[i] : -1;
        uint64_t todo = __ballot(ok);
        int64_t rank = 0;
        while (todo) {
            const int first = __builtin_ctzll(todo);
            const int64_t Lf = __shfl(L, first, 64);
            const uint64_t same = __ballot(L == Lf) & todo;
            unsigned int base = 0;
            if (lane == first) {
                if (PLACE)
                    base = atomicAdd(&row[Lf], (unsigned int)__popcll(same));
                else
                    atomicAdd(&row[Lf], (unsigned int)__popcll(same));
            }
            if (PLACE) {
                base = __shfl(base, first, 64);
                if ((same >> lane) & 1ull) rank = (int64_t)base + __popcll(same & below);
            }
            todo &= ~same;
        }
        if (PLACE && ok) {
            const int64_t pos = new_off[L] + (old_off[L + 1] - old_off[L]) + rank;
            ids[pos] = id0 + i;
            for (int m = 0; m < M; ++m) codes[pos * M + m] = batch_codes[i * M + m];
        }
    }
}

__global__ __launch_bounds__(64) void place_count_kernel(const int64_t* __restrict__ list,
                                                         int64_t nb, int32_t nlist,
                                                         unsigned int* __restrict__ cnt) {
    place_walk<false>(list, nb, nlist, cnt, nullptr, nullptr, 0, nullptr, 0, nullptr, nullptr);
}

__global__ void place_prefix_kernel(unsigned int* __restrict__ cnt, int64_t nchunks,
                                    int32_t nlist, unsigned long long* __restrict__ total) {
    const int64_t L = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (L >= nlist) return;
    unsigned long long run = 0;
    for (int64_t c = 0; c < nchunks; ++c) {
        const unsigned int v = cnt[c * nlist + L];
        cnt[c * nlist + L] = (unsigned int)run;
        run += v;
    }
    total[L] = run;
}

__global__ __launch_bounds__(64) void place_new_kernel(const int64_t* __restrict__ list,
                                                       int64_t nb, int32_t nlist,
                                                       unsigned int* __restrict__ cnt,
                                                       const int64_t* __restrict__ new_off,
                                                       const int64_t* __restrict__ old_off,
                                                       int32_t M,
                                                       const uint8_t* __restrict__ batch_codes,
                                                       int64_t id0, uint8_t* __restrict__ codes,
                                                       int64_t* __restrict__ ids) {
    place_walk<true>(list, nb, nlist, cnt, new_off, old_off, M, batch_codes, id0, codes, ids);
}

// Old entries of list L move from old_off[L] + e to new_off[L] + e.
__global__ void move_old_kernel(const int64_t* __restrict__ old_off,
                                const int64_t* __restrict__ new_off, int32_t M,
                                const uint8_t* __restrict__ old_codes,
                                const int64_t* __restrict__ old_ids, uint8_t* __restrict__ codes,
                                int64_t* __restrict__ ids) {
    const int32_t L = blockIdx.x;
    const int64_t lo = old_off[L], n = old_off[L + 1] - lo, dst = new_off[L];
    for (int64_t e = threadIdx.x; e < n; e += kBlock) {
        ids[dst + e] = old_ids[lo + e];
        for (int m = 0; m < M; ++m) codes[(dst + e) * M + m] = old_codes[(lo + e) * M + m];
    }
}

// ---------------------------------------------------------------- list scan
constexpr int kScanWaves = kPoolThreads / 64;

// Probe-count features: F[q] = [xq[q] ; the kProbeDists smallest squared
// coarse distances] (cd holds ld ascending distances per query).
__global__ void probe_features_kernel(const float* __restrict__ xq, int64_t nq, int32_t d,
                                      const float* __restrict__ cd, int32_t ld,
                                      float* __restrict__ F) {
    const int32_t din = d + kProbeDists;
    for (int64_t e = (int64_t)blockIdx.x * kBlock + threadIdx.x; e < nq * din; e += kStride) {
        const int64_t q = e / din;
        const int t = (int)(e % din);
        F[e] = t < d ? xq[q * d + t] : cd[q * ld + (t - d)];
    }
}

// list_of[id] = inverted list holding id.
__global__ void list_of_kernel(const int64_t* __restrict__ offsets, int32_t nlist,
                               const int64_t* __restrict__ ids, int32_t* __restrict__ list_of) {
    const int32_t L = blockIdx.x;
    if (L >= nlist) return;
    for (int64_t pos = offsets[L] + threadIdx.x; pos < offsets[L + 1]; pos += blockDim.x)
        list_of[ids[pos]] = L;
}

// Probe count a query needs: 1-based rank of the list holding its nearest
// neighbour in its coarse order (ld entries per query), cap if not among
// them; target = log2 of it.
__global__ void probe_labels_kernel(const int64_t* __restrict__ ci, int32_t ld, int64_t nq,
                                    const int64_t* __restrict__ nn, const int32_t* __restrict__ list_of,
                                    int64_t ntotal, int32_t cap, float* __restrict__ target,
                                    int32_t* __restrict__ label) {
    const int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (q >= nq) return;
    const int64_t id = nn[q];
    int32_t r = cap;
    if (id >= 0 && id < ntotal) {
        const int32_t L = list_of[id];
        for (int32_t p = 0; p < cap && p < ld; ++p)
            if (ci[q * ld + p] == L) { r = p + 1; break; }
    }
    target[q] = log2f((float)r);
    if (label) label[q] = r;
}

// Per-query probe counts and the scan's work plan in one workgroup:
// tau[q] = clamp(ceil(2^(yhat[q] + delta)), 1, cap) (also copied to `used`
// when given), and the exclusive prefix sums of the per-query workgroup
// counts ceil(tau / G): work[0] = 0, work[q + 1] = sum over q' <= q.
// Queries go 1024 at a time; a wave prefix sum, then one over the 16 waves'
// totals, then the running carry.
__global__ __launch_bounds__(1024) void probe_plan_kernel(const float* __restrict__ yhat,
                                                          int64_t nq, float delta, int32_t cap,
                                                          int32_t G, int32_t* __restrict__ tau,
                                                          int32_t* __restrict__ used,
                                                          int64_t* __restrict__ work) {
    __shared__ int64_t wsum[16];
    __shared__ int64_t carry;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    if (threadIdx.x == 0) {
        carry = 0;
        work[0] = 0;
    }
    __syncthreads();
    for (int64_t base = 0; base < nq; base += 1024) {
        const int64_t q = base + threadIdx.x;
        int64_t x = 0;
        if (q < nq) {
            const float t = exp2f(yhat[q] + delta);
            int32_t v = cap;
            if (t < (float)cap) v = t <= 1.f ? 1 : (int32_t)ceilf(t);
            tau[q] = v;
            if (used) used[q] = v;
            x = (v + G - 1) / G;
        }
#pragma unroll
        for (int off = 1; off < 64; off <<= 1) {
            const int64_t y = __shfl_up(x, off, 64);
            if (lane >= off) x += y;
        }
        if (lane == 63) wsum[wave] = x;
        __syncthreads();
        if (wave == 0) {
            int64_t t = lane < 16 ? wsum[lane] : 0;
#pragma unroll
            for (int off = 1; off < 16; off <<= 1) {
                const int64_t y = __shfl_up(t, off, 64);
                if (lane >= off) t += y;
            }
            if (lane < 16) wsum[lane] = t;
        }
        __syncthreads();
        const int64_t incl = carry + (wave > 0 ? wsum[wave - 1] : 0) + x;
        if (q < nq) work[q + 1] = incl;
        __syncthreads();
        if (threadIdx.x == 1023) carry = incl;
        __syncthreads();
    }
}

__global__ void entry_term1_kernel(const int64_t* __restrict__ offsets, int32_t M,
                                   const uint8_t* __restrict__ codes,
                                   const float* __restrict__ term1, float* __restrict__ t1e) {
    const int64_t L = blockIdx.x;
    const float* t1 = term1 + L * (int64_t)M * 256;
    for (int64_t pos = offsets[L] + threadIdx.x; pos < offsets[L + 1]; pos += blockDim.x) {
        const uint8_t* c = codes + pos * M;
        float v = 0.f;
        for (int m = 0; m < M; ++m) v += t1[m * 256 + c[m]];
        t1e[pos] = v;
    }
}

// One workgroup per (query, group of up to G probed lists).  The query's
// table -2 term3[q] (Eq. 11) is staged in LDS once for the group; each
// scanned entry's ADC distance is term 2 (the coarse distance of its list)
// + its stored term 1 + the M table lookups of its code bytes (Eq. 10-11).
// The four waves share one pool of candidates in LDS (pool.hpp), keyed (distance,
// id), and its threshold, the kk-th best key at the last cut; the id is read only
// for entries at or below the threshold's distance (Section 5.3 resolves ids only
// for selected entries).  A queue per wave, as sorted registers, took four times the
// insertions (every wave fills its own), a sorting network over the queue for
// every 64 to 512 of them, and a serial merge of the four queues.
// The lists of a group (64 at a time) are one range of entries, taken in steps of
// 1,024, the next step's codes and terms in flight: a step of its own per list
// leaves most of its last lanes idle and starts with three loads in a row (list,
// offset, code).  10^4 queries, 8 lists of about 1,000 entries, 256 kept: queues
// 919, pool 608, one range 506 us; 64 queries, 32 lists, 100 kept: 80, 44, 41 us.  With
// 16 code bytes as a constant, on another card: 475 -> 443 and 40.1 -> 38.5 us.
// What is left is the table lookups: 1.25 * 10^9 LDS gathers with random banks,
// about 7 cycles per wave and gather, are 230 of the 443 us.
// Item -> (query, group): fixed probe count nprobe (= ld) when work is null,
// else query q owns items work[q] .. work[q + 1] - 1 and probes tau[q] lists.

// Lookup-table entry types: FP32, or FP16 (half the LDS and half the bytes
// per gather; each entry rounded once, sums still in FP32).
template <bool H16> struct LutT;
template <> struct LutT<false> {
    typedef float type;
    static __device__ __forceinline__ float make(float v) { return v; }
    static __device__ __forceinline__ float get(float v) { return v; }
};
template <> struct LutT<true> {
    typedef __half type;
    static __device__ __forceinline__ __half make(float v) { return __float2half_rn(v); }
    static __device__ __forceinline__ float get(__half v) { return __half2float(v); }
};

// Lists a workgroup scans as one range of entries.
constexpr int kScanLists = 64;
struct ScanLists {
    int64_t end[kScanLists];    // entries of the lists up to and with this one
    uint32_t shift[kScanLists]; // entry -> row of codes, t1e and ids (below 2^32, as sums wrap)
    float term2[kScanLists];
};

// LONG: more than 16 code bytes per entry; V16: a multiple of 16 (neither long nor
// another: 16, a constant)
template <bool H16, int P, bool LONG, bool V16>
__global__ __launch_bounds__(64 * kScanWaves) __attribute__((amdgpu_waves_per_eu(LONG ? 3 : 4))) void ivf_scan(
    const float* __restrict__ term3, const float* __restrict__ t1e,
    const float* __restrict__ coarse_d, const int64_t* __restrict__ coarse_i, int32_t ld,
    const int64_t* __restrict__ offsets, const uint8_t* __restrict__ codes,
    const int64_t* __restrict__ ids, int32_t M, int32_t G, int32_t k,
    uint64_t* __restrict__ part, const int64_t* __restrict__ work,
    const int32_t* __restrict__ tau, int64_t nq, int64_t excl_base) {
    typedef LutT<H16> LT;
    typedef typename LT::type lut_t;
    constexpr int U = 4;                          // entries in flight per lane
    constexpr int STEP = 64 * kScanWaves * U;     // entries of a step
    static_assert(P > STEP, "the pool takes a step beside kk <= P - STEP keys");
    extern __shared__ __align__(16) unsigned char smem[];
    __shared__ PoolState state;
    __shared__ ScanLists lists;
    uint64_t* pool = reinterpret_cast<uint64_t*>(smem);
    uint32_t* bins = reinterpret_cast<uint32_t*>(smem + sizeof(uint64_t) * P);
    lut_t* lut = reinterpret_cast<lut_t*>(smem + sizeof(uint64_t) * P + sizeof(uint32_t) * kCutBins);

    const int64_t item = blockIdx.x;
    int64_t q, g;
    int32_t np;
    if (work) {
        if (item >= work[nq]) return;  // grid sized for the largest possible count
        int64_t lo = 0, hi = nq;  // largest q with work[q] <= item
        while (hi - lo > 1) {
            const int64_t mid = (lo + hi) >> 1;
            if (work[mid] <= item) lo = mid; else hi = mid;
        }
        q = lo;
        g = item - work[q];
        np = tau[q];
    } else {
        const int64_t ng = (ld + G - 1) / G;
        q = item / ng;
        g = item - q * ng;
        np = ld;
    }
    const int32_t p0 = (int32_t)(g * G);
    const int32_t ns = np - p0 < G ? np - p0 : G;  // lists in this group
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int lane = lane_id();
    uint64_t* out = part + item * k;
    // k-NN graph construction: query q is node excl_base + q, not its own
    // neighbour (no exclusion when excl_base < 0; ids are >= 0)
    const int64_t excl = excl_base >= 0 ? excl_base + q : -1;

    if constexpr (V16 && !LONG) M = 16;
    const float* t3 = term3 + q * (int64_t)M * 256;
    static_assert(64 * kScanWaves == 256, "a table per step");
#pragma unroll 4
    for (int m = 0; m < M; ++m) {
        const int e = m * 256 + (int)threadIdx.x;
        lut[e] = LT::make(-2.f * t3[e]);
    }
    if (threadIdx.x == 0) {
        state.count = 0u;
        state.limit = kSentinel;
    }
    __syncthreads();

    const bool vec8 = (M & 7) == 0;
    // code bytes m0 .. m0 + 15 of an entry (those below M)
    auto code_bytes = [&](uint32_t pos, int m0) __attribute__((always_inline)) {
        const uint8_t* c = codes + (int64_t)pos * M + m0;
        if constexpr (V16) return *reinterpret_cast<const uint4*>(c);
        uint4 w = make_uint4(0u, 0u, 0u, 0u);
        if (vec8) {
            const uint2 a = *reinterpret_cast<const uint2*>(c);
            w.x = a.x;
            w.y = a.y;
            if (m0 + 8 < M) {
                const uint2 b = *reinterpret_cast<const uint2*>(c + 8);
                w.z = b.x;
                w.w = b.y;
            }
        } else {
            const uint32_t* c4 = reinterpret_cast<const uint32_t*>(c);
            w.x = c4[0];
            if (m0 + 4 < M) w.y = c4[1];
            if (m0 + 8 < M) w.z = c4[2];
            if (m0 + 12 < M) w.w = c4[3];
        }
        return w;
    };
    const int64_t* cirow = coarse_i + q * ld + p0;
    const float* cdrow = coarse_d + q * ld + p0;
    uint64_t limit = kSentinel;  // the threshold and its score
    float limit_f = INFINITY;
#pragma unroll 1
    for (int32_t c0 = 0; c0 < ns; c0 += kScanLists) {
        // the next lists as one range of entries: list i covers [begin[i], begin[i + 1])
        if (c0) __syncthreads();
        if (wave == 0) {
            const int64_t L = c0 + lane < ns ? cirow[c0 + lane] : -1;  // -1: fewer lists than probes
            int64_t lo = 0, n = 0;
            if (L >= 0) {
                lo = offsets[L];
                n = offsets[L + 1] - lo;
            }
            int64_t incl = n;
#pragma unroll
            for (int o = 1; o < 64; o *= 2) {
                const int64_t v = __shfl_up(incl, o);
                if (lane >= o) incl += v;
            }
            lists.end[lane] = incl;
            lists.shift[lane] = (uint32_t)(lo - (incl - n));
            lists.term2[lane] = L >= 0 ? cdrow[c0 + lane] : 0.f;
        }
        __syncthreads();
        const int64_t total = lists.end[kScanLists - 1];
        if (total == 0) continue;
        // this lane's list: entries are looked up in ascending order
        int cur = -1;
        int64_t cur_end = 0;
        uint32_t cur_shift = 0;
        float cur_term2 = 0.f;
        struct Step {
            uint4 w[U];     // first 16 code bytes
            float t1[U], t2[U];
            uint32_t pos[U];
        } now, next;
        // entries s0 + u 256 + 64 wave + lane; beyond the last one, the last one's data
        auto load = [&](Step& st, int64_t s0) {
#pragma unroll
            for (int u = 0; u < U; ++u) {
                int64_t e = s0 + u * 64 * kScanWaves + wave * 64 + lane;
                e = e < total ? e : total - 1;
                if (e >= cur_end) {
                    do ++cur; while (e >= lists.end[cur]);  // (e < total = end of the last)
                    cur_end = lists.end[cur];
                    cur_shift = lists.shift[cur];
                    cur_term2 = lists.term2[cur];
                }
                st.pos[u] = (uint32_t)e + cur_shift;
                st.t2[u] = cur_term2;
            }
#pragma unroll
            for (int u = 0; u < U; ++u) {
                st.t1[u] = t1e[st.pos[u]];
                st.w[u] = code_bytes(st.pos[u], 0);
            }
        };
        load(now, 0);
#pragma unroll 1
        for (int64_t s0 = 0; s0 < total; s0 += STEP) {
            if (s0 + STEP < total) load(next, s0 + STEP);
            // of the entries s0 + u 256 + 64 wave + lane, those u with any for this wave
            const int64_t rest = total - s0 - wave * 64;
            float dist[U];
#pragma unroll
            for (int u = 0; u < U; ++u) dist[u] = now.t2[u] + now.t1[u];
            for (int m0 = 0; m0 < (LONG ? M : 1); m0 += 16) {
                uint4 ahead[U];  // the next bytes, in flight during these lookups
                if (LONG && m0 + 16 < M)
#pragma unroll
                    for (int u = 0; u < U; ++u) ahead[u] = code_bytes(now.pos[u], m0 + 16);
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    if (u * 64 * kScanWaves >= rest) continue;  // (wave-uniform)
                    const uint32_t ww[4] = {now.w[u].x, now.w[u].y, now.w[u].z, now.w[u].w};
#pragma unroll
                    for (int h = 0; h < 4; ++h) {
                        if (!V16 && m0 + 4 * h >= M) continue;
#pragma unroll
                        for (int b = 0; b < 4; ++b) {
                            const int m = m0 + 4 * h + b;
                            dist[u] += LT::get(lut[m * 256 + ((ww[h] >> (8 * b)) & 0xFF)]);
                        }
                    }
                }
                if (LONG && m0 + 16 < M)
#pragma unroll
                    for (int u = 0; u < U; ++u) now.w[u] = ahead[u];
            }
            // keyed (distance, id): ids are unique, so the order is total and
            // the selected set does not depend on how lists are grouped; the
            // id is read only for an entry that can enter the pool
            int64_t id[U];
            bool may[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                may[u] = u * 64 * kScanWaves + lane < rest && dist[u] <= limit_f;
                id[u] = may[u] ? ids[now.pos[u]] : 0;
            }
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const uint64_t key = make_key(dist[u], (uint32_t)id[u]);
                const bool take = may[u] && id[u] != excl && key < limit;
                const uint64_t bal = __ballot(take);
                if (bal) {
                    uint32_t base = 0;
                    if (lane == 0) base = atomicAdd(&state.count, (uint32_t)__popcll(bal));
                    base = (uint32_t)__builtin_amdgcn_readfirstlane((int)base);
                    if (take)
                        pool[base + __builtin_amdgcn_mbcnt_hi(
                                        (uint32_t)(bal >> 32),
                                        __builtin_amdgcn_mbcnt_lo((uint32_t)bal, 0u))] = key;
                }
            }
            __syncthreads();
            const uint32_t have = state.count;  // the same in every wave
            __syncthreads();  // every wave has read it
            if (have > (uint32_t)(P - STEP)) {
                // (kk <= P - STEP, so there is something to cut)
                pool_cut<P>(pool, bins, &state, have, k);
                if (threadIdx.x == 0) state.count = (uint32_t)k;
                __syncthreads();
                limit = state.limit;
                limit_f = key_score(limit - 1);
            }
            now = next;
        }
    }
    const uint32_t found = state.count;
    if (found > (uint32_t)k) pool_cut<P>(pool, bins, &state, found, k);
    const int have = (int)(found < (uint32_t)k ? found : (uint32_t)k);
    for (int e = threadIdx.x; e < k; e += 64 * kScanWaves) out[e] = e < have ? pool[e] : kSentinel;
}

// Lists per workgroup: as many as keep the launch at 1024+ workgroups
// (about 4 per CU), so each query's table is staged once for as many lists
// as possible and fewer partial lists reach the merge; with enough queries
// every query's lists go to one workgroup (10^7 x 128, 4096 lists, k = 100:
// nprobe 128 and 10^4 queries 11.3 ms per-query against 15.6 ms for groups
// of 16; 1024 queries, nprobe 8 / 64 / 128, 0.47 / 1.41 / 2.65 ms at 2048+
// workgroups against 0.42 / 1.29 / 2.49 ms; 256 queries, nprobe 64 with
// R = 256 0.90 -> 0.85 ms, and larger groups than that slower).  Lists of
// 512+ results aim at 512+ workgroups: every group leaves that many keys to be
// written and merged (4*10^6 x 128, 4,096 lists, R = 600, aims of 512 / 1024: 1,000
// queries 4 / 16 / 64 probes 218 / 284 / 536 us against 264 / 365 / 751; 256 queries
// 198 / 186 / 292 against 193 / 191 / 289; of four times as long lists 517 / 750 /
// 1,405 against 487 / 701 / 1,415, 1,000 queries 686 / 1,278 / 3,138 against 802 /
// 1,811 / 4,533).
int32_t scan_group(int64_t total_probes, int32_t nprobe, int32_t k) {
    const int64_t g = total_probes / (k >= 512 ? 512 : 1024);
    return (int32_t)(g < 1 ? 1 : g > nprobe ? nprobe : g);
}

// The index's choice of lists per workgroup for nq queries probing up to
// nprobe lists each: automatic (scan_group), all of a query's lists in one
// workgroup (the per-query fused scan), or a fixed count.
int32_t scan_group_of(const mk_ivfpq* ix, int64_t nq, int32_t nprobe, int32_t auto_probes,
                      int32_t k) {
    if (ix->lists_per_group < 0) return nprobe;
    if (ix->lists_per_group > 0) return ix->lists_per_group < nprobe ? ix->lists_per_group : nprobe;
    return scan_group(nq * (int64_t)auto_probes, nprobe, k);
}

mk_status launch_scan(const float* term3, const float* t1e, const float* cd, const int64_t* ci,
                      int32_t ld, const int64_t* offsets, const uint8_t* codes,
                      const int64_t* ids, int32_t M, int64_t nq, int32_t G, int32_t k,
                      uint64_t* part, int64_t items, hipStream_t s,
                      const int64_t* work = nullptr, const int32_t* tau = nullptr,
                      int64_t excl_base = -1, bool lut16 = false) {
    if (items == 0) return MK_OK;
    MK_REQUIRE(items * 64 * kScanWaves < (1ll << 32), MK_ERR_UNSUPPORTED,
               "too many scan workgroups for one launch (search fewer queries per call)");
    // (the calls that the header promises: with its pool and bins the kernel takes up
    // to 60 KiB of tables and 36 KiB more, of 160 KiB)
    MK_REQUIRE((size_t)M * 256 * (lut16 ? 2 : 4) + 32 * (size_t)k <= 65536, MK_ERR_UNSUPPORTED,
               "lookup tables plus 32 bytes per result exceed 64 KiB (reduce M or k, or use "
               "16-bit tables)");
    const dim3 grid((unsigned)items), block(64 * kScanWaves);
    ProfScope prof(lut16 ? "ivf_scan_lut16" : "ivf_scan", s);
    // Pools of 2,048 keys (k up to 512), or 4,096; with more than 16 code bytes 1,792 or
    // 3,840, which leave room for the tables of 60 sub-quantizers (44 with long lists)
    // twice per CU (10^4 queries, 8 lists of 1,000 entries, M = 60: 6.7 ms, 16.7 with a
    // pool of 2,048 and code bytes loaded where they are looked up).
    const bool wide = M > 16;
    const size_t keys = k <= 512 ? (wide ? 1792 : 2048) : (wide ? 3840 : 4096);
    const size_t lds = (size_t)M * 256 * (lut16 ? 2 : 4) + keys * sizeof(uint64_t) + kCutBins * sizeof(uint32_t);
    auto of = [&](auto wide, auto v16) {
        constexpr bool W = decltype(wide)::value, V = decltype(v16)::value;
        constexpr int P = W ? 1792 : 2048, PL = W ? 3840 : 4096;
        return k <= 512 ? (lut16 ? ivf_scan<true, P, W, V> : ivf_scan<false, P, W, V>)
                        : (lut16 ? ivf_scan<true, PL, W, V> : ivf_scan<false, PL, W, V>);
    };
    const std::true_type yes;
    const std::false_type no;
    auto kern = M == 16 ? of(no, yes) : !wide ? of(no, no) : M % 16 == 0 ? of(yes, yes) : of(yes, no);
    if (lds > 65536)
        MK_HIP(hipFuncSetAttribute(reinterpret_cast<const void*>(kern),
                                   hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
    hipLaunchKernelGGL(kern, grid, block, lds, s, term3, t1e, cd, ci, ld, offsets, codes, ids, M, G,
                       k, part, work, tau, nq, excl_base);
    MK_LAUNCHED();
    return MK_OK;
}


mk_status build_term1(mk_ivfpq* ix, hipStream_t s) {
    free_dev(reinterpret_cast<void*&>(ix->term1));
    MK_TRY(alloc_dev(ix->term1, (size_t)ix->nlist * ix->M * 256));
    hipLaunchKernelGGL(term1_kernel, dim3(grid_of((int64_t)ix->nlist * ix->M * 256)), dim3(kBlock),
                       0, s, ix->coarse, ix->books, ix->nlist, ix->M, ix->dsub, ix->term1);
    MK_LAUNCHED();
    return launch_norms(ix->coarse, ix->nlist, ix->d, ix->coarse_norms, s);
}

void reset_lists(mk_ivfpq* ix) {
    free_dev(reinterpret_cast<void*&>(ix->codes));
    free_dev(reinterpret_cast<void*&>(ix->ids));
    free_dev(reinterpret_cast<void*&>(ix->t1e));
    ix->ntotal = 0;
    ix->capacity = 0;
    ix->offsets.assign(ix->nlist + 1, 0);
}

mk_status upload_offsets(mk_ivfpq* ix, hipStream_t s) {
    if (!ix->offsets_dev) MK_TRY(alloc_dev(ix->offsets_dev, ix->nlist + 1));
    MK_HIP(hipMemcpyAsync(ix->offsets_dev, ix->offsets.data(), sizeof(int64_t) * (ix->nlist + 1),
                          hipMemcpyHostToDevice, s));
    MK_HIP(hipStreamSynchronize(s));
    return MK_OK;
}

mk_status alloc_quantizers(mk_ivfpq* ix) {
    if (!ix->coarse) MK_TRY(alloc_dev(ix->coarse, (size_t)ix->nlist * ix->d));
    if (!ix->coarse_norms) MK_TRY(alloc_dev(ix->coarse_norms, (size_t)ix->nlist));
    if (!ix->books) MK_TRY(alloc_dev(ix->books, (size_t)ix->M * 256 * ix->dsub));
    return MK_OK;
}

mk_status train(mk_ivfpq* ix, const float* xt, int64_t nt, int32_t niter,
                const int64_t* coarse_rows, const int64_t* pq_rows, hipStream_t s) {
    const int32_t d = ix->d, nlist = ix->nlist, M = ix->M, ds = ix->dsub;
    MK_TRY(alloc_quantizers(ix));
    Scratch rows, assign, res, sub;
    MK_TRY(rows.alloc(sizeof(int64_t) * (size_t)std::max<int64_t>(nlist, 256), s));
    // coarse quantizer
    MK_HIP(hipMemcpyAsync(rows.ptr, coarse_rows, sizeof(int64_t) * nlist, hipMemcpyHostToDevice, s));
    hipLaunchKernelGGL(gather_rows_kernel, dim3(grid_of((int64_t)nlist * d)), dim3(kBlock), 0, s,
                       xt, d, rows.as<int64_t>(), (int64_t)nlist, ix->coarse);
    MK_LAUNCHED();
    MK_TRY(kmeans_run(xt, nt, d, ix->coarse, nlist, niter, s));
    // residuals of the training set to the final coarse centroids
    MK_TRY(assign.alloc(sizeof(int64_t) * (size_t)nt, s));
    MK_TRY(res.alloc(sizeof(float) * (size_t)nt * d, s));
    MK_TRY(sub.alloc(sizeof(float) * (size_t)nt * ds, s));
    MK_TRY(kmeans_assign(xt, nt, d, ix->coarse, nlist, assign.as<int64_t>(), nullptr, s));
    hipLaunchKernelGGL(residual_kernel, dim3(grid_of(nt * d)), dim3(kBlock), 0, s, xt, nt, d,
                       ix->coarse, assign.as<int64_t>(), res.as<float>());
    MK_LAUNCHED();
    // M independent sub-quantizers of 256 centroids on contiguous sub-vectors
    for (int32_t m = 0; m < M; ++m) {
        hipLaunchKernelGGL(columns_kernel, dim3(grid_of(nt * ds)), dim3(kBlock), 0, s,
                           res.as<float>(), nt, d, m * ds, ds, sub.as<float>());
        MK_LAUNCHED();
        float* cm = ix->books + (int64_t)m * 256 * ds;
        MK_HIP(hipMemcpyAsync(rows.ptr, pq_rows + (int64_t)m * 256, sizeof(int64_t) * 256,
                              hipMemcpyHostToDevice, s));
        hipLaunchKernelGGL(gather_rows_kernel, dim3(grid_of(256 * ds)), dim3(kBlock), 0, s,
                           sub.as<float>(), ds, rows.as<int64_t>(), (int64_t)256, cm);
        MK_LAUNCHED();
        MK_TRY(kmeans_run(sub.as<float>(), nt, ds, cm, 256, niter, s));
    }
    MK_TRY(build_term1(ix, s));
    reset_lists(ix);
    MK_TRY(upload_offsets(ix, s));
    ix->trained = true;
    return MK_OK;
}

mk_status add(mk_ivfpq* ix, const float* xb, int64_t nb, hipStream_t s) {
    const int32_t d = ix->d, nlist = ix->nlist, M = ix->M;
    if (nb == 0) return MK_OK;
    Scratch list, res, bcodes, cnt, tot, oldoff, newoff;
    MK_TRY(list.alloc(sizeof(int64_t) * nb, s));
    MK_TRY(res.alloc(sizeof(float) * nb * d, s));
    MK_TRY(bcodes.alloc((size_t)nb * M, s));
    MK_TRY(kmeans_assign(xb, nb, d, ix->coarse, nlist, list.as<int64_t>(), nullptr, s));
    hipLaunchKernelGGL(residual_kernel, dim3(grid_of(nb * d)), dim3(kBlock), 0, s, xb, nb, d,
                       ix->coarse, list.as<int64_t>(), res.as<float>());
    MK_LAUNCHED();
    MK_TRY(pq_encode(res.as<float>(), nb, d, M, ix->books, bcodes.as<uint8_t>(), s));
    // per-chunk, per-list counts of the batch, their prefix over chunks and
    // the per-list totals
    const int64_t nchunks = ceil_div(nb, kPlaceChunk);
    MK_TRY(cnt.alloc(sizeof(unsigned int) * (size_t)nchunks * nlist, s));
    MK_TRY(tot.alloc(sizeof(unsigned long long) * nlist, s));
    hipLaunchKernelGGL(fill_u32_kernel, dim3(grid_of(nchunks * nlist)), dim3(kBlock), 0, s,
                       cnt.as<unsigned int>(), nchunks * nlist);
    MK_LAUNCHED();
    hipLaunchKernelGGL(place_count_kernel, dim3((unsigned)nchunks), dim3(64), 0, s,
                       list.as<int64_t>(), nb, nlist, cnt.as<unsigned int>());
    MK_LAUNCHED();
    hipLaunchKernelGGL(place_prefix_kernel, dim3(grid_of(nlist)), dim3(kBlock), 0, s,
                       cnt.as<unsigned int>(), nchunks, nlist, tot.as<unsigned long long>());
    MK_LAUNCHED();
    std::vector<unsigned long long> hc(nlist);
    MK_HIP(hipMemcpyAsync(hc.data(), tot.ptr, sizeof(unsigned long long) * nlist,
                          hipMemcpyDeviceToHost, s));
    MK_HIP(hipStreamSynchronize(s));
    // new CSR offsets (host bookkeeping of nlist + 1 integers)
    std::vector<int64_t> no(nlist + 1, 0);
    for (int32_t L = 0; L < nlist; ++L)
        no[L + 1] = no[L] + (ix->offsets[L + 1] - ix->offsets[L]) + (int64_t)hc[L];
    const int64_t total = no[nlist];
    MK_REQUIRE(total < (1ll << 32) - 1, MK_ERR_UNSUPPORTED, "an index holds fewer than 2^32 - 1 vectors");
    uint8_t* ncodes = nullptr;
    int64_t* nids = nullptr;
    MK_TRY(alloc_dev(ncodes, (size_t)total * M));
    MK_TRY(alloc_dev(nids, (size_t)total));
    MK_TRY(oldoff.alloc(sizeof(int64_t) * (nlist + 1), s));
    MK_TRY(newoff.alloc(sizeof(int64_t) * (nlist + 1), s));
    MK_HIP(hipMemcpyAsync(oldoff.ptr, ix->offsets.data(), sizeof(int64_t) * (nlist + 1),
                          hipMemcpyHostToDevice, s));
    MK_HIP(hipMemcpyAsync(newoff.ptr, no.data(), sizeof(int64_t) * (nlist + 1),
                          hipMemcpyHostToDevice, s));
    if (ix->ntotal > 0) {
        hipLaunchKernelGGL(move_old_kernel, dim3(nlist), dim3(kBlock), 0, s, oldoff.as<int64_t>(),
                           newoff.as<int64_t>(), M, ix->codes, ix->ids, ncodes, nids);
        MK_LAUNCHED();
    }
    hipLaunchKernelGGL(place_new_kernel, dim3((unsigned)nchunks), dim3(64), 0, s,
                       list.as<int64_t>(), nb, nlist, cnt.as<unsigned int>(),
                       newoff.as<int64_t>(), oldoff.as<int64_t>(), M, bcodes.as<uint8_t>(),
                       ix->ntotal, ncodes, nids);
    MK_LAUNCHED();
    MK_HIP(hipStreamSynchronize(s));
    free_dev(reinterpret_cast<void*&>(ix->codes));
    free_dev(reinterpret_cast<void*&>(ix->ids));
    ix->codes = ncodes;
    ix->ids = nids;
    ix->capacity = total;
    ix->ntotal = total;
    ix->offsets = no;
    MK_TRY(upload_offsets(ix, s));
    // per-entry term 1 of Eq. 11 for the new list layout
    free_dev(reinterpret_cast<void*&>(ix->t1e));
    MK_TRY(alloc_dev(ix->t1e, (size_t)total));
    hipLaunchKernelGGL(entry_term1_kernel, dim3(nlist), dim3(kBlock), 0, s, ix->offsets_dev, M,
                       ix->codes, ix->term1, ix->t1e);
    MK_LAUNCHED();
    MK_HIP(hipStreamSynchronize(s));
    return MK_OK;
}

// Steps shared by the fixed-probe searches: the probe set and term 2 by exact
// search over the coarse centroids (Eq. 5), term 3 per query, and the list
// scan into `part` = per query `ngroups` partial lists of kk keys.
mk_status scan_fixed(mk_ivfpq* ix, const float* xq, int64_t nq, int32_t nprobe, int32_t kk,
                     Scratch& part, int64_t* ngroups, hipStream_t s, int64_t excl_base = -1) {
    const int32_t M = ix->M;
    Scratch cd, ci, t3;
    MK_TRY(cd.alloc(sizeof(float) * nq * nprobe, s));
    MK_TRY(ci.alloc(sizeof(int64_t) * nq * nprobe, s));
    MK_TRY(t3.alloc(sizeof(float) * nq * M * 256, s));
    const int32_t G = scan_group_of(ix, nq, nprobe, nprobe, kk);
    *ngroups = ceil_div(nprobe, G);
    MK_TRY(part.alloc(sizeof(uint64_t) * nq * *ngroups * kk, s));
    // (the tables' memory is free until they are built)
    const Lend lend{t3.ptr, sizeof(float) * (size_t)nq * M * 256};
    MK_TRY(knn_search(xq, nq, ix->coarse, ix->coarse_norms, ix->nlist, ix->d, nprobe,
                      MK_METRIC_L2, cd.as<float>(), ci.as<int64_t>(), s, nullptr, &lend));
    {
        ProfScope prof("ivf_term3", s);
        MK_TRY(launch_term3(xq, nq, M, ix->dsub, ix->books, t3.as<float>(), s));
    }
    return launch_scan(t3.as<float>(), ix->t1e, cd.as<float>(), ci.as<int64_t>(), nprobe,
                       ix->offsets_dev, ix->codes, ix->ids, M, nq, G, kk, part.as<uint64_t>(),
                       nq * *ngroups, s, nullptr, nullptr, excl_base, ix->lut16);
}

mk_status search(mk_ivfpq* ix, const float* xq, int64_t nq, int32_t k, int32_t nprobe, float* D,
                 int64_t* I, hipStream_t s, int64_t excl_base = -1) {
    Scratch part;
    int64_t ng = 0;
    MK_TRY(scan_fixed(ix, xq, nq, nprobe, k, part, &ng, s, excl_base));
    ProfScope prof("ivf_merge", s);
    return merge_key_lists(part.as<uint64_t>(), nq, (int32_t)ng, k, D, I, s);
}

// IVFADC short list of R entries per query, then exact re-ranking of that
// list against the full-precision database rows (row id of xb = vector id).
mk_status search_rerank(mk_ivfpq* ix, const float* xq, int64_t nq, int32_t k, int32_t nprobe,
                        int32_t R, const float* xb, float* D, int64_t* I, hipStream_t s,
                        int64_t excl_base = -1) {
    Scratch part, keys;
    int64_t ng = 0;
    MK_TRY(scan_fixed(ix, xq, nq, nprobe, R, part, &ng, s, excl_base));
    if (ng == 1)  // the scan's list is the short list
        return rerank_keys(part.as<uint64_t>(), nq, R, xq, xb, ix->d, true, k, D, I, s, R);
    MK_TRY(keys.alloc(sizeof(uint64_t) * nq * 64 * queue_regs(R), s));
    {
        ProfScope prof("ivf_merge", s);
        MK_TRY(merge_key_lists(part.as<uint64_t>(), nq, (int32_t)ng, R, nullptr, nullptr, s,
                               keys.as<uint64_t>()));
    }
    return rerank_keys(keys.as<uint64_t>(), nq, R, xq, xb, ix->d, true, k, D, I, s);
}

mk_status probe_features(const mk_ivfpq* ix, const float* xq, int64_t nq, float* F,
                         hipStream_t s) {
    Scratch cd, ci;
    MK_TRY(cd.alloc(sizeof(float) * nq * kProbeDists, s));
    MK_TRY(ci.alloc(sizeof(int64_t) * nq * kProbeDists, s));
    MK_TRY(knn_search(xq, nq, ix->coarse, ix->coarse_norms, ix->nlist, ix->d, kProbeDists,
                      MK_METRIC_L2, cd.as<float>(), ci.as<int64_t>(), s));
    hipLaunchKernelGGL(probe_features_kernel,
                       dim3(grid_of(nq * (ix->d + kProbeDists))), dim3(kBlock), 0, s, xq, nq,
                       ix->d, cd.as<float>(), kProbeDists, F);
    MK_LAUNCHED();
    return MK_OK;
}

mk_status probe_labels(const mk_ivfpq* ix, const float* xq, int64_t nq, const int64_t* nn,
                       int32_t cap, float* target, int32_t* label, hipStream_t s) {
    Scratch cd, ci, lof;
    MK_TRY(cd.alloc(sizeof(float) * nq * cap, s));
    MK_TRY(ci.alloc(sizeof(int64_t) * nq * cap, s));
    MK_TRY(lof.alloc(sizeof(int32_t) * (ix->ntotal > 0 ? ix->ntotal : 1), s));
    MK_TRY(knn_search(xq, nq, ix->coarse, ix->coarse_norms, ix->nlist, ix->d, cap, MK_METRIC_L2,
                      cd.as<float>(), ci.as<int64_t>(), s));
    hipLaunchKernelGGL(list_of_kernel, dim3(ix->nlist), dim3(kBlock), 0, s, ix->offsets_dev,
                       ix->nlist, ix->ids, lof.as<int32_t>());
    MK_LAUNCHED();
    hipLaunchKernelGGL(probe_labels_kernel, dim3(grid_of(nq)), dim3(kBlock), 0, s,
                       ci.as<int64_t>(), cap, nq, nn, lof.as<int32_t>(), ix->ntotal, cap, target,
                       label);
    MK_LAUNCHED();
    return MK_OK;
}

// IVFADC search with a per-query probe count predicted by the network from
// the query and its coarse distances; R > 0 adds the exact re-rank of an
// R-entry short list against xb.
mk_status search_learned(mk_ivfpq* ix, const mk_mlp* net, float delta, const float* xq,
                         int64_t nq, int32_t k, int32_t cap, int32_t R, const float* xb,
                         float* D, int64_t* I, int32_t* used, hipStream_t s) {
    const int32_t M = ix->M;
    const int32_t kk = R > 0 ? R : k;
    Scratch cd, ci, F, yhat, tau, work, t3, part, keys;
    MK_TRY(cd.alloc(sizeof(float) * nq * cap, s));
    MK_TRY(ci.alloc(sizeof(int64_t) * nq * cap, s));
    MK_TRY(F.alloc(sizeof(float) * nq * (ix->d + kProbeDists), s));
    MK_TRY(yhat.alloc(sizeof(float) * nq, s));
    MK_TRY(tau.alloc(sizeof(int32_t) * nq, s));
    MK_TRY(work.alloc(sizeof(int64_t) * (nq + 1), s));
    // coarse order up to cap probes; its first kProbeDists distances are the
    // network's distance features (the tables' memory is free until they are
    // built)
    MK_TRY(t3.alloc(sizeof(float) * nq * M * 256, s));
    const Lend lend{t3.ptr, sizeof(float) * (size_t)nq * M * 256};
    MK_TRY(knn_search(xq, nq, ix->coarse, ix->coarse_norms, ix->nlist, ix->d, cap, MK_METRIC_L2,
                      cd.as<float>(), ci.as<int64_t>(), s, nullptr, &lend));
    hipLaunchKernelGGL(probe_features_kernel,
                       dim3(grid_of(nq * (ix->d + kProbeDists))), dim3(kBlock), 0, s, xq, nq,
                       ix->d, cd.as<float>(), cap, F.as<float>());
    MK_LAUNCHED();
    {
        ProfScope prof("mlp_forward", s);
        MK_TRY(mlp_forward_dev(net, F.as<float>(), nq, yhat.as<float>(), s));
    }
    // probe counts and the scan's work plan on the device: the scan grid is
    // sized for tau = cap everywhere and the surplus workgroups return at
    // once, so the search never waits for the host
    const int32_t G = scan_group_of(ix, nq, cap, cap < 8 ? cap : 8, kk);
    const int64_t max_items = nq * ceil_div(cap, G);
    hipLaunchKernelGGL(probe_plan_kernel, dim3(1), dim3(1024), 0, s, yhat.as<float>(), nq, delta,
                       cap, G, tau.as<int32_t>(), used, work.as<int64_t>());
    MK_LAUNCHED();
    MK_TRY(part.alloc(sizeof(uint64_t) * max_items * kk, s));
    {
        ProfScope prof("ivf_term3", s);
        MK_TRY(launch_term3(xq, nq, M, ix->dsub, ix->books, t3.as<float>(), s));
    }
    MK_TRY(launch_scan(t3.as<float>(), ix->t1e, cd.as<float>(), ci.as<int64_t>(), cap,
                       ix->offsets_dev, ix->codes, ix->ids, M, nq, G, kk, part.as<uint64_t>(),
                       max_items, s, work.as<int64_t>(), tau.as<int32_t>(), -1, ix->lut16));
    if (R <= 0) {
        ProfScope prof("ivf_merge", s);
        return merge_key_lists(part.as<uint64_t>(), nq, 0, k, D, I, s, nullptr,
                               work.as<int64_t>());
    }
    MK_TRY(keys.alloc(sizeof(uint64_t) * nq * 64 * queue_regs(R), s));
    {
        ProfScope prof("ivf_merge", s);
        MK_TRY(merge_key_lists(part.as<uint64_t>(), nq, 0, R, nullptr, nullptr, s,
                               keys.as<uint64_t>(), work.as<int64_t>()));
    }
    return rerank_keys(keys.as<uint64_t>(), nq, R, xq, xb, ix->d, true, k, D, I, s);
}

}  // namespace

}  // namespace mk

// ---------------------------------------------------------------- C ABI
extern "C" mk_status mk_kmeans_assign(const float* x, int64_t n, int32_t d, const float* c,
                                      int32_t K, int64_t* assign, float* dist,
                                      mk_stream_t stream) {
    MK_REQUIRE(n >= 0 && d >= 1 && K >= 1, MK_ERR_INVALID_ARG, "need n >= 0, d >= 1, K >= 1");
    if (n == 0) return MK_OK;
    MK_REQUIRE(x && c && assign, MK_ERR_INVALID_ARG, "null pointer");
    return mk::kmeans_assign(x, n, d, c, K, assign, dist, static_cast<hipStream_t>(stream));
}

extern "C" mk_status mk_kmeans_update(const float* x, int64_t n, int32_t d, const int64_t* assign,
                                      int32_t K, float* c, int64_t* counts, mk_stream_t stream) {
    MK_REQUIRE(n >= 0 && d >= 1 && K >= 1, MK_ERR_INVALID_ARG, "need n >= 0, d >= 1, K >= 1");
    MK_REQUIRE(c && (n == 0 || (x && assign)), MK_ERR_INVALID_ARG, "null pointer");
    return mk::kmeans_update(x, n, d, assign, K, c, counts, static_cast<hipStream_t>(stream));
}

extern "C" mk_status mk_pq_encode(const float* r, int64_t n, int32_t d, int32_t M,
                                  const float* codebooks, uint8_t* codes, mk_stream_t stream) {
    MK_REQUIRE(n >= 0 && d >= 1 && M >= 1 && d % M == 0 && d / M <= 64, MK_ERR_INVALID_ARG,
               "need d % M == 0 and d / M <= 64");
    if (n == 0) return MK_OK;
    MK_REQUIRE(r && codebooks && codes, MK_ERR_INVALID_ARG, "null pointer");
    return mk::pq_encode(r, n, d, M, codebooks, codes, static_cast<hipStream_t>(stream));
}

extern "C" mk_status mk_ivfpq_create(int32_t d, int32_t nlist, int32_t M, mk_ivfpq** out) {
    MK_REQUIRE(out, MK_ERR_INVALID_ARG, "null output pointer");
    MK_REQUIRE(d >= 1 && d <= 256, MK_ERR_UNSUPPORTED, "d must be in [1, 256]");
    MK_REQUIRE(nlist >= 1 && nlist <= (1 << 24), MK_ERR_INVALID_ARG, "nlist must be in [1, 2^24]");
    MK_REQUIRE(M >= 4 && M <= 128 && M % 4 == 0, MK_ERR_UNSUPPORTED,
               "M must be a multiple of 4 in [4, 128]");
    MK_REQUIRE(d % M == 0, MK_ERR_INVALID_ARG, "d must be a multiple of M");
    mk_ivfpq* ix = new (std::nothrow) mk_ivfpq();
    MK_REQUIRE(ix, MK_ERR_OOM, "host allocation failed");
    ix->d = d;
    ix->nlist = nlist;
    ix->M = M;
    ix->dsub = d / M;
    ix->offsets.assign(nlist + 1, 0);
    *out = ix;
    return MK_OK;
}

extern "C" void mk_ivfpq_destroy(mk_ivfpq* ix) {
    if (!ix) return;
    mk::free_dev(reinterpret_cast<void*&>(ix->coarse));
    mk::free_dev(reinterpret_cast<void*&>(ix->coarse_norms));
    mk::free_dev(reinterpret_cast<void*&>(ix->books));
    mk::free_dev(reinterpret_cast<void*&>(ix->term1));
    mk::free_dev(reinterpret_cast<void*&>(ix->codes));
    mk::free_dev(reinterpret_cast<void*&>(ix->ids));
    mk::free_dev(reinterpret_cast<void*&>(ix->t1e));
    mk::free_dev(reinterpret_cast<void*&>(ix->offsets_dev));
    delete ix;
}

extern "C" mk_status mk_ivfpq_train(mk_ivfpq* ix, const float* xt, int64_t nt, int32_t niter,
                                    const int64_t* coarse_init_rows, const int64_t* pq_init_rows,
                                    mk_stream_t stream) {
    MK_REQUIRE(ix && xt && coarse_init_rows && pq_init_rows, MK_ERR_INVALID_ARG, "null pointer");
    MK_REQUIRE(nt >= ix->nlist && nt >= 256, MK_ERR_INVALID_ARG, "need nt >= nlist and nt >= 256");
    MK_REQUIRE(niter >= 0, MK_ERR_INVALID_ARG, "niter must be >= 0");
    MK_REQUIRE(nt < (1ll << 31), MK_ERR_UNSUPPORTED, "nt must be < 2^31");
    for (int32_t i = 0; i < ix->nlist; ++i)
        MK_REQUIRE(coarse_init_rows[i] >= 0 && coarse_init_rows[i] < nt, MK_ERR_INVALID_ARG,
                   "coarse init row out of range");
    for (int64_t i = 0; i < (int64_t)ix->M * 256; ++i)
        MK_REQUIRE(pq_init_rows[i] >= 0 && pq_init_rows[i] < nt, MK_ERR_INVALID_ARG,
                   "PQ init row out of range");
    return mk::train(ix, xt, nt, niter, coarse_init_rows, pq_init_rows,
                     static_cast<hipStream_t>(stream));
}

extern "C" mk_status mk_ivfpq_add(mk_ivfpq* ix, const float* xb, int64_t nb, mk_stream_t stream) {
    MK_REQUIRE(ix, MK_ERR_INVALID_ARG, "null index");
    MK_REQUIRE(ix->trained, MK_ERR_STATE, "index is not trained");
    MK_REQUIRE(nb >= 0, MK_ERR_INVALID_ARG, "nb must be >= 0");
    MK_REQUIRE(nb == 0 || xb, MK_ERR_INVALID_ARG, "null pointer");
    MK_REQUIRE(ix->ntotal + nb < 0xFFFFFFFFll, MK_ERR_UNSUPPORTED,
               "an index holds fewer than 2^32 - 1 vectors");
    return mk::add(ix, xb, nb, static_cast<hipStream_t>(stream));
}

extern "C" int64_t mk_ivfpq_ntotal(const mk_ivfpq* ix) { return ix ? ix->ntotal : 0; }

extern "C" mk_status mk_ivfpq_search(mk_ivfpq* ix, const float* xq, int64_t nq, int32_t k,
                                     int32_t nprobe, float* D, int64_t* I, mk_stream_t stream) {
    MK_REQUIRE(ix, MK_ERR_INVALID_ARG, "null index");
    MK_REQUIRE(ix->trained, MK_ERR_STATE, "index is not trained");
    MK_REQUIRE(nq >= 0, MK_ERR_INVALID_ARG, "nq must be >= 0");
    MK_REQUIRE(k >= 1, MK_ERR_INVALID_ARG, "k must be >= 1");
    MK_REQUIRE(k <= mk::kMaxK, MK_ERR_UNSUPPORTED, "k must be <= 1024");
    MK_REQUIRE(nprobe >= 1 && nprobe <= ix->nlist && nprobe <= mk::kMaxK, MK_ERR_INVALID_ARG,
               "need 1 <= nprobe <= min(nlist, 1024)");
    if (nq == 0) return MK_OK;
    MK_REQUIRE(xq && D && I, MK_ERR_INVALID_ARG, "null pointer");
    return mk::search(ix, xq, nq, k, nprobe, D, I, static_cast<hipStream_t>(stream));
}

extern "C" mk_status mk_ivfpq_knn_graph(mk_ivfpq* ix, const float* xb, int64_t node0,
                                        int64_t nnodes, int32_t k, int32_t nprobe, int32_t R,
                                        float* D, int64_t* I, mk_stream_t stream) {
    MK_REQUIRE(ix, MK_ERR_INVALID_ARG, "null index");
    MK_REQUIRE(ix->trained, MK_ERR_STATE, "index is not trained");
    MK_REQUIRE(node0 >= 0 && nnodes >= 0 && node0 + nnodes <= ix->ntotal, MK_ERR_INVALID_ARG,
               "nodes node0 .. node0 + nnodes - 1 must be ids of added vectors");
    MK_REQUIRE(k >= 1, MK_ERR_INVALID_ARG, "k must be >= 1");
    MK_REQUIRE(k <= mk::kMaxK, MK_ERR_UNSUPPORTED, "k must be <= 1024");
    MK_REQUIRE(nprobe >= 1 && nprobe <= ix->nlist && nprobe <= mk::kMaxK, MK_ERR_INVALID_ARG,
               "need 1 <= nprobe <= min(nlist, 1024)");
    MK_REQUIRE(R == 0 || (R >= k && R <= mk::kMaxK), MK_ERR_INVALID_ARG,
               "R must be 0 (no re-rank) or in [k, 1024]");
    if (nnodes == 0) return MK_OK;
    MK_REQUIRE(xb && D && I, MK_ERR_INVALID_ARG, "null pointer");
    const hipStream_t s = static_cast<hipStream_t>(stream);
    // batches bound the scratch (coarse results, term 3, partial lists)
    constexpr int64_t kBatch = 32768;
    for (int64_t b = 0; b < nnodes; b += kBatch) {
        const int64_t n = nnodes - b < kBatch ? nnodes - b : kBatch;
        const int64_t first = node0 + b;
        const float* xq = xb + first * ix->d;
        if (R > 0)
            MK_TRY(mk::search_rerank(ix, xq, n, k, nprobe, R, xb, D + b * k, I + b * k, s, first));
        else
            MK_TRY(mk::search(ix, xq, n, k, nprobe, D + b * k, I + b * k, s, first));
    }
    return MK_OK;
}

extern "C" mk_status mk_ivfpq_search_rerank(mk_ivfpq* ix, const float* xq, int64_t nq,
                                            int32_t k, int32_t nprobe, int32_t R,
                                            const float* xb, int64_t nb, float* D, int64_t* I,
                                            mk_stream_t stream) {
    MK_REQUIRE(ix, MK_ERR_INVALID_ARG, "null index");
    MK_REQUIRE(ix->trained, MK_ERR_STATE, "index is not trained");
    MK_REQUIRE(nq >= 0, MK_ERR_INVALID_ARG, "nq must be >= 0");
    MK_REQUIRE(k >= 1 && k <= R, MK_ERR_INVALID_ARG, "need 1 <= k <= R");
    MK_REQUIRE(R <= mk::kMaxK, MK_ERR_UNSUPPORTED, "R must be <= 1024");
    MK_REQUIRE(nprobe >= 1 && nprobe <= ix->nlist && nprobe <= mk::kMaxK, MK_ERR_INVALID_ARG,
               "need 1 <= nprobe <= min(nlist, 1024)");
    MK_REQUIRE(nb >= ix->ntotal, MK_ERR_INVALID_ARG,
               "the database must hold a row for every added id");
    if (nq == 0) return MK_OK;
    MK_REQUIRE(xq && D && I && (xb || nb == 0), MK_ERR_INVALID_ARG, "null pointer");
    return mk::search_rerank(ix, xq, nq, k, nprobe, R, xb, D, I,
                             static_cast<hipStream_t>(stream));
}

extern "C" mk_status mk_ivfpq_probe_features(const mk_ivfpq* ix, const float* xq, int64_t nq,
                                             float* F, mk_stream_t stream) {
    MK_REQUIRE(ix, MK_ERR_INVALID_ARG, "null index");
    MK_REQUIRE(ix->trained, MK_ERR_STATE, "index is not trained");
    MK_REQUIRE(ix->nlist >= mk::kProbeDists, MK_ERR_UNSUPPORTED, "needs nlist >= 32");
    MK_REQUIRE(nq >= 0, MK_ERR_INVALID_ARG, "nq must be >= 0");
    if (nq == 0) return MK_OK;
    MK_REQUIRE(xq && F, MK_ERR_INVALID_ARG, "null pointer");
    return mk::probe_features(ix, xq, nq, F, static_cast<hipStream_t>(stream));
}

extern "C" mk_status mk_ivfpq_probe_labels(const mk_ivfpq* ix, const float* xq, int64_t nq,
                                           const int64_t* nn_ids, int32_t cap, float* target,
                                           int32_t* label, mk_stream_t stream) {
    MK_REQUIRE(ix, MK_ERR_INVALID_ARG, "null index");
    MK_REQUIRE(ix->trained, MK_ERR_STATE, "index is not trained");
    MK_REQUIRE(nq >= 0, MK_ERR_INVALID_ARG, "nq must be >= 0");
    MK_REQUIRE(cap >= 1 && cap <= ix->nlist && cap <= mk::kMaxK, MK_ERR_INVALID_ARG,
               "need 1 <= cap <= min(nlist, 1024)");
    if (nq == 0) return MK_OK;
    MK_REQUIRE(xq && nn_ids && target, MK_ERR_INVALID_ARG, "null pointer");
    return mk::probe_labels(ix, xq, nq, nn_ids, cap, target, label,
                            static_cast<hipStream_t>(stream));
}

extern "C" mk_status mk_ivfpq_search_learned(mk_ivfpq* ix, const mk_mlp* net, float delta,
                                             const float* xq, int64_t nq, int32_t k, int32_t cap,
                                             int32_t R, const float* xb, int64_t nb, float* D,
                                             int64_t* I, int32_t* nprobe_used,
                                             mk_stream_t stream) {
    MK_REQUIRE(ix && net, MK_ERR_INVALID_ARG, "null index or network");
    MK_REQUIRE(ix->trained, MK_ERR_STATE, "index is not trained");
    MK_REQUIRE(mk::mlp_inputs(net) == ix->d + mk::kProbeDists, MK_ERR_INVALID_ARG,
               "network inputs must be d + 32");
    MK_REQUIRE(nq >= 0, MK_ERR_INVALID_ARG, "nq must be >= 0");
    MK_REQUIRE(k >= 1, MK_ERR_INVALID_ARG, "k must be >= 1");
    MK_REQUIRE(k <= mk::kMaxK && R <= mk::kMaxK, MK_ERR_UNSUPPORTED, "k and R must be <= 1024");
    MK_REQUIRE(cap >= mk::kProbeDists && cap <= ix->nlist && cap <= mk::kMaxK,
               MK_ERR_INVALID_ARG, "need 32 <= cap <= min(nlist, 1024)");
    MK_REQUIRE(R <= 0 || R >= k, MK_ERR_INVALID_ARG, "need R >= k for the re-rank");
    MK_REQUIRE(R <= 0 || (xb && nb >= ix->ntotal), MK_ERR_INVALID_ARG,
               "the re-rank needs a database row for every added id");
    if (nq == 0) return MK_OK;
    MK_REQUIRE(xq && D && I, MK_ERR_INVALID_ARG, "null pointer");
    return mk::search_learned(ix, net, delta, xq, nq, k, cap, R, xb, D, I, nprobe_used,
                              static_cast<hipStream_t>(stream));
}

extern "C" mk_status mk_ivfpq_set_scan_options(mk_ivfpq* ix, mk_precision lut_precision,
                                               int32_t lists_per_group) {
    MK_REQUIRE(ix, MK_ERR_INVALID_ARG, "null index");
    MK_REQUIRE(lut_precision == MK_PREC_FP32 || lut_precision == MK_PREC_FP16, MK_ERR_UNSUPPORTED,
               "lookup tables are FP32 or FP16");
    MK_REQUIRE(lists_per_group >= -1 && lists_per_group <= mk::kMaxK, MK_ERR_INVALID_ARG,
               "lists_per_group must be -1, 0 or a count up to 1024");
    ix->lut16 = lut_precision == MK_PREC_FP16;
    ix->lists_per_group = lists_per_group;
    return MK_OK;
}

extern "C" int32_t mk_ivfpq_dim(const mk_ivfpq* ix) { return ix ? ix->d : 0; }

extern "C" mk_status mk_ivfpq_shape(const mk_ivfpq* ix, int32_t* d, int32_t* nlist, int32_t* M) {
    MK_REQUIRE(ix, MK_ERR_INVALID_ARG, "null index");
    if (d) *d = ix->d;
    if (nlist) *nlist = ix->nlist;
    if (M) *M = ix->M;
    return MK_OK;
}

extern "C" mk_status mk_ivfpq_search_workspace_bytes(const mk_ivfpq* ix, int64_t nq, int32_t k,
                                                     int32_t nprobe, int32_t R, size_t* bytes) {
    MK_REQUIRE(ix && bytes, MK_ERR_INVALID_ARG, "null pointer");
    MK_REQUIRE(nq >= 0 && k >= 1 && nprobe >= 1, MK_ERR_INVALID_ARG, "bad sizes");
    const int64_t kk = R > 0 ? R : k;
    const int64_t qn = nq;
    // coarse search: results, and at most min(16, nlist / (8 * queue)) chunk
    // lists (the exact search's chunk plan)
    const int64_t ks = 64 * (int64_t)mk::queue_regs(std::min(nprobe + 16, mk::kMaxK));
    const int64_t chunks = std::min<int64_t>(16, std::max<int64_t>(1, ix->nlist / (8 * ks)));
    int64_t b = qn * nprobe * (4 + 8) + qn * chunks * ks * 8 + qn * 4;
    b += qn * (int64_t)ix->M * 256 * 4;      // term-3 tables
    b += qn * nprobe * kk * 8;                // per-list partial results
    if (R > 0) b += qn * 64 * (int64_t)mk::queue_regs(R) * 8;  // short lists
    b += qn * (ix->d + mk::kProbeDists) * 4 + qn * 16;          // learned-count features
    *bytes = (size_t)b;
    return MK_OK;
}

extern "C" mk_status mk_ivfpq_get_quantizers(const mk_ivfpq* ix, float* coarse, float* codebooks) {
    MK_REQUIRE(ix, MK_ERR_INVALID_ARG, "null index");
    MK_REQUIRE(ix->trained, MK_ERR_STATE, "index is not trained");
    MK_HIP(hipDeviceSynchronize());
    if (coarse)
        MK_HIP(hipMemcpy(coarse, ix->coarse, sizeof(float) * (size_t)ix->nlist * ix->d,
                         hipMemcpyDeviceToHost));
    if (codebooks)
        MK_HIP(hipMemcpy(codebooks, ix->books, sizeof(float) * (size_t)ix->M * 256 * ix->dsub,
                         hipMemcpyDeviceToHost));
    return MK_OK;
}

extern "C" mk_status mk_ivfpq_set_quantizers(mk_ivfpq* ix, const float* coarse,
                                             const float* codebooks, mk_stream_t stream) {
    MK_REQUIRE(ix && coarse && codebooks, MK_ERR_INVALID_ARG, "null pointer");
    hipStream_t s = static_cast<hipStream_t>(stream);
    {
        mk_status st = mk::alloc_quantizers(ix);
        if (st != MK_OK) return st;
    }
    MK_HIP(hipMemcpyAsync(ix->coarse, coarse, sizeof(float) * (size_t)ix->nlist * ix->d,
                          hipMemcpyHostToDevice, s));
    MK_HIP(hipMemcpyAsync(ix->books, codebooks, sizeof(float) * (size_t)ix->M * 256 * ix->dsub,
                          hipMemcpyHostToDevice, s));
    mk_status st = mk::build_term1(ix, s);
    if (st != MK_OK) return st;
    mk::reset_lists(ix);
    st = mk::upload_offsets(ix, s);
    if (st != MK_OK) return st;
    ix->trained = true;
    return MK_OK;
}

extern "C" mk_status mk_ivfpq_get_lists(const mk_ivfpq* ix, int64_t* offsets, uint8_t* codes,
                                        int64_t* ids) {
    MK_REQUIRE(ix, MK_ERR_INVALID_ARG, "null index");
    MK_HIP(hipDeviceSynchronize());
    if (offsets) std::memcpy(offsets, ix->offsets.data(), sizeof(int64_t) * (ix->nlist + 1));
    if (codes && ix->ntotal)
        MK_HIP(hipMemcpy(codes, ix->codes, (size_t)ix->ntotal * ix->M, hipMemcpyDeviceToHost));
    if (ids && ix->ntotal)
        MK_HIP(hipMemcpy(ids, ix->ids, sizeof(int64_t) * ix->ntotal, hipMemcpyDeviceToHost));
    return MK_OK;
}

// ---------------------------------------------------------------- save / load
namespace mk {
namespace {
constexpr char kIndexMagic[8] = {'M', 'K', 'I', 'V', 'F', 'P', 'Q', '\0'};
constexpr uint32_t kIndexVersion = 1;

// Fills a freshly created index from the body of an index file (after the
// header) and rebuilds the derived tables with the same kernels as
// train/add, so searches after a load equal searches before the save.
mk_status load_body(mk_ivfpq* ix, BinFile& f, int64_t ntotal, hipStream_t s) {
    const int32_t nlist = ix->nlist, M = ix->M;
    MK_TRY(alloc_quantizers(ix));
    MK_TRY(get_device(f, ix->coarse, sizeof(float) * (size_t)nlist * ix->d));
    MK_TRY(get_device(f, ix->books, sizeof(float) * (size_t)M * 256 * ix->dsub));
    std::vector<int64_t> offs(nlist + 1);
    MK_REQUIRE(f.get(offs.data(), sizeof(int64_t) * offs.size()), MK_ERR_INVALID_ARG,
               f.path + " is truncated");
    MK_REQUIRE(offs[0] == 0 && offs[nlist] == ntotal, MK_ERR_INVALID_ARG,
               f.path + ": list offsets do not span the stored entries");
    for (int32_t L = 0; L < nlist; ++L)
        MK_REQUIRE(offs[L + 1] >= offs[L], MK_ERR_INVALID_ARG, f.path + ": list offsets decrease");
    MK_TRY(alloc_dev(ix->codes, (size_t)ntotal * M));
    MK_TRY(alloc_dev(ix->ids, (size_t)ntotal));
    MK_TRY(get_device(f, ix->codes, (size_t)ntotal * M));
    MK_TRY(get_device(f, ix->ids, sizeof(int64_t) * (size_t)ntotal));
    MK_REQUIRE(f.at_end(), MK_ERR_INVALID_ARG, f.path + " has trailing bytes");
    MK_TRY(build_term1(ix, s));
    ix->offsets = offs;
    ix->ntotal = ntotal;
    ix->capacity = ntotal;
    MK_TRY(upload_offsets(ix, s));
    MK_TRY(alloc_dev(ix->t1e, (size_t)(ntotal > 0 ? ntotal : 1)));
    hipLaunchKernelGGL(entry_term1_kernel, dim3(nlist), dim3(kBlock), 0, s, ix->offsets_dev, M,
                       ix->codes, ix->term1, ix->t1e);
    MK_LAUNCHED();
    MK_HIP(hipStreamSynchronize(s));
    ix->trained = true;
    return MK_OK;
}
}  // namespace
}  // namespace mk

extern "C" mk_status mk_ivfpq_save(const mk_ivfpq* ix, const char* path) {
    MK_REQUIRE(ix && path, MK_ERR_INVALID_ARG, "null pointer");
    MK_REQUIRE(ix->trained, MK_ERR_STATE, "index is not trained");
    MK_HIP(hipDeviceSynchronize());
    mk::BinFile f(path, "wb");
    MK_REQUIRE(f.ok(), MK_ERR_INVALID_ARG, std::string("cannot open ") + path + " for writing");
    const bool head = f.put(mk::kIndexMagic, 8) && f.put_v(mk::kIndexVersion) && f.put_v(ix->d) &&
                      f.put_v(ix->nlist) && f.put_v(ix->M) && f.put_v(ix->ntotal);
    MK_REQUIRE(head, MK_ERR_INVALID_ARG, std::string("write to ") + path + " failed");
    MK_TRY(mk::put_device(f, ix->coarse, sizeof(float) * (size_t)ix->nlist * ix->d));
    MK_TRY(mk::put_device(f, ix->books, sizeof(float) * (size_t)ix->M * 256 * ix->dsub));
    MK_REQUIRE(f.put(ix->offsets.data(), sizeof(int64_t) * (ix->nlist + 1)), MK_ERR_INVALID_ARG,
               std::string("write to ") + path + " failed");
    MK_TRY(mk::put_device(f, ix->codes, (size_t)ix->ntotal * ix->M));
    MK_TRY(mk::put_device(f, ix->ids, sizeof(int64_t) * (size_t)ix->ntotal));
    MK_REQUIRE(f.close(), MK_ERR_INVALID_ARG, std::string("write to ") + path + " failed");
    return MK_OK;
}

extern "C" mk_status mk_ivfpq_load(const char* path, mk_ivfpq** out) {
    MK_REQUIRE(path && out, MK_ERR_INVALID_ARG, "null pointer");
    *out = nullptr;
    mk::BinFile f(path, "rb");
    MK_REQUIRE(f.ok(), MK_ERR_INVALID_ARG, std::string("cannot open ") + path);
    char magic[8];
    uint32_t version = 0;
    int32_t d = 0, nlist = 0, M = 0;
    int64_t ntotal = 0;
    const bool head = f.get(magic, 8) && f.get_v(version) && f.get_v(d) && f.get_v(nlist) &&
                      f.get_v(M) && f.get_v(ntotal);
    MK_REQUIRE(head && std::memcmp(magic, mk::kIndexMagic, 8) == 0, MK_ERR_INVALID_ARG,
               std::string(path) + " is not an IVFPQ index file");
    MK_REQUIRE(version == mk::kIndexVersion, MK_ERR_UNSUPPORTED,
               std::string(path) + ": unknown index file version");
    MK_REQUIRE(ntotal >= 0 && ntotal < 0xFFFFFFFFll, MK_ERR_INVALID_ARG,
               std::string(path) + ": bad entry count");
    mk_ivfpq* ix = nullptr;
    MK_TRY(mk_ivfpq_create(d, nlist, M, &ix));
    const mk_status st = mk::load_body(ix, f, ntotal, nullptr);
    if (st != MK_OK) {
        mk_ivfpq_destroy(ix);
        return st;
    }
    *out = ix;
    return MK_OK;
}
