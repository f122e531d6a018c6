// Row-wise k-selection of a resident matrix (Section 2 problem statement,
// Section 4.2 selection, Section 6.1 benchmark shape) and the generic merge of
// per-segment partial results (the second pass of the two-pass k-selection of
// Section 5.3).
//
// Pass 1 streams each (row, segment) once with 16-byte coalesced loads: k <= 64 (128 for
// short rows) one wave and its sorted register queue, more one workgroup and an unsorted
// LDS pool (pool.hpp).  A row that fits one segment writes its final result directly;
// otherwise its k best keys go to a scratch list and pass 2 (one workgroup per
// row) selects over the segments' keys.
#include <algorithm>

#include "common.hpp"
#include "kselect.hpp"
#include "pool.hpp"
#include "profile.hpp"
#include "wave_select.hpp"

namespace mk {

namespace {

constexpr int kWavesPerBlock = 4;

template <bool LARGEST>
__device__ __forceinline__ uint64_t value_key(float v, uint32_t idx) {
    return make_key(LARGEST ? -v : v, idx);
}

// Write the first k keys of a lane-stride queue as (value, index) pairs.
template <int KR, bool LARGEST>
__device__ __forceinline__ void emit_values(const uint64_t (&w)[KR], int k, float* vals,
                                            int64_t* idx) {
    const int lane = lane_id();
#pragma unroll
    for (int r = 0; r < KR; ++r) {
        const int e = r * 64 + lane;
        if (e < k) {
            const uint64_t key = w[r];
            if (key == kSentinel) {
                vals[e] = LARGEST ? -INFINITY : INFINITY;
                idx[e] = -1;
            } else {
                const float s = key_score(key);
                vals[e] = LARGEST ? -s : s;
                idx[e] = (int64_t)key_index(key);
            }
        }
    }
}

template <int KR>
__device__ __forceinline__ void emit_keys(const uint64_t (&w)[KR], int k, uint64_t* out) {
    const int lane = lane_id();
#pragma unroll
    for (int r = 0; r < KR; ++r) {
        const int e = r * 64 + lane;
        if (e < k) out[e] = w[r];
    }
}

template <int KR, int T, bool LARGEST>
__global__ __launch_bounds__(64 * kWavesPerBlock) void kselect_pass1(
    const float* __restrict__ a, int64_t nrows, int64_t len, int32_t k, int32_t nseg,
    int64_t seg_len, float* __restrict__ vals, int64_t* __restrict__ idx,
    uint64_t* __restrict__ partial) {
    constexpr int U = 4;  // float4 loads in flight per lane
    __shared__ float stage[kWavesPerBlock][4 * U][64];
    const int wave = threadIdx.x / 64;
    const int lane = lane_id();
    const int64_t unit = (int64_t)blockIdx.x * kWavesPerBlock + wave;
    if (unit >= nrows * (int64_t)nseg) return;  // wave-uniform
    const int64_t row = unit / nseg;
    const int64_t seg = unit % nseg;
    const int64_t lo = seg * seg_len;
    const int64_t hi = lo + seg_len < len ? lo + seg_len : len;
    const float* rp = a + row * len;

    WaveSelect<KR, T> ws;
    ws.init(k);

    // Vector body over 16-byte aligned rows: lane takes 4 consecutive values
    // per load, U loads in flight.  Most groups are rejected by one compare
    // per value against the current k-th score; a group with any candidate
    // is staged in LDS and offered value by value from a single loop, so the
    // merge network appears once in the kernel.
    const bool aligned = (reinterpret_cast<uintptr_t>(rp + lo) & 15) == 0;
    const int64_t vec_end = aligned ? lo + ((hi - lo) / (256 * U)) * (256 * U) : lo;
    for (int64_t e = lo; e < vec_end; e += 256 * U) {
        float4 v[U];
#pragma unroll
        for (int u = 0; u < U; ++u)
            v[u] = *reinterpret_cast<const float4*>(rp + e + u * 256 + lane * 4);
        bool cand = false;
#pragma unroll
        for (int u = 0; u < U; ++u) {
            cand |= ws.may_take(LARGEST ? -v[u].x : v[u].x);
            cand |= ws.may_take(LARGEST ? -v[u].y : v[u].y);
            cand |= ws.may_take(LARGEST ? -v[u].z : v[u].z);
            cand |= ws.may_take(LARGEST ? -v[u].w : v[u].w);
        }
        if (__any(cand)) {
#pragma unroll
            for (int u = 0; u < U; ++u) {
                stage[wave][4 * u + 0][lane] = v[u].x;
                stage[wave][4 * u + 1][lane] = v[u].y;
                stage[wave][4 * u + 2][lane] = v[u].z;
                stage[wave][4 * u + 3][lane] = v[u].w;
            }
            __builtin_amdgcn_wave_barrier();
#pragma unroll 1
            for (int j = 0; j < 4 * U; ++j) {
                const float val = stage[wave][j][lane];
                const uint32_t i = (uint32_t)(e + (j >> 2) * 256 + lane * 4 + (j & 3));
                if (ws.push(value_key<LARGEST>(val, i))) ws.merge();
            }
            __builtin_amdgcn_wave_barrier();
        }
    }
    // Scalar remainder (and unaligned rows): one value per lane per step.
#pragma unroll 1
    for (int64_t e = vec_end; e < hi; e += 64) {
        const int64_t i = e + lane;
        const uint64_t key = i < hi ? value_key<LARGEST>(rp[i], (uint32_t)i) : kSentinel;
        if (ws.push(key)) ws.merge();
    }
    ws.finish();
    if (nseg == 1) {
        emit_values<KR, LARGEST>(ws.w, k, vals + row * k, idx + row * k);
    } else {
        emit_keys<KR>(ws.w, k, partial + unit * k);
    }
}

// Pass 1 for k > 64: a workgroup per (row, segment), one candidate pool in LDS
// (pool_values).
//
// 10^4 rows, k = 100 / 300 / 1000, against a wave per row with a sorted queue (or,
// for 300 and more and long rows, a pool in device memory): 128,000 values 896 /
// 960 / 1,251 us (972 / 1,209 / 1,414), 16,000 values 201 / 228 / 367 (238 / 414 /
// 1,049), 1,000 values 56 / 62 / 98 (80 / 158 / 263); 1,000 rows of 128,000, 140 /
// 144 / 202 us (230 / 395 / 830).
template <int P, bool LARGEST>  // k <= P - 2048
__global__ __launch_bounds__(kPoolThreads) void kselect_rows(
    const float* __restrict__ a, int64_t len, int32_t k, int32_t nseg, int64_t seg_len,
    float* __restrict__ vals, int64_t* __restrict__ idx, uint64_t* __restrict__ partial) {
    __shared__ uint64_t pool[P];
    __shared__ uint32_t bins[kCutBins];
    __shared__ PoolState st;
    __shared__ uint32_t ws[2][kPoolWaves];
    const int tid = threadIdx.x;
    const int64_t unit = blockIdx.x;
    const int64_t row = unit / nseg, seg = unit % nseg;
    // (rows are shorter than 2^32: 32-bit places inside the segment)
    const int64_t lo = seg * seg_len;
    const uint32_t n = (uint32_t)(lo + seg_len < len ? seg_len : len - lo);
    const float* rp = a + row * len + lo;
    const uint32_t have = pool_values<P, 2, LARGEST>(rp, n, (uint32_t)lo, k, pool, bins, &st, ws);
    if (nseg > 1) {
        if (have > (uint32_t)k) pool_cut<P>(pool, bins, &st, have, k);
        __syncthreads();
        for (int e = tid; e < k; e += kPoolThreads)
            partial[unit * k + e] = e < (int)have ? pool[e] : kSentinel;
        return;
    }
    float* vr = vals + row * k;
    int64_t* ir = idx + row * k;
    pool_emit<P>(pool, bins, &st, have, (uint32_t)k, [&](uint32_t r, uint64_t key) {
        const float s = key_score(key);
        vr[r] = LARGEST ? -s : s;
        ir[r] = (int64_t)key_index(key);
    });
    for (int e = tid; e < k; e += kPoolThreads)
        if (e >= (int)have) {
            vr[e] = LARGEST ? -INFINITY : INFINITY;
            ir[e] = -1;
        }
}

// Pass 2 for k > 64: the k best of a row's lists of k keys by one workgroup.
template <int P, bool LARGEST>
__global__ __launch_bounds__(kPoolThreads) void kselect_lists(
    const uint64_t* __restrict__ partial, int32_t nseg, int32_t k, float* __restrict__ vals,
    int64_t* __restrict__ idx, uint64_t* __restrict__ keys_out, int32_t out_len,
    const int64_t* __restrict__ seg_offs) {
    __shared__ uint64_t pool[P];
    __shared__ uint32_t bins[kCutBins];
    __shared__ PoolState st;
    const int64_t row = blockIdx.x;
    const int64_t s0 = seg_offs ? seg_offs[row] : row * (int64_t)nseg;
    const int64_t s1 = seg_offs ? seg_offs[row + 1] : s0 + nseg;
    uint64_t limit;
    const uint32_t have = pool_stream<P>(partial + s0 * k, (s1 - s0) * k, pool, bins, &st, k, limit);
    if (keys_out) {
        uint64_t* o = keys_out + row * out_len;
        pool_emit<P>(pool, bins, &st, have, (uint32_t)k, [&](uint32_t r, uint64_t key) { o[r] = key; });
        for (int e = threadIdx.x; e < out_len; e += kPoolThreads)
            if (e >= (int)have) o[e] = kSentinel;
        return;
    }
    float* vr = vals + row * k;
    int64_t* ir = idx + row * k;
    pool_emit<P>(pool, bins, &st, have, (uint32_t)k, [&](uint32_t r, uint64_t key) {
        const float s = key_score(key);
        const bool pad = key == kSentinel;
        vr[r] = pad ? (LARGEST ? -INFINITY : INFINITY) : LARGEST ? -s : s;
        ir[r] = pad ? -1 : (int64_t)key_index(key);
    });
    for (int e = threadIdx.x; e < k; e += kPoolThreads)
        if (e >= (int)have) {
            vr[e] = LARGEST ? -INFINITY : INFINITY;
            ir[e] = -1;
        }
}

// Pass 2: per row, select the k best of nseg * k partial keys (or, with
// seg_offs, of the lists seg_offs[row] .. seg_offs[row + 1] - 1), written as
// (value, index) pairs or, with keys_out, as the 64*KR-entry sorted key list.
template <int KR, int T, bool LARGEST>
__global__ __launch_bounds__(64 * kWavesPerBlock) void kselect_merge(
    const uint64_t* __restrict__ partial, int64_t nrows, int32_t nseg, int32_t k,
    float* __restrict__ vals, int64_t* __restrict__ idx, uint64_t* __restrict__ keys_out,
    const int64_t* __restrict__ seg_offs) {
    const int wave = threadIdx.x / 64;
    const int lane = lane_id();
    const int64_t row = (int64_t)blockIdx.x * kWavesPerBlock + wave;
    if (row >= nrows) return;
    const int64_t s0 = seg_offs ? seg_offs[row] : row * (int64_t)nseg;
    const int64_t s1 = seg_offs ? seg_offs[row + 1] : s0 + nseg;
    const uint64_t* p = partial + s0 * k;
    const int64_t n = (s1 - s0) * k;
    WaveSelect<KR, T> ws;
    ws.init(k);
#pragma unroll 1
    for (int64_t e = 0; e < n; e += 64) {
        const int64_t i = e + lane;
        if (ws.push(i < n ? p[i] : kSentinel)) ws.merge();
    }
    ws.finish();
    if (keys_out)
        emit_keys<KR>(ws.w, 64 * KR, keys_out + row * 64 * KR);
    else
        emit_values<KR, LARGEST>(ws.w, k, vals + row * k, idx + row * k);
}

template <int KR, bool LARGEST>
mk_status kselect_waves(const float* a, int64_t nrows, int64_t len, int32_t k, float* vals,
                        int64_t* idx, hipStream_t stream) {
    constexpr int KS = 64 * KR, T = SelParams<KR>::T;
    // Enough waves to fill the chip, but segments long enough that the
    // partial keys stay a small fraction of the input.
    int64_t want = ceil_div(8192, nrows > 0 ? nrows : 1);
    int64_t max_by_len = len / (int64_t)(16 * KS > 4096 ? 16 * KS : 4096);
    int64_t nseg = want < max_by_len ? want : max_by_len;
    if (nseg < 1) nseg = 1;
    if (nseg > 4096) nseg = 4096;
    int64_t seg_len = ceil_div(ceil_div(len, nseg), 256) * 256;
    nseg = len > 0 ? ceil_div(len, seg_len) : 1;
    if (seg_len == 0) seg_len = 256;

    Scratch part;
    if (nseg > 1) MK_TRY(part.alloc(sizeof(uint64_t) * (size_t)nrows * (size_t)nseg * (size_t)k, stream));
    const int64_t units = nrows * nseg;
    {
        ProfScope prof("kselect_pass1", stream);
        hipLaunchKernelGGL((kselect_pass1<KR, T, LARGEST>),
                           dim3((unsigned)ceil_div(units, kWavesPerBlock)),
                           dim3(64 * kWavesPerBlock), 0, stream, a, nrows, len, k,
                           (int32_t)nseg, seg_len, vals, idx, part.as<uint64_t>());
        MK_LAUNCHED();
    }
    if (nseg > 1) {
        hipLaunchKernelGGL((kselect_merge<KR, T, LARGEST>),
                           dim3((unsigned)ceil_div(nrows, kWavesPerBlock)), dim3(64 * kWavesPerBlock),
                           0, stream, part.as<uint64_t>(), nrows, (int32_t)nseg, k, vals, idx,
                           (uint64_t*)nullptr, (const int64_t*)nullptr);
        MK_LAUNCHED();
    }
    return MK_OK;
}

template <int P, bool LARGEST>
mk_status kselect_pools(const float* a, int64_t nrows, int64_t len, int32_t k, float* vals,
                        int64_t* idx, hipStream_t stream) {
    // segments that give about 1,024 workgroups, of at least 16,384 values and
    // 16 result lists
    int64_t nseg = std::min(ceil_div(1024, nrows), len / std::max<int64_t>(16384, 16 * (int64_t)k));
    if (nseg < 1) nseg = 1;
    int64_t seg_len = ceil_div(ceil_div(len, nseg), 256) * 256;
    if (seg_len == 0) seg_len = 256;
    nseg = len > 0 ? ceil_div(len, seg_len) : 1;
    Scratch part;
    if (nseg > 1) MK_TRY(part.alloc(sizeof(uint64_t) * (size_t)nrows * (size_t)nseg * (size_t)k, stream));
    {
        ProfScope prof("kselect_pass1", stream);
        hipLaunchKernelGGL((kselect_rows<P, LARGEST>), dim3((unsigned)(nrows * nseg)),
                           dim3(kPoolThreads), 0, stream, a, len, k, (int32_t)nseg, seg_len, vals,
                           idx, part.as<uint64_t>());
        MK_LAUNCHED();
    }
    if (nseg > 1) {
        constexpr int PL = P > 2560 ? 4096 : 2048;
        hipLaunchKernelGGL((kselect_lists<PL, LARGEST>), dim3((unsigned)nrows), dim3(kPoolThreads), 0,
                           stream, part.as<uint64_t>(), (int32_t)nseg, k, vals, idx,
                           (uint64_t*)nullptr, 0, (const int64_t*)nullptr);
        MK_LAUNCHED();
    }
    return MK_OK;
}

template <bool LARGEST>
mk_status kselect_dispatch(const float* a, int64_t nrows, int64_t len, int32_t k, float* vals,
                           int64_t* idx, hipStream_t s) {
    // a register queue of 64 costs a wave little; from there on, as a rule, a pool per
    // workgroup (one dimension of a grid: fewer than 2^24 workgroups of 256)
    if (k <= 64) return kselect_waves<1, LARGEST>(a, nrows, len, k, vals, idx, s);
    if (nrows >= (1ll << 23)) {
        const int64_t half = nrows / 2;
        MK_TRY((kselect_dispatch<LARGEST>(a, half, len, k, vals, idx, s)));
        return kselect_dispatch<LARGEST>(a + half * len, nrows - half, len, k, vals + half * k,
                                         idx + half * k, s);
    }
    // (short rows, for which a pool's passes are the larger part: 30,000 rows of 100 / 300 /
    // 500 values, k = 65: 75 / 106 / 124 us by a queue of 128, 122 / 127 / 130 by a pool)
    if (k <= 128 && len <= 512) {
        ProfScope prof("kselect_pass1", s);
        hipLaunchKernelGGL((kselect_pass1<2, SelParams<2>::T, LARGEST>),
                           dim3((unsigned)ceil_div(nrows, kWavesPerBlock)), dim3(64 * kWavesPerBlock),
                           0, s, a, nrows, len, k, 1, (int64_t)512, vals, idx, (uint64_t*)nullptr);
        MK_LAUNCHED();
        return MK_OK;
    }
    return k <= 512 ? kselect_pools<2560, LARGEST>(a, nrows, len, k, vals, idx, s)
                    : kselect_pools<3072, LARGEST>(a, nrows, len, k, vals, idx, s);
}

}  // namespace

mk_status merge_key_lists(const uint64_t* partial, int64_t nrows, int32_t nseg, int32_t k,
                          float* vals, int64_t* idx, hipStream_t s, uint64_t* keys_out,
                          const int64_t* seg_offs, bool largest) {
    if (nrows == 0) return MK_OK;
    MK_REQUIRE(!(largest && keys_out), MK_ERR_INVALID_ARG, "largest-first merges emit values");
    const int32_t out_len = 64 * queue_regs(k);
    if (k <= 64) {
        auto kern = largest ? kselect_merge<1, SelParams<1>::T, true> : kselect_merge<1, SelParams<1>::T, false>;
        hipLaunchKernelGGL(kern, dim3((unsigned)ceil_div(nrows, kWavesPerBlock)),
                           dim3(64 * kWavesPerBlock), 0, s, partial, nrows, nseg, k, vals, idx,
                           keys_out, seg_offs);
        MK_LAUNCHED();
        return MK_OK;
    }
    auto kern = k <= 512 ? (largest ? kselect_lists<2048, true> : kselect_lists<2048, false>)
                         : (largest ? kselect_lists<4096, true> : kselect_lists<4096, false>);
    constexpr int64_t kRows = 1ll << 23;  // (one dimension of a grid)
    for (int64_t r0 = 0; r0 < nrows; r0 += kRows) {
        const int64_t n = std::min(kRows, nrows - r0);
        hipLaunchKernelGGL(kern, dim3((unsigned)n), dim3(kPoolThreads), 0, s,
                           seg_offs ? partial : partial + r0 * nseg * k, nseg, k,
                           vals ? vals + r0 * k : nullptr, idx ? idx + r0 * k : nullptr,
                           keys_out ? keys_out + r0 * out_len : nullptr, out_len,
                           seg_offs ? seg_offs + r0 : nullptr);
        MK_LAUNCHED();
    }
    return MK_OK;
}

mk_status kselect_segments(const float* a, int64_t nrows, int64_t len, int32_t k, int64_t seg_len,
                           uint64_t* partial, hipStream_t s) {
    const int64_t nseg = ceil_div(len, seg_len);
    MK_REQUIRE(nrows * nseg < (1ll << 24), MK_ERR_UNSUPPORTED, "too many segments for one launch");
    auto kern = k <= 512 ? kselect_rows<2560, false> : kselect_rows<3072, false>;
    ProfScope prof("kselect_pass1", s);
    hipLaunchKernelGGL(kern, dim3((unsigned)(nrows * nseg)), dim3(kPoolThreads), 0, s, a, len, k,
                       (int32_t)nseg, seg_len, (float*)nullptr, (int64_t*)nullptr, partial);
    MK_LAUNCHED();
    return MK_OK;
}

}  // namespace mk

extern "C" mk_status mk_kselect(const float* a, int64_t nrows, int64_t len, int32_t k,
                                int32_t largest, float* vals, int64_t* idx, mk_stream_t stream) {
    MK_REQUIRE(nrows >= 0 && len >= 0, MK_ERR_INVALID_ARG, "nrows and len must be >= 0");
    MK_REQUIRE(k >= 1, MK_ERR_INVALID_ARG, "k must be >= 1");
    MK_REQUIRE(k <= mk::kMaxK, MK_ERR_UNSUPPORTED, "k must be <= 1024");
    MK_REQUIRE(len < (int64_t)0xFFFFFFFF, MK_ERR_UNSUPPORTED, "rows must be shorter than 2^32-1");
    if (nrows == 0) return MK_OK;
    MK_REQUIRE(vals && idx && (a || len == 0), MK_ERR_INVALID_ARG, "null pointer");
    hipStream_t s = static_cast<hipStream_t>(stream);
    return largest ? mk::kselect_dispatch<true>(a, nrows, len, k, vals, idx, s)
                   : mk::kselect_dispatch<false>(a, nrows, len, k, vals, idx, s);
}
