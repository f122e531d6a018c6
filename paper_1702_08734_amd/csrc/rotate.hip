// Linear pre-processing of rows (an OPQ rotation or a projection, Sections 1
// and 6.4): out[i][j] = sum_t x[i][t] * rot[j][t] on the FP32 matrix cores.
//
// One workgroup per 64 x 64 output tile, four waves of 2 x 2 blocks of
// 16 x 16 (v_mfma_f32_16x16x4f32).  K goes in chunks of 32 staged whole in
// LDS (rows of x and of rot, both K-contiguous, one barrier pair per chunk);
// LDS rows are 34 floats apart so that the operand reads of a 32-lane half
// (16 rows x 2 k-groups) fall in 32 distinct banks.  The 17 KB of LDS per
// workgroup let the CU hold as many workgroups as its wave slots allow, and
// their staging overlaps each other's matrix work (chunks of 64, 34 KB:
// 4.9 ms for 10^7 x 128 rows; chunks of 32: 4.0 ms).  Consecutive workgroups
// share a row tile (its loads hit L2).  Every output element sums its
// products in one fixed order, so the result is deterministic.
//
// Many rows of up to 128 components take the BF16 matrix cores instead
// (rotate_split_kernel), with every factor as three BF16 numbers that add up to
// it exactly.
#include <algorithm>

#include "common.hpp"

namespace mk {
namespace {

typedef float floatx4 __attribute__((ext_vector_type(4)));

constexpr int kTile = 64;   // rows and columns of an output tile
constexpr int kKC = 32;     // K per LDS stage
constexpr int kLds = kKC + 2;

// Rows [r0, r0 + 64) x k [k0, k0 + 32) of a row-major [rows, d] matrix into
// S (zero outside), 256 threads; float4 loads when vec.
__device__ __forceinline__ void stage(float (*S)[kLds], const float* __restrict__ m, int64_t rows,
                                      int32_t d, int64_t r0, int32_t k0, bool vec) {
    const int tid = threadIdx.x;
    if (vec) {
#pragma unroll
        for (int e = tid; e < kTile * (kKC / 4); e += 256) {
            const int r = e / (kKC / 4), c = 4 * (e % (kKC / 4));
            const int64_t row = r0 + r;
            const int32_t k = k0 + c;
            float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
            if (row < rows && k < d) v = *reinterpret_cast<const float4*>(m + row * d + k);
            *reinterpret_cast<float2*>(&S[r][c]) = make_float2(v.x, v.y);
            *reinterpret_cast<float2*>(&S[r][c + 2]) = make_float2(v.z, v.w);
        }
    } else {
        for (int e = tid; e < kTile * kKC; e += 256) {
            const int r = e / kKC, c = e % kKC;
            const int64_t row = r0 + r;
            const int32_t k = k0 + c;
            S[r][c] = (row < rows && k < d) ? m[row * d + k] : 0.f;
        }
    }
}

__global__ __launch_bounds__(256) void rotate_rows_kernel(const float* __restrict__ x, int64_t n,
                                                          int32_t d, const float* __restrict__ rot,
                                                          int32_t dout, float* __restrict__ out,
                                                          int64_t ncb, int32_t vec) {
    __shared__ __align__(16) float As[kTile][kLds];
    __shared__ __align__(16) float Bs[kTile][kLds];
    const int64_t b = blockIdx.x;
    const int64_t r0 = (b / ncb) * kTile, c0 = (b % ncb) * kTile;
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
    const int li = lane & 15, lh = lane >> 4;
    const int wm = (wave >> 1) * 32, wn = (wave & 1) * 32;
    floatx4 acc[2][2];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) acc[i][j] = floatx4{0.f, 0.f, 0.f, 0.f};
    for (int32_t k0 = 0; k0 < d; k0 += kKC) {
        if (k0 > 0) __syncthreads();  // the previous chunk's reads are done
        stage(As, x, n, d, r0, k0, vec != 0);
        stage(Bs, rot, dout, d, c0, k0, vec != 0);
        __syncthreads();
#pragma unroll
        for (int kk = 0; kk < kKC / 4; ++kk) {
            float av[2], bv[2];
#pragma unroll
            for (int i = 0; i < 2; ++i) av[i] = As[wm + i * 16 + li][kk * 4 + lh];
#pragma unroll
            for (int j = 0; j < 2; ++j) bv[j] = Bs[wn + j * 16 + li][kk * 4 + lh];
#pragma unroll
            for (int i = 0; i < 2; ++i)
#pragma unroll
                for (int j = 0; j < 2; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(av[i], bv[j], acc[i][j], 0, 0, 0);
        }
    }
    // D[i][j] of a 16 x 16 block sits in lane j + 16 (i / 4), element i % 4
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int64_t row = r0 + wm + i * 16 + 4 * lh + r;
                const int64_t col = c0 + wn + j * 16 + li;
                if (row < n && col < dout) out[row * dout + col] = acc[i][j][r];
            }
}

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));

// x = h + m + l, three BF16 numbers (8 + 8 + 8 bits: exact for 2^-50 <= |x| <
// 2^60 and zero).
__device__ __forceinline__ void split3(const float (&v)[8], bf16x8& h, bf16x8& m, bf16x8& l) {
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        h[e] = (__bf16)v[e];
        const float r = v[e] - (float)h[e];
        m[e] = (__bf16)r;
        l[e] = (__bf16)(r - (float)m[e]);
    }
}
__device__ __forceinline__ bool splittable(float v) {
    const float a = fabsf(v);
    return a == 0.f || (a >= 0x1p-50f && a < 0x1p60f);
}

// Products of BF16 triples on v_mfma_f32_16x16x32_bf16: h h in one accumulator,
// the five products of 2^-8 and 2^-16 of it in another (l l, m l and l m, under
// 2^-26 of a product, are left out): six times the FP32 kernel's products at
// sixteen times its rate, with FP32 accumulation.  The error against 64 bits is
// smaller than the FP32 chain's (measured below).
//
// A workgroup keeps the triples of up to 96 KB of rot (128 x 128: all of it) in
// LDS in operand order (A: 16 outputs) and walks the rows, 32 per wave and step
// (B: lane = row; component 32 s + 16 half + 4 lh + e in slot 8 lh + 4 half + e,
// so that each load takes 64 consecutive bytes of a row), the next rows' loads in
// flight.  Lane (row, lh) ends up with outputs 4 lh .. 4 lh + 3: one 16-byte
// store.  Rows with a component that the triples cannot hold (not finite, huge or
// tiny) take FP32 products, a wave at a time.
//
// Bound by memory: 2*10^6 x 128 rows, 2 GB in and out, 779 -> 500 us (4.1 TB/s); error
// against 64 bits 2.0e-7 -> 6.5e-8 of the largest value.
template <int S, bool VEC>
__global__ __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(2, 2))) void rotate_split_kernel(
    const float* __restrict__ x, int64_t n, int32_t d, const float* __restrict__ rot, int32_t dout,
    float* __restrict__ out, int32_t tiles_per_wg, int32_t nchunks, int32_t vec_out) {
    constexpr int NB = 2, WAVES = 8;
    extern __shared__ __align__(16) unsigned char smem[];
    bf16x8* planes = reinterpret_cast<bf16x8*>(smem);  // [tile][s][plane][lane]
    __shared__ uint32_t rot_bad;
    const int lane = threadIdx.x & 63, li = lane & 15, lh = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int chunk = blockIdx.x % nchunks;
    const int64_t wg = blockIdx.x / nchunks, nwg = gridDim.x / nchunks;
    const int t0 = chunk * tiles_per_wg;
    const int all = (dout + 15) / 16;
    const int ntiles = all - t0 < tiles_per_wg ? all - t0 : tiles_per_wg;
    if (threadIdx.x == 0) rot_bad = 0u;
    __syncthreads();
    // component of slot e of step s
    auto comp = [&](int s, int e) __attribute__((always_inline)) {
        return 32 * s + 16 * (e >> 2) + 4 * lh + (e & 3);
    };
    for (int f = wave; f < ntiles * S; f += WAVES) {
        const int tile = f / S, s = f % S;
        const int j = (t0 + tile) * 16 + li;
        float v[8];
        bool ok = true;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const int t = comp(s, e);
            v[e] = j < dout && t < d ? rot[(int64_t)j * d + t] : 0.f;
            ok = ok && splittable(v[e]);
        }
        if (!ok) rot_bad = 1u;
        bf16x8 h, m, l;
        split3(v, h, m, l);
        planes[(f * 3 + 0) * 64 + lane] = h;
        planes[(f * 3 + 1) * 64 + lane] = m;
        planes[(f * 3 + 2) * 64 + lane] = l;
    }
    __syncthreads();
    const bool rot_ok = rot_bad == 0u;

    float next[NB][S][8];
    auto load = [&](int64_t r0) __attribute__((always_inline)) {
#pragma unroll
        for (int b = 0; b < NB; ++b) {
            int64_t row = r0 + b * 16 + li;
            row = row < n ? row : n - 1;
            const float* p = x + row * d;
#pragma unroll
            for (int s = 0; s < S; ++s)
#pragma unroll
                for (int half = 0; half < 2; ++half) {
                    const int t = 32 * s + 16 * half + 4 * lh;
                    if constexpr (VEC) {
                        float4 w = make_float4(0.f, 0.f, 0.f, 0.f);
                        if (t < d) w = *reinterpret_cast<const float4*>(p + t);
                        next[b][s][4 * half] = w.x;
                        next[b][s][4 * half + 1] = w.y;
                        next[b][s][4 * half + 2] = w.z;
                        next[b][s][4 * half + 3] = w.w;
                    } else {
#pragma unroll
                        for (int e = 0; e < 4; ++e)
                            next[b][s][4 * half + e] = t + e < d ? p[t + e] : 0.f;
                    }
                }
        }
    };
    auto store = [&](int64_t row, int col, floatx4 v) __attribute__((always_inline)) {
        if (row >= n) return;
        float* o = out + row * dout + col;
        if (vec_out && col + 4 <= dout) {
            *reinterpret_cast<floatx4*>(o) = v;
        } else {
#pragma unroll
            for (int e = 0; e < 4; ++e)
                if (col + e < dout) o[e] = v[e];
        }
    };
    const int64_t step = nwg * WAVES * 16 * NB;
    const int64_t start = (wg * WAVES + wave) * 16 * NB;
    if (start < n) load(start);
#pragma unroll 1
    for (int64_t r0 = start; r0 < n; r0 += step) {
        bool ok = rot_ok;
#pragma unroll
        for (int b = 0; b < NB; ++b)
#pragma unroll
            for (int s = 0; s < S; ++s)
#pragma unroll
                for (int e = 0; e < 8; ++e) ok = ok && splittable(next[b][s][e]);
        if (__ballot(!ok)) {
            // FP32 products, rot from memory
#pragma unroll 1
            for (int tile = 0; tile < ntiles; ++tile) {
                const int j = (t0 + tile) * 16 + li;
                floatx4 acc[NB];
#pragma unroll
                for (int b = 0; b < NB; ++b) acc[b] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int s = 0; s < S; ++s)
#pragma unroll
                    for (int e = 0; e < 8; ++e) {
                        const int t = comp(s, e);
                        const float a = j < dout && t < d ? rot[(int64_t)j * d + t] : 0.f;
#pragma unroll
                        for (int b = 0; b < NB; ++b)
                            acc[b] = __builtin_amdgcn_mfma_f32_16x16x4f32(a, next[b][s][e], acc[b], 0, 0, 0);
                    }
#pragma unroll
                for (int b = 0; b < NB; ++b)
                    store(r0 + b * 16 + li, (t0 + tile) * 16 + 4 * lh, acc[b]);
            }
            if (r0 + step < n) load(r0 + step);
            continue;
        }
        bf16x8 h[NB][S], m[NB][S], l[NB][S];
#pragma unroll
        for (int b = 0; b < NB; ++b)
#pragma unroll
            for (int s = 0; s < S; ++s) split3(next[b][s], h[b][s], m[b][s], l[b][s]);
        if (r0 + step < n) load(r0 + step);
#pragma unroll 1
        for (int tile = 0; tile < ntiles; ++tile) {
            const bf16x8* a = planes + (int64_t)tile * S * 3 * 64 + lane;
            floatx4 big[NB], rest[NB];
#pragma unroll
            for (int b = 0; b < NB; ++b) big[b] = rest[b] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int s = 0; s < S; ++s) {
                const bf16x8 ah = a[(s * 3 + 0) * 64], am = a[(s * 3 + 1) * 64], al = a[(s * 3 + 2) * 64];
#define MK_MFMA(acc, p, q) \
    _Pragma("unroll") for (int b = 0; b < NB; ++b) \
        acc[b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(p, q[b][s], acc[b], 0, 0, 0)
                MK_MFMA(rest, al, h);
                MK_MFMA(big, ah, h);
                MK_MFMA(rest, ah, l);
                MK_MFMA(rest, am, m);
                MK_MFMA(rest, am, h);
                MK_MFMA(rest, ah, m);
#undef MK_MFMA
            }
#pragma unroll
            for (int b = 0; b < NB; ++b)
                store(r0 + b * 16 + li, (t0 + tile) * 16 + 4 * lh, big[b] + rest[b]);
        }
    }
}

template <int S>
mk_status rotate_split(const float* x, int64_t n, int32_t d, const float* rot, int32_t dout,
                       float* out, bool vec, hipStream_t s) {
    // at most 96 KB of rot's triples per workgroup, one workgroup per CU
    constexpr int kTileBytes = S * 3 * 1024;
    const int32_t all = (int32_t)ceil_div(dout, 16);
    const int32_t nchunks = (int32_t)ceil_div(all, 98304 / kTileBytes);
    const int32_t tiles = (int32_t)ceil_div(all, nchunks);
    const int64_t wgs = std::min<int64_t>(std::max<int64_t>(256 / nchunks, 1), ceil_div(n, 256));
    const size_t lds = (size_t)tiles * kTileBytes;
    const bool vec_out = dout % 4 == 0 && reinterpret_cast<uintptr_t>(out) % 16 == 0;
    auto kern = vec ? rotate_split_kernel<S, true> : rotate_split_kernel<S, false>;
    if (lds > 65536)
        MK_HIP(hipFuncSetAttribute(reinterpret_cast<const void*>(kern),
                                   hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
    hipLaunchKernelGGL(kern, dim3((unsigned)(wgs * nchunks)), dim3(512), lds, s, x, n, d, rot, dout,
                       out, tiles, nchunks, (int32_t)vec_out);
    MK_LAUNCHED();
    return MK_OK;
}

}  // namespace
}  // namespace mk

extern "C" mk_status mk_rotate_rows(const float* x, int64_t n, int32_t d, const float* rot,
                                    int32_t dout, float* out, mk_stream_t stream) {
    MK_REQUIRE(n >= 0 && d >= 1 && dout >= 1, MK_ERR_INVALID_ARG, "need n >= 0, d >= 1, dout >= 1");
    if (n == 0) return MK_OK;
    MK_REQUIRE(x && rot && out, MK_ERR_INVALID_ARG, "null pointer");
    const char* xe = reinterpret_cast<const char*>(x + n * (int64_t)d);
    const char* oe = reinterpret_cast<const char*>(out + n * (int64_t)dout);
    MK_REQUIRE(xe <= reinterpret_cast<const char*>(out) || oe <= reinterpret_cast<const char*>(x),
               MK_ERR_INVALID_ARG, "out must not overlap x");
    const int64_t ncb = mk::ceil_div(dout, mk::kTile);
    const int64_t blocks = mk::ceil_div(n, mk::kTile) * ncb;
    MK_REQUIRE(blocks < ((int64_t)1 << 32), MK_ERR_UNSUPPORTED, "too many rows for one call");
    const bool vec = d % 4 == 0 && reinterpret_cast<uintptr_t>(x) % 16 == 0 &&
                     reinterpret_cast<uintptr_t>(rot) % 16 == 0;
    // enough rows that a workgroup's set-up (rot into triples) is small beside
    // them; rows of 128 components are what the registers hold; sums of a few
    // products are rounded less often in FP32 (d = 1: once)
    if (d >= 24 && d <= 128 && n >= 16384) {
        const bool vx = d % 4 == 0 && reinterpret_cast<uintptr_t>(x) % 16 == 0;
        const hipStream_t s = static_cast<hipStream_t>(stream);
        if (d <= 32) return mk::rotate_split<1>(x, n, d, rot, dout, out, vx, s);
        if (d <= 64) return mk::rotate_split<2>(x, n, d, rot, dout, out, vx, s);
        if (d <= 96) return mk::rotate_split<3>(x, n, d, rot, dout, out, vx, s);
        return mk::rotate_split<4>(x, n, d, rot, dout, out, vx, s);
    }
    hipLaunchKernelGGL(mk::rotate_rows_kernel, dim3((unsigned)blocks), dim3(256), 0,
                       static_cast<hipStream_t>(stream), x, n, d, rot, dout, out, ncb,
                       (int32_t)vec);
    MK_LAUNCHED();
    return MK_OK;
}
