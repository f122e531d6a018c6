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

// x = h + m + l, three BF16 numbers (8 + 8 + 8 bits: exact for 2^-100 <= |x| <
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

// Products of BF16 triples on v_mfma_f32_16x16x32_bf16: h h in one accumulator,
// the five products of 2^-8 and 2^-16 of it in another (l l, m l and l m, under
// 2^-26 of a product, are left out): six times the FP32 kernel's products at
// sixteen times its rate, with FP32 accumulation.  The error against 64 bits is
// smaller than the FP32 chain's (measured below).
//
// A workgroup keeps the triples of up to 96 KB of rot (128 x 128: all of it; less
// where the rows alone do not fill the chip) in LDS in operand order (16 outputs)
// and walks the rows, 32 per wave and step (lane = row; component 32 s + 16 half +
// 4 lh + e in slot 8 lh + 4 half + e, so that each load takes 64 consecutive bytes
// of a row), the next rows' loads in flight.  Where 16-byte stores are aligned (kQuads)
// rows are the columns of a product: lane (row, lh) ends up with outputs 4 lh ..
// 4 lh + 3.  Others are its rows: lane li has output li of four rows.  These go out
// as 64 consecutive bytes of a row at a time (kColumns) or, where a workgroup has
// short rows whole, through LDS as the one block that 16 rows of the result are
// (kBlocks: 2*10^6 x 64 rows, 57 outputs 318 -> 197 us).
//
// Triples hold a component exactly from 2^-100 on, and every product of parts stays
// a normal number where the least |x| (zeros aside) times the least |rot| is 2^-100
// or more; components below 2^60 cannot overflow.  Rows that are out of these
// bounds take FP32 products, a wave (32 rows) at a time, with rot from LDS (one
// component of 10^-17 in rot, 2*10^6 x 128 rows: 449 us, 2,023 with every such call
// on products with rot from memory; 768 by the FP32 kernel).
//
// Bound by memory: 2*10^6 x 128 rows, 2 GB in and out, 447 us (4.6 TB/s), 765 by the
// FP32 kernel; error against 64 bits 2.0e-7 -> 6.5e-8 of the largest value.
enum RotateOut { kQuads, kColumns, kBlocks };
template <int S, int OUT>
struct SplitShape {
    // two workgroups per CU where the registers allow it (64 outputs of 64 components,
    // which they don't: 211 us with one, 229 with two and spills; 57 outputs 200, 197)
    static constexpr int WPE = S == 1 || (S == 2 && OUT == kBlocks) ? 4 : 2, WAVES = 8, NB = 2;
    static constexpr int TILE_BYTES = S * 3 * 1024;
};
constexpr uint32_t float_bits(int exponent) { return (uint32_t)(127 + exponent) << 23; }

template <int S, bool VEC, int OUT>
__global__ __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(SplitShape<S, OUT>::WPE, SplitShape<S, OUT>::WPE)))
void rotate_split_kernel(const float* __restrict__ x, int64_t n, int32_t d,
                         const float* __restrict__ rot, int32_t dout, float* __restrict__ out,
                         int32_t tiles_per_wg, int32_t nchunks, int32_t vec_rot,
                         int32_t vec_out) {
    constexpr int NB = SplitShape<S, OUT>::NB, WAVES = SplitShape<S, OUT>::WAVES;
    constexpr bool QUADS = OUT == kQuads;
    constexpr int AHEAD = S <= 2 ? 2 : 4;  // operand blocks of rot in flight per wave
    extern __shared__ __align__(16) unsigned char smem[];
    bf16x8* planes = reinterpret_cast<bf16x8*>(smem);  // [tile][s][plane][lane]
    floatx4* whole = reinterpret_cast<floatx4*>(smem);  // [tile][s][half][lane], three planes apart
    __shared__ uint32_t rot_least, rot_most;  // bits of |rot| (least: less one, zeros aside)
    const int lane = threadIdx.x & 63, li = lane & 15, lh = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int chunk = blockIdx.x % nchunks;
    const int64_t wg = blockIdx.x / nchunks, nwg = gridDim.x / nchunks;
    const int t0 = chunk * tiles_per_wg;
    const int all = (dout + 15) / 16;
    const int ntiles = all - t0 < tiles_per_wg ? all - t0 : tiles_per_wg;

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
    const int64_t step = nwg * WAVES * 16 * NB;
    const int64_t start = (wg * WAVES + wave) * 16 * NB;
    if (start < n) load(start);

    // this lane's eight components of operand block f of rot
    auto rot_block = [&](int f, float (&v)[8]) __attribute__((always_inline)) {
        const int j = (t0 + f / S) * 16 + li;
        const float* p = rot + (int64_t)j * d;
#pragma unroll
        for (int half = 0; half < 2; ++half) {
            const int t = 32 * (f % S) + 16 * half + 4 * lh;
            if (vec_rot) {
                float4 w = make_float4(0.f, 0.f, 0.f, 0.f);
                if (j < dout && t < d) w = *reinterpret_cast<const float4*>(p + t);
                v[4 * half] = w.x;
                v[4 * half + 1] = w.y;
                v[4 * half + 2] = w.z;
                v[4 * half + 3] = w.w;
            } else {
#pragma unroll
                for (int e = 0; e < 4; ++e) v[4 * half + e] = j < dout && t + e < d ? p[t + e] : 0.f;
            }
        }
    };
    auto range = [&](float v, uint32_t& least, uint32_t& most) __attribute__((always_inline)) {
        const uint32_t u = __float_as_uint(v) & 0x7FFFFFFFu;
        least = min(least, u - 1u);  // (a zero: 2^32 - 1)
        most = max(most, u);
    };
    if (threadIdx.x == 0) {
        rot_least = ~0u;
        rot_most = 0u;
    }
    __syncthreads();
    {
        uint32_t least = ~0u, most = 0u;
#pragma unroll 1
        for (int f0 = wave; f0 < ntiles * S; f0 += WAVES * AHEAD) {
            float v[AHEAD][8];
#pragma unroll
            for (int a = 0; a < AHEAD; ++a) {
                const int f = f0 + a * WAVES;
                if (f < ntiles * S) rot_block(f, v[a]);
            }
#pragma unroll
            for (int a = 0; a < AHEAD; ++a) {
                const int f = f0 + a * WAVES;
                if (f >= ntiles * S) break;
#pragma unroll
                for (int e = 0; e < 8; ++e) range(v[a][e], least, most);
                bf16x8 h, m, l;
                split3(v[a], h, m, l);
                planes[(f * 3 + 0) * 64 + lane] = h;
                planes[(f * 3 + 1) * 64 + lane] = m;
                planes[(f * 3 + 2) * 64 + lane] = l;
            }
        }
#pragma unroll
        for (int o = 1; o < 64; o *= 2) {
            least = min(least, (uint32_t)__shfl_xor((int)least, o));
            most = max(most, (uint32_t)__shfl_xor((int)most, o));
        }
        if (lane == 0) {
            atomicMin(&rot_least, least);
            atomicMax(&rot_most, most);
        }
    }
    __syncthreads();
    const bool rot_ok = rot_most < float_bits(60) && rot_least >= float_bits(-100) - 1u;
    // |x| from here on (bits, less one)
    uint32_t x_least = float_bits(-100) - 1u;
    if (rot_ok && rot_least != ~0u) {
        const int e = (int)((rot_least + 1u) >> 23) - 127;
        if (e < 0) x_least = float_bits(-100 - e) - 1u;
    }
    if (!rot_ok) {  // rot itself in the triples' place
        for (int f = wave; f < ntiles * S; f += WAVES) {
            float v[8];
            rot_block(f, v);
            whole[f * 3 * 64 + lane] = floatx4{v[0], v[1], v[2], v[3]};
            whole[(f * 3 + 1) * 64 + lane] = floatx4{v[4], v[5], v[6], v[7]};
        }
        __syncthreads();
    }

    // block b of a wave's rows, outputs of a tile
    auto store = [&](int64_t r0, int tile, floatx4 v) __attribute__((always_inline)) {
        const int64_t row = r0 + (QUADS ? li : 4 * lh);
        const int col = (t0 + tile) * 16 + (QUADS ? 4 * lh : li);
        if constexpr (QUADS) {
            if (row < n && col < dout) *reinterpret_cast<floatx4*>(out + row * dout + col) = v;
        } else if (col < dout) {
#pragma unroll
            for (int i = 0; i < 4; ++i)
                if (row + i < n) out[(row + i) * dout + col] = v[i];
        }
    };
    auto mma = [&](floatx4 acc, bf16x8 a, bf16x8 b) __attribute__((always_inline)) {
        return QUADS ? __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, acc, 0, 0, 0)
                    : __builtin_amdgcn_mfma_f32_16x16x32_bf16(b, a, acc, 0, 0, 0);
    };
#pragma unroll 1
    for (int64_t r0 = start; r0 < n; r0 += step) {
        uint32_t least = ~0u, most = 0u;
#pragma unroll
        for (int b = 0; b < NB; ++b)
#pragma unroll
            for (int s = 0; s < S; ++s)
#pragma unroll
                for (int e = 0; e < 8; ++e) range(next[b][s][e], least, most);
        if (!rot_ok || __ballot(least < x_least || most >= float_bits(60))) {
            // FP32 products
#pragma unroll 1
            for (int tile = 0; tile < ntiles; ++tile) {
                floatx4 acc[NB];
#pragma unroll
                for (int b = 0; b < NB; ++b) acc[b] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int s = 0; s < S; ++s) {
                    const int f = tile * S + s;
                    float v[8];
                    if (rot_ok) {
                        const bf16x8 h = planes[(f * 3 + 0) * 64 + lane], m = planes[(f * 3 + 1) * 64 + lane],
                                     l = planes[(f * 3 + 2) * 64 + lane];
#pragma unroll
                        for (int e = 0; e < 8; ++e) v[e] = (float)h[e] + ((float)m[e] + (float)l[e]);
                    } else {
                        const floatx4 a = whole[f * 3 * 64 + lane], c = whole[(f * 3 + 1) * 64 + lane];
#pragma unroll
                        for (int e = 0; e < 4; ++e) {
                            v[e] = a[e];
                            v[4 + e] = c[e];
                        }
                    }
#pragma unroll
                    for (int e = 0; e < 8; ++e)
#pragma unroll
                        for (int b = 0; b < NB; ++b)
                            acc[b] = QUADS ? __builtin_amdgcn_mfma_f32_16x16x4f32(v[e], next[b][s][e], acc[b], 0, 0, 0)
                                          : __builtin_amdgcn_mfma_f32_16x16x4f32(next[b][s][e], v[e], acc[b], 0, 0, 0);
                }
#pragma unroll
                for (int b = 0; b < NB; ++b) store(r0 + b * 16, tile, acc[b]);
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
        if constexpr (OUT == kBlocks) {
            float* stage = reinterpret_cast<float*>(planes + ntiles * S * 3 * 64) + wave * 16 * dout;
#pragma unroll
            for (int b = 0; b < NB; ++b) {
#pragma unroll 1
                for (int tile = 0; tile < ntiles; ++tile) {
                    const bf16x8* a = planes + (int64_t)tile * S * 3 * 64 + lane;
                    floatx4 big = {0.f, 0.f, 0.f, 0.f}, rest = big;
#pragma unroll
                    for (int s = 0; s < S; ++s) {
                        const bf16x8 ah = a[(s * 3 + 0) * 64], am = a[(s * 3 + 1) * 64], al = a[(s * 3 + 2) * 64];
                        rest = mma(rest, al, h[b][s]);
                        big = mma(big, ah, h[b][s]);
                        rest = mma(rest, ah, l[b][s]);
                        rest = mma(rest, am, m[b][s]);
                        rest = mma(rest, am, h[b][s]);
                        rest = mma(rest, ah, m[b][s]);
                    }
                    big += rest;
                    if (tile * 16 + li < dout)
#pragma unroll
                        for (int i = 0; i < 4; ++i) stage[(4 * lh + i) * dout + tile * 16 + li] = big[i];
                }
                __builtin_amdgcn_wave_barrier();
                __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "workgroup");
                const int64_t row = r0 + b * 16, rows = n - row < 16 ? n - row : 16;
                float* o = out + row * dout;
                int e = lane;
                if (vec_out) {  // (16 rows: a multiple of 64 bytes)
                    const int quads = (int)rows * dout / 4;
                    for (int g = lane; g < quads; g += 64)
                        reinterpret_cast<floatx4*>(o)[g] = reinterpret_cast<const floatx4*>(stage)[g];
                    e += 4 * quads;
                }
                for (; e < (int)rows * dout; e += 64) o[e] = stage[e];
                __builtin_amdgcn_wave_barrier();
                __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "workgroup");
            }
            continue;
        }
#pragma unroll 1
        for (int tile = 0; tile < ntiles; ++tile) {
            const bf16x8* a = planes + (int64_t)tile * S * 3 * 64 + lane;
            floatx4 big[NB], rest[NB];
#pragma unroll
            for (int b = 0; b < NB; ++b) big[b] = rest[b] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int s = 0; s < S; ++s) {
                const bf16x8 ah = a[(s * 3 + 0) * 64], am = a[(s * 3 + 1) * 64], al = a[(s * 3 + 2) * 64];
#pragma unroll
                for (int b = 0; b < NB; ++b) rest[b] = mma(rest[b], al, h[b][s]);
#pragma unroll
                for (int b = 0; b < NB; ++b) big[b] = mma(big[b], ah, h[b][s]);
#pragma unroll
                for (int b = 0; b < NB; ++b) rest[b] = mma(rest[b], ah, l[b][s]);
#pragma unroll
                for (int b = 0; b < NB; ++b) rest[b] = mma(rest[b], am, m[b][s]);
#pragma unroll
                for (int b = 0; b < NB; ++b) rest[b] = mma(rest[b], am, h[b][s]);
#pragma unroll
                for (int b = 0; b < NB; ++b) rest[b] = mma(rest[b], ah, m[b][s]);
            }
#pragma unroll
            for (int b = 0; b < NB; ++b) store(r0 + b * 16, tile, big[b] + rest[b]);
        }
    }
}

template <int S, int OUT>
mk_status rotate_split_as(const float* x, int64_t n, int32_t d, const float* rot, int32_t dout,
                          float* out, bool vec, hipStream_t s) {
    using Sh = SplitShape<S, OUT>;
    // at most 96 KB of rot's triples per CU; where the rows give fewer workgroups
    // than the chip takes, the outputs are shared out too, and each workgroup has
    // less of rot to lay out
    constexpr int64_t kWgs = 256 * (Sh::WPE / 2), kTiles = 98304 / (Sh::WPE / 2) / Sh::TILE_BYTES;
    const int64_t all = ceil_div(dout, 16), rows = ceil_div(n, 16 * Sh::NB * Sh::WAVES);
    int64_t nchunks = std::max(ceil_div(all, kTiles), std::min(all, kWgs / std::min(rows, kWgs)));
    if (OUT == kBlocks) nchunks = 1;
    const int32_t tiles = (int32_t)ceil_div(all, nchunks);
    nchunks = ceil_div(all, tiles);
    const int64_t wgs = std::min(std::max<int64_t>(kWgs / nchunks, 1), rows);
    const size_t lds = (size_t)tiles * Sh::TILE_BYTES +
                       (OUT == kBlocks ? sizeof(float) * Sh::WAVES * 16 * (size_t)dout : 0);
    const bool vec_rot = d % 4 == 0 && reinterpret_cast<uintptr_t>(rot) % 16 == 0;
    const bool vec_out = reinterpret_cast<uintptr_t>(out) % 16 == 0;
    auto kern = vec ? rotate_split_kernel<S, true, OUT> : rotate_split_kernel<S, false, OUT>;
    if (lds > 65536)
        MK_HIP(hipFuncSetAttribute(reinterpret_cast<const void*>(kern),
                                   hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
    hipLaunchKernelGGL(kern, dim3((unsigned)(wgs * nchunks)), dim3(512), lds, s, x, n, d, rot, dout,
                       out, tiles, (int32_t)nchunks, (int32_t)vec_rot, (int32_t)vec_out);
    MK_LAUNCHED();
    return MK_OK;
}

template <int S>
mk_status rotate_split(const float* x, int64_t n, int32_t d, const float* rot, int32_t dout,
                       float* out, bool vec, hipStream_t s) {
    if (dout % 4 == 0 && reinterpret_cast<uintptr_t>(out) % 16 == 0)
        return rotate_split_as<S, kQuads>(x, n, d, rot, dout, out, vec, s);
    // (two workgroups per CU with up to 64 outputs; of few rows each has a share of
    // the outputs)
    if constexpr (S <= 2)
        if (dout <= 64 && n >= 65536) return rotate_split_as<S, kBlocks>(x, n, d, rot, dout, out, vec, s);
    return rotate_split_as<S, kColumns>(x, n, d, rot, dout, out, vec, s);
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
    // Rows of 128 components are what the registers hold; sums of a few products are
    // rounded less often in FP32 (d = 1: once).  From about 30,000 rows on faster
    // (FP32 kernel, this one; 128 outputs of 128 components: 16,384 rows 10.4, 12.3 us,
    // 30,000 rows 17.4, 16.7, 50,000 rows 25.2, 21.9, 200,000 rows 77, 57, 2*10^6 rows 765,
    // 447; the worst of 24 to 128 components and 16 to 128 outputs: 100,000 x 64 rows,
    // 57 outputs 16.0, 17.6, and 200,000 rows 26.7, 26.5); between 16,384 rows and that
    // for its smaller error.
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
