// Threshold-first exact search for batches of queries: the selector of the
// fused kernel (fused.hpp) leaves the matrix waves.
//
//   1. A stratified sample of the database is scored; of every 4 to 16 of its
//      rows the least score is kept, and the r-th best of these (at least the
//      r-th best of the sample, and rarely more) is the query's threshold, r
//      chosen so that it lets a few times keff rows of the database through.
//   2. sieve_tiles streams the database once: every wave holds 64 queries
//      (32 for wide rows) as MFMA operands in registers, compares each score
//      with its query's threshold in the accumulator registers (one lane = one
//      query, so the threshold is a register and a 16 x 16 block costs a
//      minimum tree and one compare) and appends the few that pass to the
//      query's pool in device memory.
//   3. sieve_finish selects the keff best of the pool, re-ranks them in the
//      direct FP32 form and writes the k best.
//
// What bounds it: the matrix cores, and the vector operations beside them.  10,000
// queries x 1,000,000 x 128, k = 32: sieve_tiles 6.0 to 6.4 ms from card to card (1,200
// to 1,280 TFLOP/s of FP16 products; 5.8 ms when no score passes), the whole search 6.3
// to 6.6 ms against 27.1 ms by the fused kernel (95 TFLOP/s of FP32 products, and FP32
// products cannot take less than 16.3 ms); 2,000 queries, k = 1000: 1.7 against 9.6 ms.
//
// Nothing is taken on trust: a query whose pool overflowed or came out short, or (FP32
// search) whose result the error bound does not prove, goes to a list of queries that
// are searched again: few of them by dense.hpp's search, the others by the fused kernel,
// whose workgroups return at once when there are none.  (One zero query in 30, inner
// products, 10^6 x 128 rows, 10,000 queries, k = 10: whole blocks of 64 searched again by
// the fused kernel 40.0 ms, the list 8.2, 6.5 without zero queries.)
//
// FP32 rows are multiplied as pairs of FP16 rows (h + l, each row scaled by a
// power of two): three FP16 matrix products (h l, l h, h h) carry 22+ bits of
// every product at a third of the FP16 rate, 5 times the FP32 matrix rate.
#pragma once

#include "fused.hpp"
#include "pool.hpp"
#include "sieve_plan.hpp"

namespace mk {

typedef _Float16 half8 __attribute__((ext_vector_type(8)));

struct SieveSplit {  // two FP16 planes per row: h, then l
    static constexpr int EPG = 8, BYTES = 2, PLANES = 2;
    static constexpr bool SCALED = true;
    static constexpr bool SHIFTED = true;  // lower-bound shift (IP: per-row norm)
    static constexpr int MMAS = 3;         // matrix products per granule step
    template <int S4>
    __device__ static __forceinline__ floatx4 mma(floatx4 c, const uint4 (&b)[2 * S4],
                                                  const uint4 (&q)[2 * S4], int s4) {
        const half8 bh = __builtin_bit_cast(half8, b[s4]), bl = __builtin_bit_cast(half8, b[S4 + s4]);
        const half8 qh = __builtin_bit_cast(half8, q[s4]), ql = __builtin_bit_cast(half8, q[S4 + s4]);
        c = __builtin_amdgcn_mfma_f32_16x16x32_f16(bh, ql, c, 0, 0, 0);
        c = __builtin_amdgcn_mfma_f32_16x16x32_f16(bl, qh, c, 0, 0, 0);
        return __builtin_amdgcn_mfma_f32_16x16x32_f16(bh, qh, c, 0, 0, 0);
    }
};
// The low-precision formats run the products of the fused kernel in its
// order (so their scores, and with them the candidates they keep, are the
// same bit for bit).
struct SieveBF16 {
    static constexpr int EPG = 8, BYTES = 2, PLANES = 1;
    static constexpr bool SCALED = false, SHIFTED = false;
    static constexpr int MMAS = 1;
    template <int S4>
    __device__ static __forceinline__ floatx4 mma(floatx4 c, const uint4 (&b)[S4],
                                                  const uint4 (&q)[S4], int s4) {
        return OpBF16::mma(c, b[s4], q[s4]);
    }
};
struct SieveFP8 {
    static constexpr int EPG = 16, BYTES = 1, PLANES = 1;
    static constexpr bool SCALED = true, SHIFTED = false;
    static constexpr int MMAS = 2;
    template <int S4>
    __device__ static __forceinline__ floatx4 mma(floatx4 c, const uint4 (&b)[S4],
                                                  const uint4 (&q)[S4], int s4) {
        return OpFP8::mma(c, b[s4], q[s4]);
    }
};

// Workgroup of sieve_tiles: 8 waves (2 per SIMD) as 4 query groups x 2 row
// groups.  A wave reads each 16-row operand block from LDS once per QB * 16
// queries: with 64 queries of split rows the LDS reads take about a third of the
// matrix time.  Tiles of 16 to 32 KB, three in flight.
template <class Op, int DP>
struct SieveShape {
    static constexpr int WAVES = 8, QG = 4, RG = 2;
    static constexpr int GRP = DP / Op::EPG;          // granules per plane
    static constexpr int GR = Op::PLANES * GRP;       // granules per row
    static constexpr int S4 = GRP / 4;                // granule steps
    // 16-query blocks per wave: what the registers hold beside two blocks'
    // accumulators
    static constexpr int QREGS = Op::PLANES * S4 * 4;
    static constexpr int QB = 8 * QREGS <= 96 ? 8 : 4 * QREGS <= 128 ? 4 : 2;
    static constexpr int BQ = QG * QB * 16;
    static constexpr int RBW = GR >= 64 ? 1 : GR >= 24 ? 2 : 4;  // row blocks per wave and step
    static constexpr int BN = RG * RBW * 16;
    static constexpr int PER = 4 * RBW;  // rows behind one entry of a sample's least scores
    static constexpr int NBUF = 3;
    static constexpr int LPW = BN * GR / (64 * WAVES);  // tile loads per wave
    static_assert(GRP % 4 == 0 && BN * GR % (64 * WAVES) == 0, "tile loads split evenly");
};

struct SieveArgs {
    const void* xq;       // queries, rows of `stride` bytes
    const float* qscale;  // per-query 1/scale (scaled formats)
    const float* qnorm;   // per-query ||x||^2 (split, inner product)
    const void* xb;       // database rows of this launch, same format
    const float* ya;      // per-row 1/scale (scaled formats)
    const float* yb;      // per-row ||y||^2 (L2) or ||y|| (split, inner product)
    int64_t nq, nb;       // nb: rows of this launch
    uint32_t row0;        // index of its first row
    int32_t stride;       // bytes per row
    int64_t chunk_len;
    int32_t nchunks, nqb;
    const float* thr;     // filter: threshold of query q at thr[q * thr_ld]
    int64_t thr_ld;
    float tail;           // filter (split, L2): see the queries without a chance below
    const uint32_t* flags;   // filter (split): [nq] queries that the split cannot hold
    const uint32_t* bad_db;  // filter, nearest (split): a row that it cannot hold was seen
    uint32_t* cnt;        // filter: [nq] keys appended (may exceed cap)
    uint64_t* pool;       // filter: [nq][cap] keys
    uint32_t cap;
    float* scores;        // sample: [nq][ld] least scores
    int64_t ld;
    uint4* near;          // nearest: [nq] (group, second group, its score, bound of the rest)
};

// kFilter: rows that pass their query's threshold, to the pools.
// kSample: the least score of each lane's rows of a step (4 RBW of them), as the
//   entries of [nq][ld].
// kNearest: per query the two best groups of four rows (by their least scores)
//   and the least score outside them; one chunk.
enum SieveMode { kFilter = 0, kSample = 1, kNearest = 2 };

// Select and minimum as single instructions: the compiler turns chains of selects
// into branches, and quiets the inputs of fminf.
__device__ __forceinline__ uint32_t pick(uint64_t mask, uint32_t yes, uint32_t no) {
    uint32_t r;
    asm("v_cndmask_b32_e64 %0, %1, %2, %3" : "=v"(r) : "v"(no), "v"(yes), "s"(mask));
    return r;
}
__device__ __forceinline__ float min_raw(float a, float b) {
    float r;
    asm("v_min_f32_e32 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
    return r;
}

// Two best groups of four rows and a lower bound of everything else.
struct Nearest {
    float b1, b2, b3;
    uint32_t g1, g2;
    __device__ __forceinline__ void init() {
        b1 = b2 = b3 = INFINITY;
        g1 = g2 = ~0u;
    }
    __device__ __forceinline__ void offer(float s, uint32_t g) {
        b3 = __builtin_amdgcn_fmed3f(s, b2, b3);
        const uint64_t lt2 = __ballot(s < b2), lt1 = __ballot(s < b1);
        g2 = pick(lt1, g1, pick(lt2, g, g2));
        b2 = __builtin_amdgcn_fmed3f(s, b1, b2);
        g1 = pick(lt1, g, g1);
        b1 = min_raw(s, b1);
    }
    // another lane's findings; its third score has no group, so it only
    // lowers the bound (which may then lie below b1 or b2)
    __device__ __forceinline__ void merge(const Nearest& o) {
        const float third = fminf(b3, o.b3);
        b3 = INFINITY;
        offer(o.b1, o.g1);
        offer(o.b2, o.g2);
        b3 = fminf(b3, third);
    }
};

template <class Op, int DP, bool L2, int MODE>
__global__ __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(2, 2))) void sieve_tiles(
    SieveArgs args) {
    using S = SieveShape<Op, DP>;
    constexpr int GR = S::GR, S4 = S::S4, QB = S::QB, RBW = S::RBW, BN = S::BN, LPW = S::LPW;
    constexpr int BQ = S::BQ, NBUF = S::NBUF, PL = Op::PLANES;
    constexpr bool SAMPLE = MODE == kSample, FILTER = MODE == kFilter, NEAREST = MODE == kNearest;
    constexpr bool HASB = L2 || Op::SHIFTED;
    constexpr float ERR = split_err(DP);
    constexpr int NSIDE = (Op::SCALED ? 1 : 0) + (HASB ? 1 : 0);
    // granule c of tile row j sits at c ^ (j & SW), or where rows are 12
    // granules at c + j / 2 (mod 12): the rows of an operand read fall in
    // different banks
    constexpr int SW = (GR % 16 == 0) ? 15 : (GR % 8 == 0) ? 7 : 3;
    constexpr bool ROT = GR == 12;
    auto place = [](int c, int j) __attribute__((always_inline)) {
        if constexpr (ROT) {
            const int t = c + ((j >> 1) & 3);
            return t >= GR ? t - GR : t;
        } else {
            return c ^ (GR == 4 ? (j >> 1) & 3 : j & SW);
        }
    };
    constexpr int SIDE_OPS = NSIDE * ((BN + 63) / 64);  // waves with one more load per tile
    // Candidates staged in LDS by each wave for itself (no atomics, no
    // barriers).  A lane whose four scores of a block hold one that passes
    // stages all four and where they belong (7 bits of the wave's query, 25
    // bits of the row inside the chunk): a dozen instructions; which of them
    // pass is looked at when they are flushed.  Room for the 256
    // lanes of four query blocks above the level at which the waves flush.
    constexpr int CLIM = FILTER ? 112 : 0;
    constexpr int CCAP = FILTER ? CLIM + 64 * (QB < 4 ? QB : 4) : 1;
    constexpr int kRowBits = kSieveRowBits;
    __shared__ __align__(16) uint4 tiles[NBUF][BN * GR];
    __shared__ __align__(16) float side[NBUF][NSIDE > 0 ? NSIDE : 1][BN];
    __shared__ __align__(16) floatx4 cscore[FILTER ? S::WAVES : 1][CCAP];
    __shared__ uint32_t cmeta[FILTER ? S::WAVES : 1][CCAP];
    __shared__ float lthr[FILTER ? BQ : 1];
    __shared__ int flush_at;

    const int64_t logical = xcd_logical_id(blockIdx.x, (int64_t)args.nqb * args.nchunks);
    const int64_t chunk = logical / args.nqb;
    const int64_t q0 = (logical % args.nqb) * BQ;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int lane = lane_id();
    const int li = lane & 15, lh = lane >> 4;
    const int qg = wave & 3, rg = wave >> 2;
    // rows are counted from the chunk's first one (below 2^kSieveRowBits)
    const int64_t c0 = chunk * args.chunk_len;
    const int len = (int)(c0 + args.chunk_len < args.nb ? args.chunk_len : args.nb - c0);
    const int nsteps = len > 0 ? (len + BN - 1) / BN : 0;
    // (a split row is exactly its planes)
    const int row_bytes = PL > 1 ? GR * 16 : args.stride;
    const unsigned char* xb = static_cast<const unsigned char*>(args.xb) + c0 * row_bytes;

    // a row that the split cannot hold: every query is searched again
    if constexpr (PL > 1 && !SAMPLE)
        if (*args.bad_db != 0u) return;

    // ---- this wave's queries: operands, scale factors, thresholds
    uint4 qreg[QB][PL * S4];
    float mq[QB], sh[QB], thr[QB];
#pragma unroll
    for (int qb = 0; qb < QB; ++qb) {
        const int64_t q = q0 + (qg * QB + qb) * 16 + li;
        const bool ok = q < args.nq;
        const unsigned char* row =
            static_cast<const unsigned char*>(args.xq) + (ok ? q : 0) * (int64_t)row_bytes;
#pragma unroll
        for (int p = 0; p < PL; ++p)
#pragma unroll
            for (int s4 = 0; s4 < S4; ++s4) {
                const int c = 4 * s4 + lh;
                uint4 v = make_uint4(0, 0, 0, 0);
                // (the planes of a split row are whole; a low-precision row
                // may be shorter than DP)
                if (ok && (PL > 1 || c * 16 < args.stride))
                    v = *reinterpret_cast<const uint4*>(row + (p * S::GRP + c) * 16);
                qreg[qb][p * S4 + s4] = v;
            }
        const float inv = Op::SCALED && ok ? args.qscale[q] : 1.f;
        mq[qb] = (L2 ? -2.f : -1.f) * inv;
        sh[qb] = (!L2 && Op::SHIFTED && ok) ? -2.f * ERR * sqrtf(args.qnorm[q]) : 0.f;
        // (no query, or a threshold withdrawn: NaN, which lets no score through; below
        // -infinity comes the score of a row whose supplied norm is that)
        thr[qb] = (FILTER && ok) ? args.thr[q * args.thr_ld] : NAN;
        if constexpr (FILTER && PL > 1)
            if (ok && args.flags[q] != 0u) thr[qb] = NAN;
        // Queries without a chance of a proof: far from the origin the error bound of
        // the scores is more than the k-th best row and the threshold lie apart.  By the
        // sample's best `rank` scores (their number grows exponentially) these are about
        // ln(rank / (f k)) / ln(rank) of the best and the last of them apart, f the
        // sample's share of the rows; where that is less than the bound, no row is let
        // through and the finish finds too few.
        if constexpr (FILTER && L2 && PL > 1)
            if (ok) {
                const float* t = args.thr + q * args.thr_ld;
                if ((t[0] - t[1 - args.thr_ld]) * args.tail < 2.f * ERR * args.qnorm[q])
                    thr[qb] = NAN;
            }
        if (FILTER && rg == 0 && lh == 0) lthr[(qg * QB + qb) * 16 + li] = thr[qb];
    }
    if constexpr (FILTER && PL > 1) {
        // a block without a chance, or with few (the pass costs a fifth to a quarter of
        // what the fused search takes for its queries)
        __shared__ int chances;
        if (threadIdx.x == 0) chances = 0;
        __syncthreads();
        int mine = 0;
        if (rg == 0 && lh == 0)
#pragma unroll
            for (int qb = 0; qb < QB; ++qb) mine += thr[qb] == thr[qb] ? 1 : 0;
        if (mine) atomicAdd(&chances, mine);
        __syncthreads();
        if (5 * chances < (int)(args.nq - q0 < BQ ? args.nq - q0 : BQ)) return;
    }
    if (FILTER && threadIdx.x == 0) flush_at = -1;

    // ---- tile loads: row j, granule cc of load t of this lane
    auto granule_of = [&](int t, int& j, int& cc) __attribute__((always_inline)) {
        const int g = (wave + t * S::WAVES) * 64 + lane;
        j = g / GR;
        // the granule whose place is g % GR
        int c = g % GR;
        if constexpr (ROT) {
            c -= (j >> 1) & 3;
            c = c < 0 ? c + GR : c;
        } else {
            c = place(c, j);
        }
        // granules past a short row repeat granule 0 (they meet zero queries)
        cc = (PL > 1 || c * 16 < args.stride) ? c : 0;
    };
    // byte offsets inside a tile; where the loads of a lane are whole tile
    // rows apart with the same swizzle, one offset and constants
    constexpr int JT = 64 * S::WAVES / GR;  // rows between loads t and t + 1
    constexpr bool EVEN = PL > 1 && 64 * S::WAVES % GR == 0 && JT % (SW + 1) == 0;
    int32_t loff[EVEN ? 1 : LPW];
#pragma unroll
    for (int t = 0; t < (EVEN ? 1 : LPW); ++t) {
        int j, cc;
        granule_of(t, j, cc);
        loff[t] = (int32_t)(j * row_bytes + cc * 16);
    }
    // direct global-to-LDS loads from asm, as in the fused kernel: the
    // compiler does not see them, the explicit vmcnt waits below cover them
    // (scalar base, 32-bit lane offset)
    auto dma16 = [&](const unsigned char* base, int off, uint32_t m0) __attribute__((always_inline)) {
        asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1"
                     :
                     : "v"(off), "s"(base), "s"(m0)
                     : "memory", "m0");
    };
    auto dma4 = [&](const float* base, int off, uint32_t m0) __attribute__((always_inline)) {
        asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dword %0, %1"
                     :
                     : "v"(off), "s"(base), "s"(m0)
                     : "memory", "m0");
    };
    const uint32_t tiles_lds = (uint32_t)(uintptr_t)(lds_ptr_t)&tiles[0][0];
    const uint32_t side_lds = (uint32_t)(uintptr_t)(lds_ptr_t)&side[0][0][0];
    auto load_tile = [&](int t0, int buf) __attribute__((always_inline)) {
        const uint32_t base = tiles_lds + (uint32_t)(buf * BN * GR * 16 + wave * 64 * 16);
        const unsigned char* tile = xb + (int64_t)t0 * row_bytes;
        if (t0 + BN <= len) {
#pragma unroll
            for (int t = 0; t < LPW; ++t) {
                const uint32_t dst = base + (uint32_t)(t * S::WAVES * 64 * 16);
                if constexpr (EVEN)
                    dma16(tile + t * JT * GR * 16, loff[0], dst);
                else
                    dma16(tile, loff[t], dst);
            }
        } else {  // rows past the end repeat the last one
            const int last = len - 1 - t0;
#pragma unroll
            for (int t = 0; t < LPW; ++t) {
                int j, cc;
                granule_of(t, j, cc);
                j = j < last ? j : last;
                dma16(tile, j * row_bytes + cc * 16, base + (uint32_t)(t * S::WAVES * 64 * 16));
            }
        }
        if constexpr (NSIDE > 0) {
            if (wave < SIDE_OPS) {
                constexpr int PER = (BN + 63) / 64;
                const int a = wave / PER, part = wave % PER;
                const float* src = ((Op::SCALED && a == 0) ? args.ya : args.yb) + c0;
                const int last = len - 1 - t0;
                int j = part * 64 + lane;
                j = j < last ? j : last;
                const uint32_t dst = side_lds + (uint32_t)(((buf * NSIDE + a) * BN + part * 64) * 4);
                if (BN >= 64 || lane < BN) dma4(src + t0, j * 4, dst);
            }
        }
    };
    // at most the newest tile's loads of this wave outstanding
    auto wait_tile = [&]() __attribute__((always_inline)) {
        if (wave < SIDE_OPS)
            __builtin_amdgcn_s_waitcnt(waitcnt_vm<LPW + 1>());
        else
            __builtin_amdgcn_s_waitcnt(waitcnt_vm<LPW>());
    };
    auto step_barrier = [&]() __attribute__((always_inline)) {
        asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
    };
    // The staged candidates to their queries' pools, positions from the
    // queries' counters.  Stores may complete out of order with the tile
    // loads, so the wave then waits for everything (its tile waits count
    // loads only).
    // A query whose pool overflowed (ties by the thousand, a threshold that the
    // sample put too high) is searched again whatever else passes, so its threshold
    // is withdrawn, once per step (a flush is inlined in several places).
    uint32_t staged = 0;  // wave-uniform
    bool over = false;    // (as well) a pool overflowed
    auto withdraw = [&]() {
        over = false;
#pragma unroll
        for (int qb = 0; qb < QB; ++qb) {
            const int64_t q = q0 + (qg * QB + qb) * 16 + li;
            if (q < args.nq &&
                __hip_atomic_load(&args.cnt[q], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) > args.cap)
                thr[qb] = NAN;
        }
    };
    const int64_t qw0 = q0 + qg * QB * 16;
    auto flush = [&]() {
        __builtin_amdgcn_wave_barrier();
        bool full = false;
        constexpr int U = 2;  // counters asked at a time
#pragma unroll 1
        for (uint32_t e0 = 0; e0 < staged; e0 += 64 * U) {
            floatx4 c[U];
            uint32_t meta[U], take[U], pos[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const uint32_t i = e0 + u * 64 + lane;
                take[u] = 0u;
                pos[u] = 0u;
                meta[u] = 0u;
                c[u] = floatx4{0.f, 0.f, 0.f, 0.f};
                if (i < staged) {
                    c[u] = cscore[wave][i];
                    meta[u] = cmeta[wave][i];
                    const uint32_t ql = meta[u] >> kRowBits;
                    const int row = (int)(meta[u] & ((1u << kRowBits) - 1u));
                    const float t = lthr[qg * QB * 16 + ql];
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        take[u] |= (c[u][e] <= t && row + e < len) ? 1u << e : 0u;
                    if (take[u]) pos[u] = atomicAdd(&args.cnt[qw0 + ql], (uint32_t)__popc(take[u]));
                }
            }
#pragma unroll
            for (int u = 0; u < U; ++u) {
                uint64_t* p = args.pool + (qw0 + (meta[u] >> kRowBits)) * args.cap;
                const uint32_t row =
                    args.row0 + (uint32_t)c0 + (meta[u] & ((1u << kRowBits) - 1u));
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    if (take[u] & (1u << e)) {
                        if (pos[u] < args.cap) p[pos[u]] = make_key(c[u][e], row + e);
                        ++pos[u];
                    }
                full |= take[u] != 0u && pos[u] > args.cap;
            }
        }
        staged = 0;
        over |= __ballot(full) != 0;
        __builtin_amdgcn_s_waitcnt(0);
    };

    __builtin_amdgcn_s_waitcnt(0);
    if (nsteps > 0) load_tile(0, 0);
    if (nsteps > 1) load_tile(BN, 1);
    if (nsteps > 1)
        wait_tile();
    else
        __builtin_amdgcn_s_waitcnt(0);
    __syncthreads();

    // Scores of one 16-row block from its dot products, tested against the
    // thresholds (lane = query li of each 16, register i = row + i).
    auto scores_of = [&](const floatx4 (&acc)[QB], floatx4 av, floatx4 bv, float (&sc)[QB][4])
                         __attribute__((always_inline)) {
#pragma unroll
        for (int qb = 0; qb < QB; ++qb)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                float v = acc[qb][i];
                if constexpr (Op::SCALED) v *= av[i];
                if constexpr (L2)
                    sc[qb][i] = fmaf(v, mq[qb], bv[i]);
                else if constexpr (Op::SHIFTED)
                    sc[qb][i] = fmaf(bv[i], sh[qb], v * mq[qb]);
                else if constexpr (Op::SCALED)
                    sc[qb][i] = v * mq[qb];
                else
                    sc[qb][i] = v;  // negated where it is used (RAW)
            }
    };
    constexpr bool RAW = !L2 && !Op::SCALED;  // scores are -sc
    float least[QB];  // SAMPLE: of this step's rows
#pragma unroll
    for (int qb = 0; qb < QB; ++qb) least[qb] = INFINITY;
    Nearest best[NEAREST ? QB : 1];
#pragma unroll
    for (int qb = 0; qb < (NEAREST ? QB : 1); ++qb) best[qb].init();
    auto emit = [&](float (&sc)[QB][4], int row) __attribute__((always_inline)) {
        if constexpr (SAMPLE) {
#pragma unroll
            for (int qb = 0; qb < QB; ++qb) {
                float m = RAW ? -fmaxf(fmaxf(sc[qb][0], sc[qb][1]), fmaxf(sc[qb][2], sc[qb][3]))
                              : fminf(fminf(sc[qb][0], sc[qb][1]), fminf(sc[qb][2], sc[qb][3]));
                least[qb] = fminf(least[qb], m);
            }
        } else if constexpr (NEAREST) {
            if (row - 4 * lh + 16 > len) {  // (wave-uniform) rows past the end
#pragma unroll
                for (int qb = 0; qb < QB; ++qb)
#pragma unroll
                    for (int i = 0; i < 4; ++i)
                        if (row + i >= len) sc[qb][i] = INFINITY;
            }
#pragma unroll
            for (int qb = 0; qb < QB; ++qb)
                best[qb].offer(fminf(fminf(sc[qb][0], sc[qb][1]), fminf(sc[qb][2], sc[qb][3])),
                               (uint32_t)row >> 2);
        } else {
            // (room for every lane of the block: see the flush below)
#pragma unroll
            for (int qb = 0; qb < QB; ++qb) {
                bool take;
                if constexpr (RAW)
                    take = fmaxf(fmaxf(sc[qb][0], sc[qb][1]), fmaxf(sc[qb][2], sc[qb][3])) >= -thr[qb];
                else
                    take = fminf(fminf(sc[qb][0], sc[qb][1]), fminf(sc[qb][2], sc[qb][3])) <= thr[qb];
                const uint64_t bal = __ballot(take);
                if (bal) {
                    if (take) {
                        const uint32_t pos =
                            staged + __builtin_amdgcn_mbcnt_hi(
                                         (uint32_t)(bal >> 32),
                                         __builtin_amdgcn_mbcnt_lo((uint32_t)bal, 0u));
                        floatx4 v = {sc[qb][0], sc[qb][1], sc[qb][2], sc[qb][3]};
                        if constexpr (RAW) v = -v;
                        cscore[wave][pos] = v;
                        cmeta[wave][pos] =
                            ((uint32_t)(qb * 16 + li) << kRowBits) | (uint32_t)row;
                    }
                    staged += (uint32_t)__popcll(bal);
                }
                if ((qb & 3) == 3 || qb == QB - 1)
                    if (staged > CLIM) flush();
            }
        }
    };

    // Blocks are software-pipelined: the scores of one block (vector ALU) are
    // computed between the matrix products of the next, which leave three
    // issue slots of four free; the first block of the loop tests an empty
    // predecessor (row len: every row past the end).  Not where the operands of
    // one block leave no registers for it.
    constexpr bool PIPE = FILTER && PL * S4 * (QB + 1) * 4 <= 160;
    constexpr int VPM = Op::MMAS == 3 ? 2 : 4;  // vector operations per product
    floatx4 prev[QB];
#pragma unroll
    for (int qb = 0; qb < QB; ++qb) prev[qb] = floatx4{0.f, 0.f, 0.f, 0.f};
    floatx4 pav = floatx4{0.f, 0.f, 0.f, 0.f}, pbv = floatx4{INFINITY, INFINITY, INFINITY, INFINITY};
    int prow = len;
    int buf = 0;
#pragma unroll 1
    for (int s = 0; s < nsteps; ++s) {
        const int t0 = s * BN;
        const bool issue = s + 2 < nsteps;
        if (issue) load_tile(t0 + 2 * BN, buf >= 1 ? buf - 1 : NBUF - 1);
#pragma unroll
        for (int rb = 0; rb < RBW; ++rb) {
            const int r0 = (rg * RBW + rb) * 16;
            const uint4* bt = &tiles[buf][(r0 + li) * GR];
            uint4 b[PL * S4];
#pragma unroll
            for (int p = 0; p < PL; ++p)
#pragma unroll
                for (int s4 = 0; s4 < S4; ++s4)
                    b[p * S4 + s4] = bt[place(p * S::GRP + 4 * s4 + lh, li)];
            floatx4 av{}, bv{};
            if constexpr (Op::SCALED)
                av = *reinterpret_cast<const floatx4*>(&side[buf][0][r0 + 4 * lh]);
            if constexpr (HASB)
                bv = *reinterpret_cast<const floatx4*>(&side[buf][NSIDE - 1][r0 + 4 * lh]);
            floatx4 acc[QB];
#pragma unroll
            for (int qb = 0; qb < QB; ++qb) acc[qb] = floatx4{0.f, 0.f, 0.f, 0.f};
            float sc[QB][4];
            if constexpr (PIPE) scores_of(prev, pav, pbv, sc);
#pragma unroll
            for (int s4 = 0; s4 < S4; ++s4)
#pragma unroll
                for (int qb = 0; qb < QB; ++qb)
                    acc[qb] = Op::template mma<S4>(acc[qb], b, qreg[qb], s4);
            if constexpr (!PIPE) {
                scores_of(acc, av, bv, sc);
                emit(sc, t0 + r0 + 4 * lh);
                continue;
            }
#pragma unroll
            for (int t = 0; t < S4 * QB * Op::MMAS; ++t) {
                __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);  // one matrix product
                __builtin_amdgcn_sched_group_barrier(0x002, VPM, 0);  // vector operations
            }
            emit(sc, prow);
            prow = t0 + r0 + 4 * lh;
            pav = av;
            pbv = bv;
#pragma unroll
            for (int qb = 0; qb < QB; ++qb) prev[qb] = acc[qb];
        }
        if constexpr (SAMPLE) {
            // (a batch has 2^28 entries at most: 32-bit places from one register; 64-bit
            // ones were spilled: FP8 sample of 3,000 queries 44.4 us, 39.8 so)
            const uint32_t ld = (uint32_t)args.ld, step = (uint32_t)(c0 / BN) + (uint32_t)s;
            const uint32_t at = (uint32_t)(q0 + qg * QB * 16 + li) * ld + (uint32_t)(rg * 4 + lh);
#pragma unroll
            for (int qb = 0; qb < QB; ++qb) {
                const int64_t q = q0 + (qg * QB + qb) * 16 + li;
                if (q < args.nq) args.scores[at + (uint32_t)(qb * 16) * ld + step * (4 * S::RG)] = least[qb];
                least[qb] = INFINITY;
            }
        }
        // the next tile has landed (stores: wait for everything, as above)
        if (!issue || SAMPLE)
            __builtin_amdgcn_s_waitcnt(0);
        else
            wait_tile();
        // waves flush together, before the fullest has to: one wave's flush
        // would hold the others up at the next barrier all the same
        if (FILTER && staged > CLIM * 3 / 4 && lane == 0) flush_at = s;
        step_barrier();
        if (FILTER && staged && *(volatile int*)&flush_at == s) flush();
        if (FILTER && over) withdraw();
        buf = buf + 1 < NBUF ? buf + 1 : 0;
    }
    if (PIPE && nsteps > 0) {
        float sc[QB][4];
        scores_of(prev, pav, pbv, sc);
        emit(sc, prow);
    }
    if constexpr (FILTER)
        if (staged) flush();
    if constexpr (NEAREST) {
        // the four lanes of a query, then the two row groups (through the
        // tile buffers, which the last barrier has freed)
        Nearest* other = reinterpret_cast<Nearest*>(&tiles[0][0]);
#pragma unroll
        for (int qb = 0; qb < QB; ++qb) {
#pragma unroll
            for (int o = 16; o <= 32; o <<= 1) {
                Nearest x;
                x.b1 = __shfl_xor(best[qb].b1, o);
                x.b2 = __shfl_xor(best[qb].b2, o);
                x.b3 = __shfl_xor(best[qb].b3, o);
                x.g1 = (uint32_t)__shfl_xor((int)best[qb].g1, o);
                x.g2 = (uint32_t)__shfl_xor((int)best[qb].g2, o);
                best[qb].merge(x);
            }
            if (rg == 1 && lh == 0) other[(qg * QB + qb) * 16 + li] = best[qb];
        }
        __syncthreads();
        if (rg == 0) {
#pragma unroll
            for (int qb = 0; qb < QB; ++qb) {
                const int ql = (qg * QB + qb) * 16 + li;
                best[qb].merge(other[ql]);
                if (lh == 0 && q0 + ql < args.nq)
                    args.near[q0 + ql] =
                        make_uint4(best[qb].g1, best[qb].g2, __float_as_uint(best[qb].b2),
                                   __float_as_uint(best[qb].b3));
            }
        }
    }
}

// ------------------------------------------------------- FP16 pair rows
// Row i of a stratified sample of n out of nb rows (n a power of two): one row of each
// of n equal strata, at a hashed place inside it (no period of the data lines up with
// it).  Rows that are neighbours in the sample, whose least score is kept, come from
// strata far apart: of rows in the order of their clusters all eight behind an entry
// were of one cluster, the threshold fell outside it and its rows overflowed the pool
// (2,000 queries, 10^6 x 128 rows in the order of 200 clusters, k = 100: 8.9 ms, now 1.5).
__device__ __forceinline__ int64_t sample_row(int64_t i, int64_t n, int64_t nb) {
    const int64_t at = (int64_t)((uint64_t)i * 2654435761ull & (uint64_t)(n - 1));
    const int64_t lo = at * nb / n, hi = (at + 1) * nb / n;
    uint64_t h = (uint64_t)(i + 1) * 0x9E3779B97F4A7C15ull;
    h ^= h >> 29;
    h *= 0xBF58476D1CE4E5B9ull;
    h ^= h >> 32;
    return lo + (int64_t)(h % (uint64_t)(hi - lo));
}

constexpr int kCenterRows = 32, kCenterOn = 256;  // (see sieve_clear_kernel)

// Rows of d floats as two FP16 planes of DP elements (zero padded): x 2^p =
// h + l, p the row's own power of two with max |x| 2^p in [2^13, 2^14).  With a
// center (L2) x stands for the row less it, here and in all scores and bounds, which
// are relative to ||x||^2 + ||y||^2: distances stay the same, and rows far from the
// origin need not be far from the center (10^4 queries, 10^6 x 128 rows, 130
// standard deviations from the origin, k = 100: 19.9 ms without, 6.2 with it).
//   scale[i] = 2^-p;
//   off[i]: DB rows, L2: ||y||^2 (1 - split_err); DB rows, inner product: ||y||;
//   queries: ||x||^2;
//   raw[i] (if given): the row's own squared norm.
// Supplied norms yn: a row whose norm is infinite or NaN has no score; one that is
// not the row's norm counts by what it differs.
// A row that is not finite, or so large or small that scales and squares could
// leave the normal range, raises *bad for database rows, bad[i] for queries.
enum SplitKind { kSplitDbL2 = 0, kSplitDbIp = 1, kSplitQuery = 2 };
template <int DP>
__global__ __launch_bounds__(256) void split_rows_kernel(
    const float* __restrict__ x, int64_t n, int32_t d, int32_t vec, int32_t kind,
    const float* __restrict__ yn, const float* __restrict__ center, int64_t sample_of,
    unsigned char* __restrict__ out, float* __restrict__ scale, float* __restrict__ off,
    float* __restrict__ raw, uint32_t* __restrict__ bad) {
    constexpr int GRP = DP / 8;
    constexpr int LPR = GRP >= 16 ? 16 : GRP > 8 ? 16 : GRP;  // lanes per row
    constexpr int NG = (GRP + LPR - 1) / LPR;                 // granules per lane
    const int lane = threadIdx.x & 63;
    const int sub = lane % LPR;
    const int64_t rows_per_wave = 64 / LPR;
    const int64_t w0 = ((int64_t)blockIdx.x * 256 + threadIdx.x) >> 6;
    const int64_t nw = (int64_t)gridDim.x * 4;
    const bool centered = center && center[kCenterOn] != 0.f;
    // this lane's components of the center (kept in registers where these allow as many
    // waves with them)
    auto middle = [&](int t) __attribute__((always_inline)) {
        return centered && t < d ? center[t] : 0.f;
    };
    float mid[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) mid[e] = NG == 1 ? middle(sub * 8 + e) : 0.f;
    for (int64_t r0 = w0 * rows_per_wave; r0 < n; r0 += nw * rows_per_wave) {
        const int64_t i = r0 + lane / LPR;
        const bool live = i < n;
        const int64_t src = !live ? 0 : sample_of > 0 ? sample_row(i, n, sample_of) : i;
        const float* p = x + src * d;
        float v[NG][8];
        float m = 0.f, ss = 0.f, own = 0.f;
#pragma unroll
        for (int g = 0; g < NG; ++g) {
            const int e0 = (g * LPR + sub) * 8;
            if (vec) {
                float4 a = make_float4(0.f, 0.f, 0.f, 0.f), b = a;
                if (live && e0 < d) a = *reinterpret_cast<const float4*>(p + e0);
                if (live && e0 + 4 < d) b = *reinterpret_cast<const float4*>(p + e0 + 4);
                v[g][0] = a.x; v[g][1] = a.y; v[g][2] = a.z; v[g][3] = a.w;
                v[g][4] = b.x; v[g][5] = b.y; v[g][6] = b.z; v[g][7] = b.w;
            } else {
#pragma unroll
                for (int e = 0; e < 8; ++e) v[g][e] = (live && e0 + e < d) ? p[e0 + e] : 0.f;
            }
            if (centered)
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    own = fmaf(v[g][e], v[g][e], own);
                    v[g][e] -= NG == 1 ? mid[e] : middle(e0 + e);
                }
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                m = fmaxf(m, fabsf(v[g][e]));
                ss = fmaf(v[g][e], v[g][e], ss);
            }
        }
#pragma unroll
        for (int o = LPR / 2; o >= 1; o >>= 1) {
            m = fmaxf(m, __shfl_xor(m, o, LPR));
            ss += __shfl_xor(ss, o, LPR);
        }
        if (centered) {
#pragma unroll
            for (int o = LPR / 2; o >= 1; o >>= 1) own += __shfl_xor(own, o, LPR);
        } else {
            own = ss;
        }
        // (a NaN element leaves m alone but not the sum of squares)
        const bool fine = ss == 0.f ? m == 0.f : (m >= 0x1p-50f && m < 0x1p50f && ss < 0x1p110f);
        int ex = 0;
        if (fine && m > 0.f) ex = 13 - ((int)((__float_as_uint(m) >> 23) & 0xFF) - 127);
        const float up = __uint_as_float((uint32_t)(127 + ex) << 23);
        const float dn = __uint_as_float((uint32_t)(127 - ex) << 23);
        if (live) {
#pragma unroll
            for (int g = 0; g < NG; ++g) {
                if (g * LPR + sub >= GRP) continue;
                half8 h, l;
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    const float xs = fine ? v[g][e] * up : 0.f;
                    const _Float16 hh = (_Float16)xs;
                    h[e] = hh;
                    l[e] = (_Float16)(xs - (float)hh);
                }
                unsigned char* o = out + i * (int64_t)(DP * 4) + (g * LPR + sub) * 16;
                *reinterpret_cast<half8*>(o) = h;
                *reinterpret_cast<half8*>(o + DP * 2) = l;
            }
            if (sub == 0) {
                scale[i] = dn;
                if (raw) raw[i] = own;
                float of = ss;
                if (kind == kSplitDbL2) {
                    of *= 1.f - split_err(DP);
                    if (yn) {
                        const float y = yn[src], more = y - own;
                        if (!(fabsf(y) < INFINITY))
                            of = y;
                        else if (fabsf(more) > 0x1p-16f * own)
                            of += more - split_err(DP) * fabsf(more);
                    }
                } else if (kind == kSplitDbIp) {
                    of = sqrtf(ss);
                }
                off[i] = of;
                if (!fine) {
                    if (kind == kSplitQuery)
                        bad[i] = 1u;
                    else
                        *bad = 1u;
                }
            }
        }
    }
}

// Gather of a stratified sample of low-precision rows (16-byte granules) and
// their side values (either may be null).
static __global__ void sample_rows_kernel(const unsigned char* __restrict__ xb, int32_t stride,
                                          int64_t n, int64_t nb, const float* __restrict__ a,
                                          const float* __restrict__ b,
                                          unsigned char* __restrict__ out, float* __restrict__ oa,
                                          float* __restrict__ ob) {
    const int32_t gr = stride / 16;
    const int64_t g = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (g >= n * gr) return;
    const int64_t i = g / gr;
    const int32_t c = (int32_t)(g % gr);
    const int64_t src = sample_row(i, n, nb);
    reinterpret_cast<uint4*>(out + i * stride)[c] =
        reinterpret_cast<const uint4*>(xb + src * stride)[c];
    if (c == 0) {
        if (a) oa[i] = a[src];
        if (b) ob[i] = b[src];
    }
}

// Clears n words; with a center (a workgroup more) also takes the mean of 32 rows, as a
// point that is near the rows for their distances.  center[0 .. d), center[kCenterOn]:
// whether rows are to be taken less it: not where it is out of the split's range, nor
// where the rows are less than 8 deviations from the origin (proofs succeed there without
// it -- they did at 10 deviations at every size measured and failed from 30 on -- and the
// split is bound by vector operations too: 167 queries, 681,348 x 236 rows 668 us with
// the center, 630 without).
static __global__ __launch_bounds__(256) void sieve_clear_kernel(uint32_t* __restrict__ p, int64_t n,
                                                                const float* __restrict__ xb,
                                                                int64_t nb, int32_t d,
                                                                float* __restrict__ center) {
    const int64_t blocks = gridDim.x - (center ? 1 : 0);
    if ((int64_t)blockIdx.x == blocks) {
        __shared__ float part[2][4];
        const int t = threadIdx.x;
        const int rows = nb < kCenterRows ? (int)nb : kCenterRows;
        float v[kCenterRows], mean = 0.f, squares = 0.f;
#pragma unroll
        for (int i = 0; i < kCenterRows; ++i)
            v[i] = i < rows && t < d ? xb[(i * nb / kCenterRows) * d + t] : 0.f;
#pragma unroll
        for (int i = 0; i < kCenterRows; ++i) {
            mean += v[i];
            squares = fmaf(v[i], v[i], squares);
        }
        mean /= (float)rows;
        squares /= (float)rows;
        float own = mean * mean;
        // (one component out of range spoils the sum)
        if (!(fabsf(mean) < 0x1p50f)) own = NAN;
#pragma unroll
        for (int o = 1; o < 64; o *= 2) {
            own += __shfl_xor(own, o);
            squares += __shfl_xor(squares, o);
        }
        if ((t & 63) == 0) {
            part[0][t >> 6] = own;
            part[1][t >> 6] = squares;
        }
        __syncthreads();
        own = part[0][0] + part[0][1] + part[0][2] + part[0][3];
        squares = part[1][0] + part[1][1] + part[1][2] + part[1][3];
        if (t < d) center[t] = mean;
        if (t == 0) center[kCenterOn] = own * 64.f >= squares * 63.f ? 1.f : 0.f;
        return;
    }
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += blocks * 256) p[i] = 0u;
}
inline mk_status sieve_clear(uint32_t* p, int64_t n, const float* xb, int64_t nb, int32_t d,
                             float* center, hipStream_t s) {
    const int64_t blocks = ceil_div(n, 256);
    hipLaunchKernelGGL(sieve_clear_kernel, dim3((unsigned)((blocks < 1024 ? blocks : 1024) + (center ? 1 : 0))),
                       dim3(256), 0, s, p, n, xb, nb, d, center);
    MK_LAUNCHED();
    return MK_OK;
}

// ------------------------------------------------------------- finish
// What the direct-form value (squared distance, or negated inner product) of a row
// is at least, by its score in a pool: the scores are lower bounds of rows' true
// scores less the per-query constant err ||x||^2 (L2; err: split_err).
__device__ __forceinline__ float row_bound(float score, float nx, float err, int32_t l2) {
    return l2 ? (nx * (1.f - err) + score) * (1.f - kDirectErr) : score;
}

// Query q to the list of those that the fused search takes.
__device__ __forceinline__ void leave_query(int64_t q, uint32_t* __restrict__ rest,
                                            uint32_t* __restrict__ nrest) {
    rest[atomicAdd(nrest, 1u)] = (uint32_t)q;
}

// One workgroup per query: the keff best keys of its pool (pool.hpp), re-ranked in
// the direct FP32 form, the k best written.  A query without a proven
// result (pool overflowed or short, values the split cannot hold, or, with cert, a
// dropped row's lower bound does not clear the k-th distance) is left to the fused
// search.
//
// cert: a row of the pool that is not among the keff best has at least the keff-th
// best score, a row outside the pool at least the threshold.  When the k-th
// re-ranked value is below the bound (row_bound) of the former, no other row can
// enter.  When it is only below the bound of the latter (rows far from the origin
// for their distances, ties), the pool's other rows whose bound is not cleared are
// re-ranked as well.
// 2,000 queries, keff = 1,016, pools of about 2,500 keys: 210 us against 330 us by a
// wave per query with a sorted register queue; 10^4 queries, keff = 400: 284 against
// 450 us.  Bound by the gathers of the re-ranked rows (4.8 TB/s and 5.4 TB/s).
// The registers are held to what the first round needs (the second one, in its place or
// spilled, cost 10^4 queries with keff = 116 / 1,016 50 / 72 us more by fewer waves).
template <int P>  // keff <= P / 2
__global__ __launch_bounds__(kPoolThreads)
__attribute__((amdgpu_waves_per_eu(P == 1024 ? 8 : P == 2048 ? 5 : 4))) void sieve_finish(
    const uint64_t* __restrict__ pools, const uint32_t* __restrict__ cnt, uint32_t cap,
    const float* __restrict__ thr, int64_t thr_ld,
    const float* __restrict__ xq, const float* __restrict__ xb, int32_t d, int32_t vec,
    int32_t l2, int32_t k, int32_t keff, int32_t cert, float err, const float* __restrict__ qnorm,
    const uint32_t* __restrict__ bad_db, const uint32_t* __restrict__ flags,
    uint32_t* __restrict__ rest, uint32_t* __restrict__ nrest, float* __restrict__ D,
    int64_t* __restrict__ I) {
    __shared__ uint64_t pool[P];
    __shared__ __align__(8) uint32_t bins[kCutBins];
    __shared__ PoolState st;
    __shared__ __align__(16) float xs[kMaxDim];
    __shared__ float dist[P / 2];
    const int tid = threadIdx.x;
    const int64_t q = blockIdx.x;
    const uint32_t n = cnt[q];
    // (with cert some key has to be dropped for the bound to come from)
    if (n > cap || n < (uint32_t)(keff + (cert ? 1 : 0)) || flags[q] != 0u ||
        (bad_db && *bad_db != 0u)) {
        if (tid == 0) leave_query(q, rest, nrest);
        return;
    }
    for (int t = tid; t < d; t += kPoolThreads) xs[t] = xq[q * d + t];
    uint64_t limit;
    (void)pool_stream<P>(pools + q * (int64_t)cap, n, pool, bins, &st, keff, limit);
    __syncthreads();
#pragma unroll 1
    for (int e0 = 16 * (tid >> 6); e0 < keff; e0 += 16 * kPoolWaves)
        rerank_rows16(xs, pool, e0, keff, xb, d, vec, l2, dist);
    __syncthreads();
    for (int e = tid; e < keff; e += kPoolThreads)
        pool[e] = make_key(l2 ? dist[e] : -dist[e], key_index(pool[e]));
    uint32_t left = (uint32_t)keff;
    if (cert) {
        pool_cut<P>(pool, bins, &st, left, k);
        left = (uint32_t)k;
        const float worst = key_score(st.limit - 1), s_last = key_score(limit - 1), nx = qnorm[q];
        if (!(worst < row_bound(s_last, nx, err, l2))) {  // (uniform)
            if (!(worst < row_bound(thr[q * thr_ld], nx, err, l2))) {
                if (tid == 0) leave_query(q, rest, nrest);
                return;
            }
            // the rest of the pool's rows whose bound does not clear the k-th
            uint64_t* strip = reinterpret_cast<uint64_t*>(bins);  // (free between cuts)
            uint64_t enter = st.limit;
#pragma unroll 1
            for (uint32_t e0 = 0; e0 < n; e0 += kPoolThreads) {
                uint64_t key = e0 + tid < n ? pools[q * (int64_t)cap + e0 + tid] : kSentinel;
                if (key < limit || !(row_bound(key_score(key), nx, err, l2) <= worst)) key = kSentinel;
                if (!__syncthreads_or(key != kSentinel)) continue;
                strip[tid] = key;
                __syncthreads();
#pragma unroll 1
                for (int e = 16 * (tid >> 6); e < kPoolThreads; e += 16 * kPoolWaves)
                    rerank_rows16(xs, strip, e, kPoolThreads, xb, d, vec, l2, dist);
                __syncthreads();
                const uint64_t nk =
                    key != kSentinel ? make_key(l2 ? dist[tid] : -dist[tid], key_index(key)) : kSentinel;
                const bool take = nk < enter;
                uint32_t at;
                const uint32_t add = pool_sum(take ? 1u : 0u, st.wsum, at);
                if (take) pool[left + at] = nk;
                left += add;
                if (left > (uint32_t)(P - kPoolThreads)) {
                    pool_cut<P>(pool, bins, &st, left, k);
                    left = (uint32_t)k;
                    enter = st.limit;
                }
                __syncthreads();
            }
        }
    }
    pool_emit<P>(pool, bins, &st, left, (uint32_t)k, [&](uint32_t r, uint64_t key) {
        const float s = key_score(key);
        D[q * k + r] = l2 ? s : -s;
        I[q * k + r] = (int64_t)key_index(key);
    });
}

// The same with one wave per query and a sorted register queue, for keff <= 64: no
// barriers, and a queue of one key per lane is cheap (10^4 queries, keff = 48: 60 us
// against 104 by a workgroup each).
static __global__ __launch_bounds__(64 * kMergeWaves) void sieve_finish_wave(
    const uint64_t* __restrict__ pool, const uint32_t* __restrict__ cnt, uint32_t cap,
    const float* __restrict__ thr, int64_t thr_ld, const float* __restrict__ xq, int64_t nq, const float* __restrict__ xb, int32_t d, int32_t vec,
    int32_t l2, int32_t k, int32_t keff, int32_t cert, float err, const float* __restrict__ qnorm,
    const uint32_t* __restrict__ bad_db, const uint32_t* __restrict__ flags,
    uint32_t* __restrict__ rest, uint32_t* __restrict__ nrest, float* __restrict__ D,
    int64_t* __restrict__ I) {
    constexpr int KR = 1, T = SelParams<KR>::T, KS = 64 * KR;
    __shared__ __align__(16) float xs[kMergeWaves][kMaxDim];
    __shared__ uint64_t kl[kMergeWaves][KS];
    __shared__ float dist[kMergeWaves][KS];
    const int wave = threadIdx.x >> 6;
    const int lane = lane_id();
    const int64_t q = (int64_t)blockIdx.x * kMergeWaves + wave;
    if (q >= nq) return;
    const uint32_t n = cnt[q];
    if (n > cap || n < (uint32_t)(keff + (cert ? 1 : 0)) || flags[q] != 0u ||
        (bad_db && *bad_db != 0u)) {
        if (lane == 0) leave_query(q, rest, nrest);
        return;
    }
    WaveSelect<KR, T> ws;
    ws.init(keff);
    const uint64_t* p = pool + q * (int64_t)cap;
#pragma unroll 1
    for (uint32_t e = 0; e < n; e += 64) {
        const uint32_t i = e + lane;
        if (ws.push(i < n ? p[i] : kSentinel)) ws.merge();
    }
    ws.finish();
    const uint64_t last = ws_element<KR>(ws.w, keff - 1);

    const float* x = xq + q * d;
    for (int t = lane; t < d; t += 64) xs[wave][t] = x[t];
#pragma unroll
    for (int r = 0; r < KR; ++r) kl[wave][r * 64 + lane] = ws.w[r];
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "workgroup");
    const float* xw = xs[wave];
#pragma unroll 1
    for (int e0 = 0; e0 < keff; e0 += 16)
        rerank_rows16(xw, kl[wave], e0, keff, xb, d, vec, l2, dist[wave]);
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "workgroup");
    uint64_t nk[KR];
#pragma unroll
    for (int r = 0; r < KR; ++r) {
        const uint64_t key = ws.w[r];
        const int e = r * 64 + lane;
        nk[r] = kSentinel;
        if (key != kSentinel && e < keff) {
            const float sv = dist[wave][e];
            nk[r] = make_key(l2 ? sv : -sv, key_index(key));
        }
    }
    bitonic_sort<false, KR>(nk);
    if (cert) {
        const float worst = key_score(ws_element<KR>(nk, k - 1));
        const float nx = qnorm[q];
        if (!(worst < row_bound(key_score(last), nx, err, l2))) {
            if (!(worst < row_bound(thr[q * thr_ld], nx, err, l2))) {
                if (lane == 0) leave_query(q, rest, nrest);
                return;
            }
            // the rest of the pool's rows whose bound does not clear the k-th
            ws.init(k);
            if (ws.push(nk[0])) ws.merge();
#pragma unroll 1
            for (uint32_t e0 = 0; e0 < n; e0 += 64) {
                uint64_t key = e0 + lane < n ? p[e0 + lane] : kSentinel;
                if (key <= last || !(row_bound(key_score(key), nx, err, l2) <= worst)) key = kSentinel;
                if (!__ballot(key != kSentinel)) continue;
                kl[wave][lane] = key;
                __builtin_amdgcn_wave_barrier();
                __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "workgroup");
#pragma unroll 1
                for (int e = 0; e < 64; e += 16)
                    rerank_rows16(xw, kl[wave], e, 64, xb, d, vec, l2, dist[wave]);
                __builtin_amdgcn_wave_barrier();
                __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "workgroup");
                const float v = dist[wave][lane];
                if (ws.push(key != kSentinel ? make_key(l2 ? v : -v, key_index(key)) : kSentinel))
                    ws.merge();
                __builtin_amdgcn_wave_barrier();
            }
            ws.finish();
            nk[0] = ws.w[0];
        }
    }
    emit_reranked<KR>(nk, k, l2, D + q * k, I + q * k);
}

// Nearest row of each query from kNearest's groups (L2): the rows of the best
// group, in the direct form, and those of the second only when the first
// distance does not clear its score; flagged when the rest's bound is not
// cleared either (the bound: see sieve_finish).  Rows that the supplied norms yn
// (or null) leave out are no candidates, as they had no score.  16 lanes per row as
// in rerank_rows16, so the same distances; a wave does four queries at a time.
static __global__ __launch_bounds__(256) void nearest_finish(
    const uint4* __restrict__ near, const float* __restrict__ xq, int64_t nq,
    const float* __restrict__ xb, const float* __restrict__ yn, int32_t nb, int32_t d, int32_t vec,
    float err, const float* __restrict__ qnorm, const uint32_t* __restrict__ bad_db,
    const uint32_t* __restrict__ flags, uint32_t* __restrict__ rest, uint32_t* __restrict__ nrest,
    float* __restrict__ D, int64_t* __restrict__ I) {
    constexpr int NQ = 4;
    __shared__ uint32_t leaving[4], first_place;
    const int lane = lane_id(), sub = lane & 15, rsel = lane >> 4;
    const int64_t w = ((int64_t)blockIdx.x * 256 + threadIdx.x) >> 6;
    const int64_t q0 = w * NQ;  // (a wave without queries goes along, on query nq - 1's data)
    // distances of the four rows of group g[p] to query q0 + p, as keys; the
    // least of the four in every lane
    auto group_best = [&](const uint32_t (&g)[NQ], uint64_t (&key)[NQ]) __attribute__((always_inline)) {
        float acc[NQ];
        const float *x[NQ], *y[NQ];
        bool live[NQ];
#pragma unroll
        for (int p = 0; p < NQ; ++p) {
            const int64_t row = (int64_t)g[p] * 4 + rsel;
            live[p] = q0 + p < nq && row < nb && has_score(yn, xb, row, d);
            x[p] = xq + (q0 + p < nq ? q0 + p : nq - 1) * d;
            y[p] = xb + (live[p] ? row : 0) * d;
            acc[p] = 0.f;
        }
        if (vec) {
            for (int t = 4 * sub; t < d; t += 64) {
                float4 a[NQ], b[NQ];
#pragma unroll
                for (int p = 0; p < NQ; ++p) {
                    a[p] = *reinterpret_cast<const float4*>(x[p] + t);
                    b[p] = *reinterpret_cast<const float4*>(y[p] + t);
                }
#pragma unroll
                for (int p = 0; p < NQ; ++p) {
                    const float e0 = a[p].x - b[p].x, e1 = a[p].y - b[p].y, e2 = a[p].z - b[p].z,
                                e3 = a[p].w - b[p].w;
                    acc[p] = fmaf(e0, e0, acc[p]);
                    acc[p] = fmaf(e1, e1, acc[p]);
                    acc[p] = fmaf(e2, e2, acc[p]);
                    acc[p] = fmaf(e3, e3, acc[p]);
                }
            }
        } else {
            for (int t = sub; t < d; t += 16) {
#pragma unroll
                for (int p = 0; p < NQ; ++p) {
                    const float e = x[p][t] - y[p][t];
                    acc[p] = fmaf(e, e, acc[p]);
                }
            }
        }
#pragma unroll
        for (int p = 0; p < NQ; ++p) {
            float v = acc[p];
#pragma unroll
            for (int o = 8; o >= 1; o >>= 1) v += __shfl_xor(v, o, 16);
            uint64_t k = live[p] ? make_key(v, g[p] * 4u + (uint32_t)rsel) : kSentinel;
            k = umin64(k, xor_lane64<16>(k));
            key[p] = umin64(k, xor_lane64<32>(k));
        }
    };
    uint4 c[NQ];
    uint32_t g[NQ];
    uint64_t key[NQ];
    bool bad[NQ], more = false;
    float edge[NQ];
#pragma unroll
    for (int p = 0; p < NQ; ++p) {
        const int64_t q = q0 + p < nq ? q0 + p : nq - 1;
        c[p] = near[q];
        g[p] = c[p].x;
        const float nx = qnorm[q];
        edge[p] = nx * (1.f - err);
        bad[p] = flags[q] != 0u || *bad_db != 0u;
    }
    group_best(g, key);
    uint32_t g2[NQ];
#pragma unroll
    for (int p = 0; p < NQ; ++p) {
        const float s = fminf(__uint_as_float(c[p].z), __uint_as_float(c[p].w));
        const bool sure = key_score(key[p]) < (edge[p] + s) * (1.f - kDirectErr);
        g2[p] = sure ? 0x3FFFFFFFu : c[p].y;  // (no such group)
        if (!sure && c[p].y >= 0x3FFFFFFFu) g2[p] = 0x3FFFFFFFu;
        more |= !sure;
    }
    if (__ballot(more)) {
        uint64_t k2[NQ];
        group_best(g2, k2);
#pragma unroll
        for (int p = 0; p < NQ; ++p) {
            const float s1 = fminf(__uint_as_float(c[p].z), __uint_as_float(c[p].w));
            if (!(key_score(key[p]) < (edge[p] + s1) * (1.f - kDirectErr))) {
                key[p] = umin64(key[p], k2[p]);
                if (!(key_score(key[p]) < (edge[p] + __uint_as_float(c[p].w)) * (1.f - kDirectErr)))
                    bad[p] = true;
            }
        }
    }
    // (one entry into the list per workgroup: 500,000 queries, all of them left, 5 ms for
    // an entry each)
    uint32_t mine = 0;
#pragma unroll
    for (int p = 0; p < NQ; ++p)
        if (q0 + p < nq && bad[p]) ++mine;
    if (lane == 0) leaving[threadIdx.x >> 6] = mine;
    __syncthreads();
    uint32_t before = 0, all = 0;
#pragma unroll
    for (int w4 = 0; w4 < 4; ++w4) {
        before += w4 < (int)(threadIdx.x >> 6) ? leaving[w4] : 0u;
        all += leaving[w4];
    }
    if (threadIdx.x == 0 && all) first_place = atomicAdd(nrest, all);
    __syncthreads();
    uint32_t place = first_place + before;
#pragma unroll
    for (int p = 0; p < NQ; ++p) {
        if (q0 + p >= nq) break;
        if (bad[p]) {
            if (lane == p) rest[place] = (uint32_t)(q0 + p);
            ++place;
        } else if (lane == p) {
            D[q0 + p] = key_score(key[p]);
            I[q0 + p] = (int64_t)key_index(key[p]);
        }
    }
}

// ------------------------------------------------------------- host side
// Device words and buffers of one search.
struct SieveScratch {
    uint64_t* pool = nullptr;    // [nq][cap]
    uint32_t cap = 0;
    uint32_t* cnt = nullptr;     // [nq]
    uint32_t* flags = nullptr;   // [nq] queries that the split cannot hold
    uint32_t* bad_db = nullptr;  // [1] (may be null)
    uint32_t* rest = nullptr;    // [nq] queries that are left to the fused search
    uint32_t* nrest = nullptr;   // [1] how many
    const float* qnorm = nullptr;
    const float* thr = nullptr;  // threshold of query q at thr[q * thr_ld] (exact search)
    int64_t thr_ld = 0;
    float err = 0.f;             // split_err (exact search)
};

// Selection, re-rank and proof of every query of a search (sieve.hip).
mk_status sieve_finish_any(const SieveScratch& w, const float* xq, int64_t nq, const float* xb,
                           int32_t d, bool vec, bool l2, int32_t k, int32_t keff, bool cert,
                           float* D, int64_t* I, hipStream_t s);

}  // namespace mk
