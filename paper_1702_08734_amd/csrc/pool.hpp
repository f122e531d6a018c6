// Candidate pools of a workgroup in LDS: unsorted 64-bit keys that are cut back
// to the kk smallest by a histogram selection, and sorted at the end by bucket.
// Four waves share one pool, so its threshold is the workgroup's, and no step is
// done by one wave alone.  A cut of 2,048 or 4,096 keys is a handful of barriers;
// a sorted register queue per wave pays a network over the whole queue for every
// few hundred insertions and a serial merge of the queues.
#pragma once

#include "wave_select.hpp"

namespace mk {

constexpr int kPoolThreads = 256;
constexpr int kPoolWaves = kPoolThreads / 64;
constexpr int kCutBins = 1024;

// LDS words beside a pool and its kCutBins bins.
struct PoolState {
    uint64_t limit;             // threshold key: only smaller keys are kept
    unsigned long long lo, hi;  // range of the keys looked at
    uint32_t count;             // (for the user) keys in the pool
    uint32_t bin, below, edge;  // bin of the rank looked for, keys below it, keys in it
    uint32_t front, back;       // cursors
    uint32_t wsum[kPoolWaves];
};

// Sum of v over the workgroup, in every thread; before: this thread's exclusive
// prefix.  ws: kPoolWaves words that no other call since the last barrier uses.
__device__ __forceinline__ uint32_t pool_sum(uint32_t v, uint32_t* ws, uint32_t& before) {
    const int lane = lane_id(), wave = threadIdx.x >> 6;
    const uint32_t incl = (uint32_t)wave_inclusive_sum((int)v);
    if (lane == 63) ws[wave] = incl;
    __syncthreads();
    uint32_t all = 0;
    before = incl - v;
#pragma unroll
    for (int w = 0; w < kPoolWaves; ++w) {
        before += w < wave ? ws[w] : 0u;
        all += ws[w];
    }
    return all;
}

// Histogram of key[0 .. PER) (keys of index below n) over their range into bins;
// false when all keys are equal.  Leaves a barrier behind it.
template <int PER>
__device__ __forceinline__ bool pool_histogram(const uint64_t (&key)[PER], uint32_t n,
                                               uint32_t* bins, PoolState* st, uint64_t& base,
                                               int& shift) {
    const int tid = threadIdx.x;
    uint64_t lo = ~0ull, hi = 0ull;
#pragma unroll
    for (int j = 0; j < PER; ++j) {
        if ((uint32_t)(j * kPoolThreads + tid) < n) {
            lo = umin64(lo, key[j]);
            hi = umax64(hi, key[j]);
        }
    }
    if (tid == 0) {
        st->lo = ~0ull;
        st->hi = 0ull;
        st->front = st->back = 0u;
    }
#pragma unroll
    for (int j = 0; j < kCutBins / kPoolThreads; ++j) bins[j * kPoolThreads + tid] = 0u;
    __syncthreads();
    lo = wave_min64(lo);
    hi = wave_max64(hi);
    if (lane_id() == 0) {
        atomicMin(&st->lo, (unsigned long long)lo);
        atomicMax(&st->hi, (unsigned long long)hi);
    }
    __syncthreads();
    base = st->lo;
    const uint64_t range = st->hi - base;
    const int bits = range ? 64 - __builtin_clzll(range) : 0;
    shift = bits > 10 ? bits - 10 : 0;
    if (range)
#pragma unroll
        for (int j = 0; j < PER; ++j)
            if ((uint32_t)(j * kPoolThreads + tid) < n)
                atomicAdd(&bins[(key[j] - base) >> shift], 1u);
    __syncthreads();
    return range != 0;
}

// Cut the pool of n > kk keys to exactly its kk smallest, and set the threshold
// to the largest of them + 1 (keys are unique, as a rule).  All threads of the
// workgroup; the keys pass through registers (PER per thread).  A histogram of
// the keys over their range finds the bin of rank kk; the keys of that bin (a
// few, as a rule) are ranked against each other, or, where they are many, cut
// again by their own range.
template <int P>
__device__ __forceinline__ void pool_cut(uint64_t* pool, uint32_t* bins, PoolState* st, uint32_t n,
                                         int kk) {
    constexpr int NT = kPoolThreads, PER = P / NT, BPT = kCutBins / NT;
    const int tid = threadIdx.x;
    uint32_t first = 0, want = (uint32_t)kk;  // where the keys looked at start, and the rank
    __syncthreads();
#pragma unroll 1
    while (n > 64) {
        uint64_t key[PER];
#pragma unroll
        for (int j = 0; j < PER; ++j) {
            const uint32_t i = j * NT + tid;
            key[j] = i < n ? pool[first + i] : kSentinel;
        }
        uint64_t base;
        int shift;
        if (!pool_histogram(key, n, bins, st, base, shift)) {
            // equal keys (a list that repeats ids): any of them will do
            if (tid == 0) st->limit = base + 1;
            __syncthreads();
            return;
        }
        // prefix over the bins, BPT consecutive ones per thread
        uint32_t c[BPT], tot = 0, run;
#pragma unroll
        for (int j = 0; j < BPT; ++j) {
            c[j] = bins[tid * BPT + j];
            tot += c[j];
        }
        (void)pool_sum(tot, st->wsum, run);
#pragma unroll
        for (int j = 0; j < BPT; ++j) {
            if (run < want && run + c[j] >= want) {
                st->bin = tid * BPT + j;
                st->below = run;
                st->edge = c[j];
            }
            run += c[j];
        }
        __syncthreads();
        const uint32_t bin = st->bin, below = st->below;
        // keys below the bin to the front, the bin's own behind them
#pragma unroll
        for (int j = 0; j < PER; ++j) {
            if ((uint32_t)(j * NT + tid) < n) {
                const uint32_t b = (uint32_t)((key[j] - base) >> shift);
                if (b < bin) pool[first + atomicAdd(&st->front, 1u)] = key[j];
                if (b == bin) pool[first + below + atomicAdd(&st->back, 1u)] = key[j];
            }
        }
        first += below;
        want -= below;
        n = st->edge;
        __syncthreads();
    }
    // up to 64 keys: each counts the smaller ones
    const bool live = tid < (int)n;
    const uint64_t mine = live ? pool[first + tid] : kSentinel;
    uint32_t rank = 0;
    if (live)
        for (uint32_t e = 0; e < n; ++e) {
            const uint64_t o = pool[first + e];
            rank += o < mine || (o == mine && e < (uint32_t)tid) ? 1u : 0u;
        }
    __syncthreads();
    if (live && rank < want) {
        pool[first + rank] = mine;
        if (rank == want - 1) st->limit = mine + 1;
    }
    __syncthreads();
}

// The k smallest of the pool's n keys in order: emit(rank, key) for ranks below
// min(n, k).  Buckets of a histogram over the range, each key ranked inside its
// own; where a bucket is crowded (a cluster of near-equal scores far from the
// rest), the k smallest: of up to kPoolThreads keys each counts the smaller ones,
// and more go through a bitonic network (the next power of two of their number,
// <= P).
template <int P, class F>
__device__ __forceinline__ void pool_emit(uint64_t* pool, uint32_t* bins, PoolState* st, uint32_t n,
                                          uint32_t k, F emit) {
    constexpr int NT = kPoolThreads, PER = P / NT, BPT = kCutBins / NT;
    constexpr uint32_t kCrowd = 48;
    const int tid = threadIdx.x;
    __syncthreads();
    uint64_t key[PER];
#pragma unroll
    for (int j = 0; j < PER; ++j) {
        const uint32_t i = j * NT + tid;
        key[j] = i < n ? pool[i] : kSentinel;
    }
    uint64_t base;
    int shift;
    bool crowded = !pool_histogram(key, n, bins, st, base, shift) && n > kCrowd;
    uint32_t c[BPT], tot = 0, run, most = 0;
#pragma unroll
    for (int j = 0; j < BPT; ++j) {
        c[j] = bins[tid * BPT + j];
        tot += c[j];
        most = max(most, c[j]);
    }
    (void)pool_sum(tot, st->wsum, run);
    if (__syncthreads_or(crowded || most > kCrowd)) {
        if (n > (uint32_t)NT && n > k) {
            pool_cut<P>(pool, bins, st, n, (int)k);
            n = k;
        }
        if (n <= (uint32_t)NT) {  // each counts the smaller ones
            const uint64_t mine = tid < (int)n ? pool[tid] : kSentinel;
            uint32_t rank = 0;
#pragma unroll 4
            for (uint32_t e = 0; e < n; ++e) {
                const uint64_t o = pool[e];
                rank += o < mine || (o == mine && e < (uint32_t)tid) ? 1u : 0u;
            }
            if (tid < (int)n && rank < k) emit(rank, mine);
            return;
        }
        uint32_t size = 64;
        while (size < n) size *= 2;
        for (uint32_t i = n + tid; i < size; i += NT) pool[i] = kSentinel;
        __syncthreads();
#pragma unroll 1
        for (uint32_t p = 2; p <= size; p *= 2)
#pragma unroll 1
            for (uint32_t s = p / 2; s > 0; s /= 2) {
                for (uint32_t i = tid; i < size / 2; i += NT) {
                    const uint32_t lo = 2 * i - (i & (s - 1)), hi = lo + s;
                    const uint64_t a = pool[lo], b = pool[hi];
                    const bool up = (lo & p) == 0;
                    if ((a > b) == up) {
                        pool[lo] = b;
                        pool[hi] = a;
                    }
                }
                __syncthreads();
            }
        for (uint32_t i = tid; i < n; i += NT) emit(i, pool[i]);
        return;
    }
    // bins to their start, keys into their bucket (the start moves to the end)
#pragma unroll
    for (int j = 0; j < BPT; ++j) {
        bins[tid * BPT + j] = run;
        run += c[j];
    }
    __syncthreads();
#pragma unroll
    for (int j = 0; j < PER; ++j)
        if ((uint32_t)(j * NT + tid) < n)
            pool[atomicAdd(&bins[(key[j] - base) >> shift], 1u)] = key[j];
    __syncthreads();
    for (uint32_t i = tid; i < n; i += NT) {
        const uint64_t mine = pool[i];
        const uint32_t b = (uint32_t)((mine - base) >> shift);
        const uint32_t lo = b ? bins[b - 1] : 0u, hi = bins[b];
        if (lo >= k) continue;
        uint32_t rank = lo;
        for (uint32_t e = lo; e < hi; ++e) {
            const uint64_t o = pool[e];
            rank += o < mine || (o == mine && e < i) ? 1u : 0u;
        }
        if (rank < k) emit(rank, mine);
    }
}

// Keys p[0 .. n) through the pool: afterwards it holds the kk smallest (all of
// them when n <= kk); returns how many.  limit: the threshold's key (kSentinel
// while nothing was cut).  kk <= P / 2.
template <int P>
__device__ __forceinline__ uint32_t pool_stream(const uint64_t* __restrict__ p, int64_t n,
                                                uint64_t* pool, uint32_t* bins, PoolState* st,
                                                int kk, uint64_t& limit) {
    constexpr int NT = kPoolThreads, U = P / 4 / NT;  // keys per thread and step: a quarter pool
    uint32_t have = 0;
    limit = kSentinel;
#pragma unroll 1
    for (int64_t e0 = 0; e0 < n; e0 += NT * U) {
        uint64_t key[U];
        uint32_t c = 0, at;
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int64_t i = e0 + u * NT + threadIdx.x;
            key[u] = i < n ? p[i] : kSentinel;
            c += key[u] < limit ? 1u : 0u;
        }
        const uint32_t add = pool_sum(c, st->wsum, at);
        at += have;
#pragma unroll
        for (int u = 0; u < U; ++u)
            if (key[u] < limit) pool[at++] = key[u];
        have += add;
        if (have > (uint32_t)(P - NT * U)) {
            pool_cut<P>(pool, bins, st, have, kk);
            have = (uint32_t)kk;
            limit = st->limit;
        }
        __syncthreads();
    }
    if (have > (uint32_t)kk) {
        pool_cut<P>(pool, bins, st, have, kk);
        have = (uint32_t)kk;
        limit = st->limit;
    }
    return have;
}

// Values rp[0 .. n) of one row into an empty pool, keyed (value, first + place):
// afterwards it holds the kk smallest (largest: negated values) and perhaps more,
// unsorted; returns how many.  A step is 1,024 U values, 4 U per thread, 16-byte
// loads (4-byte ones where rows start off the 16-byte grid), the next step's in
// flight; values that do not beat the pool's threshold cost one compare, and a
// step without any costs one barrier.  The pool is cut when a step's values do not
// fit beside its keys: a row of L values sees about kk (1 + ln(L / kk)) insertions
// and a cut for every P - kk of them.  (Steps of 4,096 values need a second place
// for cuts in the loop and the registers for it: fewer waves, 5 to 10% slower.)
// Places ascend from step to step, so that a value equal to the threshold's score comes
// too late (rows of few different values: 10^4 x 10,000, k = 65, 160 us when such values
// were looked at one by one, 142).  NaN never enters.  ws: LDS words of its own.
template <int P, int U, bool LARGEST>  // kk <= P - 1024 U
__device__ __forceinline__ uint32_t pool_values(const float* __restrict__ rp, uint32_t n,
                                                uint32_t first, int32_t kk, uint64_t* pool,
                                                uint32_t* bins, PoolState* st,
                                                uint32_t (*ws)[kPoolWaves]) {
    constexpr int NT = kPoolThreads, STEP = NT * 4 * U;
    const int tid = threadIdx.x;
    const bool aligned = (reinterpret_cast<uintptr_t>(rp) & 15) == 0;
    // value j of quarter u is 1,024 u + 4 tid + j (aligned) or + 256 j + tid
    const uint32_t mine = aligned ? 4u * tid : (uint32_t)tid, stride = aligned ? 1u : (uint32_t)NT;
    uint32_t have = 0;
    float limit_f = INFINITY;  // (looked at once the pool was cut)
    bool open = true;
    int turn = 0;
    auto cut = [&]() __attribute__((always_inline)) {
        pool_cut<P>(pool, bins, st, have, kk);
        have = (uint32_t)kk;
        limit_f = key_score(st->limit - 1);
        open = false;
    };
    // a step's values, the next step's while this one is looked at
    float next[U][4];
    auto load = [&](uint32_t e) __attribute__((always_inline)) {
        if (aligned && n - e >= (uint32_t)STEP) {
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const float4 w = *reinterpret_cast<const float4*>(rp + e + u * (NT * 4) + mine);
                next[u][0] = w.x;
                next[u][1] = w.y;
                next[u][2] = w.z;
                next[u][3] = w.w;
            }
        } else {
#pragma unroll
            for (int u = 0; u < U; ++u)
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const uint32_t i = u * (NT * 4) + mine + j * stride;
                    next[u][j] = i < n - e ? rp[e + i] : NAN;  // (never taken)
                }
        }
    };
    if (n > 0) load(0);
#pragma unroll 1
    for (uint32_t e0 = 0; e0 < n;) {
        float v[U][4];
        const uint32_t place = first + e0 + mine;  // column of this thread's first value
        auto at = [&](int u, int j) __attribute__((always_inline)) -> uint32_t {
            return place + u * (NT * 4) + j * stride;
        };
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int j = 0; j < 4; ++j) v[u][j] = next[u][j];
        // (e0 + STEP may pass 2^32 - 1 on the last step)
        const bool last = n - e0 <= (uint32_t)STEP;
        if (!last) load(e0 + STEP);
        e0 = last ? n : e0 + STEP;
        bool any = false;
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                if (LARGEST) v[u][j] = -v[u][j];
                any |= v[u][j] < limit_f;
            }
        if (!__syncthreads_or(any || open)) continue;
        // which values enter
        auto takes = [&](int u) __attribute__((always_inline)) {
            uint32_t mask = 0;
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const bool t = open ? v[u][j] == v[u][j] : v[u][j] < limit_f;
                mask |= t ? 1u << j : 0u;
            }
            return mask;
        };
        uint32_t mask[U], add, pos;
        auto count = [&]() __attribute__((always_inline)) {
            uint32_t c = 0;
#pragma unroll
            for (int u = 0; u < U; ++u) {
                mask[u] = takes(u);
                c += __popc(mask[u]);
            }
            add = pool_sum(c, ws[turn ^= 1], pos);
        };
        count();
        if (have + add > (uint32_t)P) {  // (kk <= P - STEP: after a cut they fit)
            cut();
            count();
        }
        pos += have;
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int j = 0; j < 4; ++j)
                if (mask[u] & (1u << j)) pool[pos++] = make_key(v[u][j], at(u, j));
        have += add;
    }
    return have;
}

}  // namespace mk
