// Sizes of the threshold-first search (sieve.hpp): what it takes, sample, pools,
// chunks and batches.  Host arithmetic alone, so that it can be checked without a GPU.
#pragma once

#include <cmath>
#include <cstdint>

namespace mk {

inline int64_t plan_div(int64_t a, int64_t b) { return (a + b - 1) / b; }

// rows of one chunk are staged as this many bits
constexpr int kSieveRowBits = 25;

// Relative bound on what the split product, the norms and their sum can err together,
// for rows of DP components: every score is lowered by split_err (||x||^2 + ||y||^2)
// (L2) or 2 split_err ||x|| ||y|| (inner product), which makes it a lower bound of the
// row's true score.  In units of 2^-24, of ||x||^2 + ||y||^2:
//   8 + 3 DP / 32  the product: two factors split to 2^-23 and l l <= 2^-22 dropped,
//                  and a rounding per matrix instruction of the chain (how an
//                  instruction adds up its 32 products is not documented: measured on
//                  10^6 pairs of rows of equal components, whose roundings all go one
//                  way, the whole errs by at most 8.5, 10.7, 12.4, 16.3 and 27.7 units
//                  for DP = 32 .. 256, where this is 11, 14, 17, 20 and 32);
//   8 NG + log2 LPR  a norm: 8 products per granule and lane, then a sum over lanes;
//   4              components less the center, each rounded once;
//   4              the norm's factor, the score's last sum, and the bound's own.
// So it is a bound if no matrix instruction rounds worse than those; the largest error
// of whole scores against float64 that was seen on five distributions, d = 17 .. 256,
// is a sixth of it (3.2e-7; the fused kernel's FP32 chain 9.5e-7).
constexpr float split_err(int DP) {
    const int granules = DP / 8, lanes = granules > 8 ? 16 : granules;
    int sum = 0;
    for (int l = lanes; l > 1; l /= 2) ++sum;
    return (float)(8 + 3 * DP / 32 + 8 * ((granules + lanes - 1) / lanes) + sum + 8) * 0x1p-24f;
}
// What the direct form of a distance errs by, of the distance: up to 16 chained sums of
// squares per lane of the rows' components (d <= 256), a sum over 16 lanes, and the
// differences, rounded before they are squared: 22 units of 2^-24, and one for the bound.
constexpr float kDirectErr = 0x1p-19f;

// Sample size, threshold rank and pool capacity.  Of the keff best rows a
// sample of fraction f holds about mu = f keff, so a rank of mu + 4.5
// sqrt(mu) + 4.5 leaves a chance of about 1e-8 that the threshold admits fewer
// than keff rows; it admits about r / f, and more than cap with a chance under
// 1e-8.  Scoring a sample row costs a query about as much as a row of the
// database, a row that passes about 40 times that: samples of the order of
// the square root of the database (8192 rows of 2^18, twice as many for every
// factor of four) keep both small.
struct SievePlan {
    int64_t sample;
    int32_t rank;
    int64_t cap;
};
inline SievePlan plan_sieve(int64_t nb, int32_t keff) {
    SievePlan p;
    p.sample = 8192;
    for (int64_t n = 1ll << 18; n < nb && p.sample < 65536; n *= 4) p.sample *= 2;
    while (p.sample > 1024 && p.sample * 8 > nb) p.sample /= 2;
    const double f = (double)p.sample / (double)nb;
    const double mu = f * keff;
    const double r = std::ceil(mu + 4.5 * std::sqrt(mu) + 4.5);
    p.rank = (int32_t)r;
    p.cap = (int64_t)std::ceil((r + 6.0 * std::sqrt(r) + 9.0) / f);
    p.cap = plan_div(p.cap < nb ? p.cap : nb, 64) * 64;
    return p;
}

// Chunks of the rows of one launch: whole rounds of one workgroup per CU.
inline void plan_sieve_chunks(int64_t nqb, int64_t nb, int BN, int64_t* nchunks,
                              int64_t* chunk_len) {
    constexpr int64_t kCUs = 256;
    const int64_t steps = plan_div(nb, BN);
    double best = 1e300;
    int64_t pick = 1;
    // (the row count of a chunk itself has to fit the bits: it marks "past the end")
    const int64_t least = plan_div(nb, (1ll << kSieveRowBits) - 4 * BN);
    for (int64_t w = 1; w <= 6; ++w) {
        int64_t n = kCUs * w / nqb;
        if (n < least) n = least;
        if (n > steps) n = steps;
        const int64_t rounds = plan_div(nqb * n, kCUs);
        // about 6 steps' worth to load the queries and fill the pipeline
        const double cost = (double)rounds * ((double)plan_div(steps, n) + 6.0);
        if (cost < best) {
            best = cost;
            pick = n;
        }
    }
    *chunk_len = plan_div(steps, pick) * BN;
    *nchunks = plan_div(nb, *chunk_len);
}

// Whether the threshold-first search takes a call that keeps keff candidates:
// the least scores of the sample (of up to 16 rows each) have to be several
// times the rank taken of them.
inline bool sieve_pays(int64_t nq, int64_t nb, int32_t keff) {
    if (nb < 16384 || nq < 64 || nq * nb < (1ll << 24)) return false;
    const SievePlan p = plan_sieve(nb, keff);
    return p.sample >= 64ll * p.rank;
}

// Whether the nearest-row search (k = 1: k-means assignment, list assignment of
// added rows) takes a call: enough queries to fill the chip with workgroups that
// each stream every row, and few enough rows for one stream of them.
inline bool nearest_pays(int64_t nq, int64_t nb) {
    return nq >= 8192 && nb >= 256 && nb <= 65536 && nq * nb >= (1ll << 25);
}

// Queries per batch: at most 1 GiB of pools, and of the sample's scores.
inline int64_t sieve_batch(int64_t nq, int64_t nb, int32_t keff) {
    const SievePlan p = plan_sieve(nb, keff);
    int64_t b = (1ll << 30) / (8 * p.cap);
    if (b > (1ll << 30) / p.sample) b = (1ll << 30) / p.sample;
    b = b >= 256 ? b / 256 * 256 : b / 64 * 64;  // (at least 64: a pool is below 8 MB)
    if (b < 64) b = 64;
    return nq < b ? nq : b;
}

}  // namespace mk
