// Exact search where either side is small (dense.hip).
#pragma once

#include "common.hpp"
#include "kselect.hpp"

namespace mk {

// Scratch bytes per query of dense_search (and up to 768 bytes of padding).
int64_t dense_query_bytes(int64_t nb, int32_t k);

// Whether dense_search takes a call: enough groups of four rows that the kept
// ones are few.
inline bool dense_pays(int64_t nq, int64_t nb, int32_t k) {
    return nq > 0 && nb >= 2048 && nb >= 32ll * k;
}

// Whether dense_search is faster than the threshold-first search where both take a
// call.  The latter starts with some 90 us of splitting, sampling and selecting,
// plus the time to split the database (2 us for 10^6 values), but scores about four
// times as fast: 2^31 products of queries, rows and dimensions take 15 us, here 50,
// after 25 us.  To either side of the line, k = 10: 64 / 512 queries, 262,144 x 64
// rows 64 / 232 us here, 143 / 180 there; 512 queries, 65,536 x 32 rows 66, 108; 128
// queries, 524,288 x 256 rows 371, 433; 1,024 queries, 32,768 x 128 rows 118, 123.
// (k = 100 draws the same line; longer lists were not measured.)
inline bool dense_beats_sieve(int64_t nq, int64_t nb, int32_t d, int32_t k) {
    const int64_t dp = d <= 128 ? (d + 31) / 32 * 32 : 256;
    const double split = (double)nb * (double)dp, work = split * (double)nq * 0x1p-31;
    return k <= 128 && dense_pays(nq, nb, k) && work * 35. < 65. + 2e-6 * split;
}

// scratch: nq * dense_query_bytes + 768 bytes of device memory, or null (then
// allocated).
mk_status dense_search(const float* xq, int64_t nq, const float* xb, const float* yn, int64_t nb,
                       int32_t d, int32_t k, bool l2, bool vec, float* D, int64_t* I,
                       void* scratch, hipStream_t s);

// The queries that another search left (there are at most nq of them), for any number
// up to dense_rest_most: up to two launches of it search them all, and *rest tells the
// fused search what is left to it.
inline int64_t dense_rest_most(int64_t nq, int64_t nb) {
    const int64_t most = (1ll << 30) / ((nb + 63) / 64 * 64);
    return most < 64 ? 0 : most < 4096 ? (most < nq ? most : nq) : nq < 4096 ? nq : 4096;
}
// Its scratch (0: it takes none of them).
inline size_t dense_rest_bytes(int64_t nq, int64_t nb, int32_t k) {
    return dense_pays(nq, nb, k) ? (size_t)dense_rest_most(nq, nb) * (size_t)((nb + 63) / 64 * 64) : 0;
}
mk_status dense_rest(const float* xq, int64_t nq, const float* xb, const float* yn, int64_t nb,
                     int32_t d, int32_t k, bool l2, bool vec, float* D, int64_t* I, RestQueries* rest,
                     hipStream_t s);

}  // namespace mk
