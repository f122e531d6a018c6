// Exact search where either side is small (dense.hip).
#pragma once

#include "common.hpp"

namespace mk {

// Scratch bytes per query of dense_search (and up to 768 bytes of padding).
int64_t dense_query_bytes(int64_t nb, int32_t k);

// Whether dense_search takes a call: enough groups of four rows that the kept
// ones are few.
inline bool dense_pays(int64_t nq, int64_t nb, int32_t k) {
    return nq > 0 && nb >= 2048 && nb >= 32ll * k;
}

// scratch: nq * dense_query_bytes + 768 bytes of device memory, or null (then
// allocated).
mk_status dense_search(const float* xq, int64_t nq, const float* xb, const float* yn, int64_t nb,
                       int32_t d, int32_t k, bool l2, bool vec, float* D, int64_t* I,
                       void* scratch, hipStream_t s);

}  // namespace mk
