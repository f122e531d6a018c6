// Exact-search entry points of the padded dimension classes, each class
// compiled in its own translation unit.
#pragma once

#include "common.hpp"
#include "kselect.hpp"

namespace mk {

// Searches for padded dimension class DP (knn_impl.hpp, one translation unit
// per class): the fused kernel, and the threshold-first batch search.
template <int DP>
mk_status knn_dispatch_k(const float* xq, int64_t nq, const float* xb, const float* yn,
                         int64_t nb, int32_t d, int32_t k, bool l2, bool vec, float* D, int64_t* I,
                         hipStream_t s, Arena* arena, const RestQueries* rest);
template <int DP>
mk_status sieve_dispatch(const float* xq, int64_t nq, const float* xb, const float* yn, int64_t nb,
                         int32_t d, int32_t k, bool l2, bool vec, float* D, int64_t* I,
                         hipStream_t s);
template <int DP>
mk_status nearest_dispatch(const float* xq, int64_t nq, const float* xb, const float* yn,
                           int64_t nb, int32_t d, bool vec, float* D, int64_t* I, hipStream_t s);
#define MK_KNN_CLASS(DP)                                                                         \
    extern template mk_status knn_dispatch_k<DP>(const float*, int64_t, const float*,            \
                                                 const float*, int64_t, int32_t, int32_t, bool,  \
                                                 bool, float*, int64_t*, hipStream_t, Arena*,    \
                                                 const RestQueries*);                               \
    extern template mk_status sieve_dispatch<DP>(const float*, int64_t, const float*,            \
                                                 const float*, int64_t, int32_t, int32_t, bool,  \
                                                 bool, float*, int64_t*, hipStream_t);           \
    extern template mk_status nearest_dispatch<DP>(const float*, int64_t, const float*,          \
                                                   const float*, int64_t, int32_t, bool, float*, \
                                                   int64_t*, hipStream_t);
MK_KNN_CLASS(32)
MK_KNN_CLASS(64)
MK_KNN_CLASS(96)
MK_KNN_CLASS(128)
MK_KNN_CLASS(256)
#undef MK_KNN_CLASS

}  // namespace mk
