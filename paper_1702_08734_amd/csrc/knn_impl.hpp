// Launch of the exact-search kernels for one padded dimension class DP
// (instantiated once per class in its own translation unit, knn_dNNN.hip,
// so that the many kernel variants compile in parallel).
#pragma once

#include "fused.hpp"

namespace mk {

// Fused search: of all queries, or of those of `rest` alone.
template <int KR, int DP>
mk_status knn_launch(const float* xq, int64_t nq, const float* xb, const float* yn, int64_t nb,
                     int32_t d, int32_t k, bool l2, bool vec, float* D, int64_t* I,
                     hipStream_t stream, Arena* arena, const RestQueries* rest) {
    using S = FusedShape<KR, DP * 4, fused_consumers<OpF32, DP>()>;
    constexpr int KS = 64 * KR;
    const int keff = k + kSlack < KS ? k + kSlack : KS;
    int64_t nqb, nchunks, chunk_len;
    plan_chunks(nq, nb, S::BQ, S::BN, KS, &nqb, &nchunks, &chunk_len);

    Scratch part, bound;
    RestPlan* plan = nullptr;
    MK_TRY((fused_scratch<S, KR>(nq, nb, nqb, nchunks, rest, part, bound, &plan, stream, arena)));
    if (sizing_only(arena)) return MK_OK;
    const int64_t nblocks = nqb * nchunks;
    // the grid's work-item count must fit 32 bits
    MK_REQUIRE(nblocks * 64 * (kProducers + S::NC) < (1ll << 32), MK_ERR_UNSUPPORTED,
               "problem too large for one launch (search fewer queries per call)");
    unsigned long long* drops = nullptr;
    MK_TRY(pool_drop_counter(&drops));
    FusedArgs a{xq, xb, yn, nullptr, nullptr, nq, nb, d, d, chunk_len, (int32_t)nchunks,
                (int32_t)nqb, keff, part.as<uint64_t>(), bound.as<uint32_t>(), drops,
                rest ? rest->list : nullptr, plan};
    {
        ProfScope prof(rest ? "knn_fused_rest" : "knn_fused", stream);
        auto kern = vec ? (l2 ? knn_fused<OpF32, KR, DP, true, true> : knn_fused<OpF32, KR, DP, true, false>)
                        : (l2 ? knn_fused<OpF32, KR, DP, false, true> : knn_fused<OpF32, KR, DP, false, false>);
        hipLaunchKernelGGL(kern, dim3((unsigned)nblocks), dim3(64 * (kProducers + S::NC)), 0, stream, a);
        MK_LAUNCHED();
    }
    {
        ProfScope prof("knn_merge_rerank", stream);
        hipLaunchKernelGGL((knn_merge_rerank<KR>), dim3((unsigned)ceil_div(nq, kMergeWaves)),
                           dim3(64 * kMergeWaves), 0, stream, part.as<uint64_t>(),
                           (int32_t)nchunks, (int32_t)S::ROW, S::mem_queues ? KS : keff, xq, nq,
                           xb, d, (int32_t)vec, (int32_t)l2, k, keff, D, I, a.qlist, plan);
        MK_LAUNCHED();
    }
    return MK_OK;
}

template <int DP>
mk_status knn_dispatch_k(const float* xq, int64_t nq, const float* xb, const float* yn,
                         int64_t nb, int32_t d, int32_t k, bool l2, bool vec, float* D, int64_t* I,
                         hipStream_t s, Arena* arena, const RestQueries* rest) {
    const int want = k + kSlack < kMaxK ? k + kSlack : kMaxK;
    switch (queue_regs(want)) {
        case 1: return knn_launch<1, DP>(xq, nq, xb, yn, nb, d, k, l2, vec, D, I, s, arena, rest);
        case 2: return knn_launch<2, DP>(xq, nq, xb, yn, nb, d, k, l2, vec, D, I, s, arena, rest);
        case 4: return knn_launch<4, DP>(xq, nq, xb, yn, nb, d, k, l2, vec, D, I, s, arena, rest);
        case 8: return knn_launch<8, DP>(xq, nq, xb, yn, nb, d, k, l2, vec, D, I, s, arena, rest);
        default: return knn_launch<16, DP>(xq, nq, xb, yn, nb, d, k, l2, vec, D, I, s, arena, rest);
    }
}

}  // namespace mk
