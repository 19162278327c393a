// The tiled matrix products (rows_gemm.h) as kernels, for the translation units that instantiate them.
#pragma once
#include "rows_gemm.h"

namespace mtp {
namespace {

// A matrix phase over the rows p.seq_lo .. p.seq_hi - 1 (all of a call's, or those that share an id list) as one tiled matrix
// product (rows_gemm.h).  PH: a BG_* index, or kHeadLogits for the output head without candidates.  One workgroup per CU (120
// to 147 KB of LDS, up to 256 registers).
constexpr int kHeadLogits = BG_COUNT;
template <int PH, class F>
__device__ __forceinline__ void with_phase(int step, F f) {
    if constexpr (PH == BG_PROJ)
        f([](const DraftParams &q) { return BgProj(q); });
    else if constexpr (PH == BG_QKV)
        f([](const DraftParams &q) { return BgQkv(q); });
    else if constexpr (PH == BG_OPROJ)
        f([](const DraftParams &q) { return BgOproj(q); });
    else if constexpr (PH == BG_GATEUP)
        f([](const DraftParams &q) { return BgGateUp(q); });
    else if constexpr (PH == BG_DOWN)
        f([](const DraftParams &q) { return BgDown(q); });
    else
        f([step](const DraftParams &q) { return BgHeadRows<PH == BG_LMHEAD>(q, step); });
}
template <int PH, class T>
__global__ __launch_bounds__(kBlock, 2) void k_rows_gemm(DraftParams p, int step, int KP) {
    extern __shared__ __align__(16) char smem[];
    with_phase<PH>(step, [&](auto make) { rows_gemm<T, decltype(make(p))>(p, make, KP, smem); });
}

} // namespace
} // namespace mtp
