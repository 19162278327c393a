// Kernels of the matrix phases of 2..16 rows (few_rows.h), a code object of their own.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "batch_launch.h"
#include "few_rows.h"

namespace mtp {
namespace {

template <int PH, bool PACKED, int T>
__global__ __launch_bounds__(kBlock) void k_few(DraftParams p, int step, int per, int rem) {
    extern __shared__ __align__(16) char smem[];
    if constexpr (PH == BG_PROJ) {
        BgProj ph(p);
        few_rows<PACKED, T>(p, ph, per, rem, smem);
    } else if constexpr (PH == BG_QKV) {
        BgQkv ph(p);
        few_rows<PACKED, T>(p, ph, per, rem, smem);
    } else if constexpr (PH == BG_OPROJ) {
        BgOproj ph(p);
        few_rows<PACKED, T>(p, ph, per, rem, smem);
    } else if constexpr (PH == BG_GATEUP) {
        BgGateUp ph(p);
        few_rows<PACKED, T>(p, ph, per, rem, smem);
    } else if constexpr (PH == BG_DOWN) {
        BgDown ph(p);
        few_rows<PACKED, T>(p, ph, per, rem, smem);
    } else {
        BgHead ph(p, step);
        few_rows<PACKED, T>(p, ph, per, rem, smem);
    }
}

typedef void (*few_kernel_t)(DraftParams, int, int, int);
// tiles: the most a workgroup has (more than eight: groups of eight)
template <int PH, bool PACKED>
few_kernel_t pick_few(int tiles) {
    if constexpr (PH == BG_PROJ || PH == BG_OPROJ || PH == BG_DOWN)
        return tiles <= 1 ? k_few<PH, PACKED, 1> : k_few<PH, PACKED, 2>;
    else if constexpr (PH == BG_GATEUP)
        return tiles <= 2 ? k_few<PH, PACKED, 2> : tiles <= 4 ? k_few<PH, PACKED, 4> : tiles <= 6 ? k_few<PH, PACKED, 6> : k_few<PH, PACKED, 8>;
    else
        return tiles <= 1   ? k_few<PH, PACKED, 1>
               : tiles <= 2 ? k_few<PH, PACKED, 2>
               : tiles <= 4 ? k_few<PH, PACKED, 4>
               : tiles <= 6 ? k_few<PH, PACKED, 6>
                            : k_few<PH, PACKED, 8>;
}
template <bool PACKED>
few_kernel_t few_kernel_of(int phase, int tiles) {
    switch (phase) {
    case BG_PROJ: return pick_few<BG_PROJ, PACKED>(tiles);
    case BG_QKV: return pick_few<BG_QKV, PACKED>(tiles);
    case BG_OPROJ: return pick_few<BG_OPROJ, PACKED>(tiles);
    case BG_GATEUP: return pick_few<BG_GATEUP, PACKED>(tiles);
    case BG_DOWN: return pick_few<BG_DOWN, PACKED>(tiles);
    default: return pick_few<BG_LMHEAD, PACKED>(tiles);
    }
}
few_kernel_t few_kernel(int phase, int rows, int tiles) {
    return rows <= kFewPacked ? few_kernel_of<true>(phase, tiles) : few_kernel_of<false>(phase, tiles);
}
int few_units(int phase, const DraftParams &p) { // tiles of sixteen weight rows (gate/up: pairs)
    const int rows = phase == BG_QKV ? p.qkv_dim : phase == BG_GATEUP ? p.F : phase == BG_LMHEAD ? p.n : p.d;
    return (rows + 15) / 16;
}

} // namespace

int few_groups(int phase, const DraftParams &p, int cus) { return std::min(cus, few_units(phase, p)); }

bool few_allow_lds(size_t lds_limit) {
    bool ok = few_lds_bytes() <= lds_limit;
    for (int rows : {kFewPacked, kFewRows})
        for (int ph = 0; ph < BG_COUNT; ++ph) {
            few_kernel_t last = nullptr; // (several tile counts share a kernel)
            for (int t : {1, 2, 4, 6, 8}) {
                const few_kernel_t k = few_kernel(ph, rows, t);
                if (k != last)
                    ok = ok && hipFuncSetAttribute((const void *)k, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds_limit) ==
                                   hipSuccess;
                last = k;
            }
        }
    return ok;
}

void launch_few(int phase, const DraftParams &p, int step, int cus, hipStream_t st) {
    const int units = few_units(phase, p), rg = few_groups(phase, p, cus);
    const int tiles = (units + rg - 1) / rg * (phase == BG_GATEUP ? 2 : 1);
    hipLaunchKernelGGL(few_kernel(phase, p.nb, tiles), dim3(rg), dim3(kBlock), few_lds_bytes(), st, p, step,
                       units / rg, units % rg);
}

} // namespace mtp
