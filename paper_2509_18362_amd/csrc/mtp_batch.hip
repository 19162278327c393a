// Kernels of the batched draft path (two or more sequences per call) for gfx950.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "attn_mfma.h"
#include "batch.h"
#include "batch_launch.h"
#include "rows_gemm.h"

namespace mtp {
namespace {

// up to 16 sequences: the waves split the reduction; more: they split the tiles and share the activations in LDS
template <int NA, class Ph>
__device__ __forceinline__ void run_phase(const DraftParams &p, Ph &ph, int which, char *smem) {
    if constexpr (NA == 1)
        bgemv<1>(p, ph, p.bg_rg[which], p.bg_kp[which], smem);
    else
        bgemv_lds<NA>(p, ph, p.bg_rg[which], p.bg_kp[which], smem);
}

template <int PH, int NA>
__global__ __launch_bounds__(kBlock) void k_bgemv(DraftParams p, int step) {
    extern __shared__ __align__(16) char smem[];
    if constexpr (PH == BG_PROJ) {
        BgProj ph(p);
        run_phase<NA>(p, ph, PH, smem);
    } else if constexpr (PH == BG_QKV) {
        BgQkv ph(p);
        run_phase<NA>(p, ph, PH, smem);
    } else if constexpr (PH == BG_OPROJ) {
        BgOproj ph(p);
        run_phase<NA>(p, ph, PH, smem);
    } else if constexpr (PH == BG_GATEUP) {
        BgGateUp ph(p);
        run_phase<NA>(p, ph, PH, smem);
    } else if constexpr (PH == BG_DOWN) {
        BgDown ph(p);
        run_phase<NA>(p, ph, PH, smem);
    } else {
        BgHead ph(p, step);
        run_phase<NA>(p, ph, PH, smem);
    }
}

template <int PH, int NA>
__global__ __launch_bounds__(kBlock) void k_bepilogue(DraftParams p, int step) {
    __shared__ __align__(16) char smem[kWaves * kBatchMaxSeq * 8 + kBatchMaxSeq * 4];
    if constexpr (PH == BG_PROJ) {
        BgProj ph(p);
        phase_bepilogue<NA>(p, ph, p.bg_kp[PH], smem);
    } else if constexpr (PH == BG_QKV) {
        BgQkv ph(p);
        phase_bepilogue<NA>(p, ph, p.bg_kp[PH], smem);
    } else if constexpr (PH == BG_OPROJ) {
        BgOproj ph(p);
        phase_bepilogue<NA>(p, ph, p.bg_kp[PH], smem);
    } else if constexpr (PH == BG_GATEUP) {
        BgGateUp ph(p);
        phase_bepilogue<NA>(p, ph, p.bg_kp[PH], smem);
    } else if constexpr (PH == BG_DOWN) {
        BgDown ph(p);
        phase_bepilogue<NA>(p, ph, p.bg_kp[PH], smem);
    } else {
        BgHead ph(p, step);
        phase_bepilogue<NA>(p, ph, p.bg_kp[PH], smem);
    }
}

__global__ __launch_bounds__(kBlock) void k_bprep(DraftParams p, int step) {
    __shared__ __align__(16) char smem[256];
    phase_bprep(p, step, smem);
}

// A matrix phase over all p.B rows as one tiled matrix product (rows_gemm.h).  PH: a BG_* index, or kHeadLogits for the
// output head without candidates.  One workgroup per CU (144 KB of LDS, up to 256 registers).
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
template <int PH, int WM, int WN, int TJ>
__global__ __launch_bounds__(kBlock, 2) void k_rows_gemm(DraftParams p, int step, int KP) {
    extern __shared__ __align__(16) char smem[];
    with_phase<PH>(step, [&](auto make) {
        rows_gemm<WM, WN, TJ, decltype(make(p))>(p, make, KP, smem);
    });
}
template <int PH>
__global__ __launch_bounds__(kBlock) void k_rows_epilogue(DraftParams p, int step, int KP, int RT) {
    __shared__ float scale[16];
    with_phase<PH>(step, [&](auto make) { rows_epilogue<decltype(make(p))>(p, make, KP, RT, scale); });
}

template <int G, int HD>
__global__ __launch_bounds__(kBlock) void k_attn_mfma(DraftParams p, int step) {
    extern __shared__ __align__(16) char smem[];
    // merges its own splits (tickets), hands its items out one by one
    phase_attn_mfma<G, HD, false, true, NoHook, true>(p, step, blockIdx.x, gridDim.x, smem);
}

// the same with the items numbered longest first, for launches with more items than workgroups
template <int G, int HD>
__global__ __launch_bounds__(kBlock) void k_attn_mfma_lpt(DraftParams p, int step) {
    extern __shared__ __align__(16) char smem[];
    phase_attn_mfma<G, HD, false, true, NoHook, true, 1, true>(p, step, blockIdx.x, gridDim.x, smem);
}

// a block of new positions per sequence (keys and values already in the cache): the positions of a sequence share its
// key/value reads, 16 / G of them beside the G query heads in the MFMA columns
template <int G, int HD>
__global__ __launch_bounds__(kBlock) void k_attn_mfma_block(DraftParams p, int step) {
    extern __shared__ __align__(16) char smem[];
    phase_attn_mfma<G, HD, false, true, NoHook, true, 16 / G>(p, step, blockIdx.x, gridDim.x, smem);
}

typedef void (*bg_kernel_t)(DraftParams, int);
bg_kernel_t attn_mfma_block_kernel(int G, int HD) {
    if (HD == 128) {
        switch (G) {
        case 1: return k_attn_mfma_block<1, 128>;
        case 2: return k_attn_mfma_block<2, 128>;
        case 4: return k_attn_mfma_block<4, 128>;
        case 8: return k_attn_mfma_block<8, 128>;
        }
    } else if (HD == 64) {
        switch (G) {
        case 1: return k_attn_mfma_block<1, 64>;
        case 2: return k_attn_mfma_block<2, 64>;
        case 4: return k_attn_mfma_block<4, 64>;
        case 8: return k_attn_mfma_block<8, 64>;
        }
    }
    return nullptr;
}
// lpt: the launch hands its items out through the counter (more items than workgroups)
bg_kernel_t attn_mfma_kernel(int G, int HD, bool lpt) {
    if (HD == 128) {
        switch (G) {
        case 1: return lpt ? k_attn_mfma_lpt<1, 128> : k_attn_mfma<1, 128>;
        case 2: return lpt ? k_attn_mfma_lpt<2, 128> : k_attn_mfma<2, 128>;
        case 4: return lpt ? k_attn_mfma_lpt<4, 128> : k_attn_mfma<4, 128>;
        case 8: return lpt ? k_attn_mfma_lpt<8, 128> : k_attn_mfma<8, 128>;
        }
    } else if (HD == 64) {
        switch (G) {
        case 1: return lpt ? k_attn_mfma_lpt<1, 64> : k_attn_mfma<1, 64>;
        case 2: return lpt ? k_attn_mfma_lpt<2, 64> : k_attn_mfma<2, 64>;
        case 4: return lpt ? k_attn_mfma_lpt<4, 64> : k_attn_mfma<4, 64>;
        case 8: return lpt ? k_attn_mfma_lpt<8, 64> : k_attn_mfma<8, 64>;
        }
    }
    return nullptr;
}
template <int PH>
bg_kernel_t pick_na(int na) {
    return na == 1 ? k_bgemv<PH, 1> : na == 2 ? k_bgemv<PH, 2> : k_bgemv<PH, 4>;
}
bg_kernel_t pick(int phase, int na) {
    switch (phase) {
    case BG_PROJ: return pick_na<BG_PROJ>(na);
    case BG_QKV: return pick_na<BG_QKV>(na);
    case BG_OPROJ: return pick_na<BG_OPROJ>(na);
    case BG_GATEUP: return pick_na<BG_GATEUP>(na);
    case BG_DOWN: return pick_na<BG_DOWN>(na);
    default: return pick_na<BG_LMHEAD>(na);
    }
}
// the tilings of the many-row matrix products
typedef void (*rows_kernel_t)(DraftParams, int, int);
struct RowsTileInfo {
    int bm, bn, lds;
    double step_us; // one reduction step of a workgroup that has its CU to itself
};
template <class T>
constexpr RowsTileInfo rows_tile_info(double step_us) {
    return RowsTileInfo{T::BM, T::BN, T::kLds, step_us};
}
constexpr int kRowsTiles = 3;
constexpr RowsTileInfo kRowsTile[kRowsTiles] = {rows_tile_info<RowsTile<4, 2, 8>>(1.3), rows_tile_info<RowsTile<2, 4, 8>>(1.3),
                                                rows_tile_info<RowsTile<2, 4, 6>>(1.0)};
constexpr int kRowsMinSteps = 8;           // reduction steps a part keeps at least
constexpr double kRowsFixedUs = 8.0;       // of a workgroup besides its steps
constexpr double kRowsEpilogueUs = 6.0;    // the launch that adds the parts
constexpr double kRowsPartUs = 8.0 / 5e6;  // a float of the parts written and read
template <int PH>
rows_kernel_t pick_rows(int tile) {
    return tile == 0 ? k_rows_gemm<PH, 4, 2, 8> : tile == 1 ? k_rows_gemm<PH, 2, 4, 8> : k_rows_gemm<PH, 2, 4, 6>;
}
rows_kernel_t rows_kernel(int phase, int tile) {
    switch (phase) {
    case BG_PROJ: return pick_rows<BG_PROJ>(tile);
    case BG_QKV: return pick_rows<BG_QKV>(tile);
    case BG_OPROJ: return pick_rows<BG_OPROJ>(tile);
    case BG_GATEUP: return pick_rows<BG_GATEUP>(tile);
    case BG_DOWN: return pick_rows<BG_DOWN>(tile);
    case BG_LMHEAD: return pick_rows<BG_LMHEAD>(tile);
    default: return pick_rows<kHeadLogits>(tile);
    }
}
void (*rows_epilogue_kernel(int phase))(DraftParams, int, int, int) {
    switch (phase) {
    case BG_PROJ: return k_rows_epilogue<BG_PROJ>;
    case BG_QKV: return k_rows_epilogue<BG_QKV>;
    case BG_OPROJ: return k_rows_epilogue<BG_OPROJ>;
    case BG_GATEUP: return k_rows_epilogue<BG_GATEUP>;
    default: return k_rows_epilogue<BG_DOWN>;
    }
}
int tiles_for(int nb) { return nb <= 16 ? 1 : nb <= 32 ? 2 : 4; }
template <int PH>
bg_kernel_t pick_epilogue_na(int na) {
    return na == 1 ? k_bepilogue<PH, 1> : na == 2 ? k_bepilogue<PH, 2> : k_bepilogue<PH, 4>;
}
bg_kernel_t pick_epilogue(int phase, int na) {
    switch (phase) {
    case BG_PROJ: return pick_epilogue_na<BG_PROJ>(na);
    case BG_QKV: return pick_epilogue_na<BG_QKV>(na);
    case BG_OPROJ: return pick_epilogue_na<BG_OPROJ>(na);
    case BG_GATEUP: return pick_epilogue_na<BG_GATEUP>(na);
    case BG_DOWN: return pick_epilogue_na<BG_DOWN>(na);
    default: return pick_epilogue_na<BG_LMHEAD>(na);
    }
}

} // namespace

size_t bgemv_lds_bytes(int rows_per_group) { return batch_lds_bytes(rows_per_group); }

int batch_epilogue_grid(int phase, const DraftParams &p, int na) {
    const int rows = phase == BG_QKV ? p.qkv_dim : phase == BG_GATEUP ? p.F : phase == BG_LMHEAD ? p.n : p.d;
    const int slots = (rows + 15) / 16 * na;
    return std::min((slots + kWaves - 1) / kWaves, 1024);
}

size_t attn_mfma_lds_bytes(int G, int HD) {
    switch (HD * 16 + G) {
    case 128 * 16 + 1: return sizeof(AttnMfmaLds<1, 128>);
    case 128 * 16 + 2: return sizeof(AttnMfmaLds<2, 128>);
    case 128 * 16 + 4: return sizeof(AttnMfmaLds<4, 128>);
    case 128 * 16 + 8: return sizeof(AttnMfmaLds<8, 128>);
    case 64 * 16 + 1: return sizeof(AttnMfmaLds<1, 64>);
    case 64 * 16 + 2: return sizeof(AttnMfmaLds<2, 64>);
    case 64 * 16 + 4: return sizeof(AttnMfmaLds<4, 64>);
    case 64 * 16 + 8: return sizeof(AttnMfmaLds<8, 64>);
    }
    return 0;
}

size_t attn_mfma_block_lds_bytes(int G, int HD) {
    switch (HD * 16 + G) {
    case 128 * 16 + 1: return sizeof(AttnMfmaLds<1, 128, 16>);
    case 128 * 16 + 2: return sizeof(AttnMfmaLds<2, 128, 8>);
    case 128 * 16 + 4: return sizeof(AttnMfmaLds<4, 128, 4>);
    case 128 * 16 + 8: return sizeof(AttnMfmaLds<8, 128, 2>);
    case 64 * 16 + 1: return sizeof(AttnMfmaLds<1, 64, 16>);
    case 64 * 16 + 2: return sizeof(AttnMfmaLds<2, 64, 8>);
    case 64 * 16 + 4: return sizeof(AttnMfmaLds<4, 64, 4>);
    case 64 * 16 + 8: return sizeof(AttnMfmaLds<8, 64, 2>);
    }
    return 0;
}

void launch_attn_mfma(int G, int HD, const DraftParams &p, int step, int grid, size_t lds, hipStream_t st) {
    hipLaunchKernelGGL(attn_mfma_kernel(G, HD, p.attn_queue != nullptr), dim3(grid), dim3(kBlock), lds, st, p, step);
}
void launch_attn_mfma_block(int G, int HD, const DraftParams &p, int step, int grid, size_t lds, hipStream_t st) {
    hipLaunchKernelGGL(attn_mfma_block_kernel(G, HD), dim3(grid), dim3(kBlock), lds, st, p, step);
}

bool batch_allow_lds(size_t lds_limit) {
    bool ok = true;
    for (int ph = 0; ph <= kHeadLogits; ++ph)
        for (int t = 0; t < kRowsTiles; ++t)
            ok = ok && hipFuncSetAttribute((const void *)rows_kernel(ph, t), hipFuncAttributeMaxDynamicSharedMemorySize,
                                           (int)lds_limit) == hipSuccess;
    for (int hd = 64; hd <= 128; hd *= 2)
        for (int g = 1; g <= 8; g *= 2)
            ok = ok && hipFuncSetAttribute((const void *)attn_mfma_kernel(g, hd, false),
                                           hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds_limit) == hipSuccess &&
                 hipFuncSetAttribute((const void *)attn_mfma_kernel(g, hd, true),
                                     hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds_limit) == hipSuccess &&
                 hipFuncSetAttribute((const void *)attn_mfma_block_kernel(g, hd),
                                     hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds_limit) == hipSuccess;
    for (int ph = 0; ph < BG_COUNT; ++ph)
        for (int na = 1; na <= 4; na *= 2)
            ok = ok && hipFuncSetAttribute((const void *)pick(ph, na), hipFuncAttributeMaxDynamicSharedMemorySize,
                                           (int)lds_limit) == hipSuccess;
    return ok;
}

void launch_bgemv(int phase, const DraftParams &p, int step, int grid, size_t lds, hipStream_t st) {
    const int na = tiles_for(p.nb);
    hipLaunchKernelGGL(pick(phase, na), dim3(grid), dim3(kBlock), lds, st, p, step);
    if (p.bg_sep[phase]) // one wave per (tile or pair of tiles, sequence tile)
        hipLaunchKernelGGL(pick_epilogue(phase, na),
                           dim3(phase == BG_LMHEAD ? p.head_grid : batch_epilogue_grid(phase, p, na)), dim3(kBlock), 0, st,
                           p, step);
}

namespace {
int rows_k(int phase, const DraftParams &p) { // reduction length of a phase
    return phase == BG_PROJ ? 2 * p.d : phase == BG_OPROJ ? p.qd : phase == BG_DOWN ? p.F : p.d;
}
int rows_n(int phase, const DraftParams &p) { // weight rows, in whole tiles of sixteen
    auto rows16 = [](int rows) { return (rows + 15) / 16 * 16; };
    return phase == BG_QKV      ? rows16(p.qkv_dim)
           : phase == BG_GATEUP ? 2 * rows16(p.F)
           : phase >= BG_LMHEAD ? rows16(p.n)
                                : p.d;
}
// The tiling and the number of reduction parts with the shortest estimated time: rounds of one workgroup per CU, each its
// share of the steps, and the parts' sums written and read once.  The constants are this kernel's own times at 512 rows
// (a step of 1.3 us in long reductions, 8 us from launch to first step and from last step to end).  Parts pay where a
// phase has few tiles: 4096 weight rows at 512 rows are 32 tiles of 256 x 256 and take 84 us in eight parts, 270 in one.
struct RowsPlan {
    int tile, kp, mb, nb;
};
RowsPlan rows_plan(int phase, const DraftParams &p, int cus, size_t part_floats) {
    const int steps = rows_k(phase, p) / kRgBK, n = rows_n(phase, p);
    RowsPlan best{};
    double best_us = 1e30;
    for (int t = 0; t < kRowsTiles; ++t) {
        const RowsTileInfo &ti = kRowsTile[t];
        const int mb = (p.B + ti.bm - 1) / ti.bm, nb = (n + ti.bn - 1) / ti.bn;
        for (int kp = 1; kp <= (phase >= BG_LMHEAD ? 1 : 16) && (kp == 1 || steps / kp >= kRowsMinSteps); ++kp) {
            const double sums = (double)kp * n * mb * ti.bm; // floats of the parts
            if (kp > 1 && sums > (double)part_floats) break;
            const int rounds = (mb * nb * kp + cus - 1) / cus;
            const double us = rounds * (kRowsFixedUs + (steps + kp - 1) / kp * ti.step_us) +
                              (kp > 1 ? kRowsEpilogueUs + sums * kRowsPartUs : 0.0);
            if (us < best_us) {
                best_us = us;
                best = RowsPlan{t, kp, mb, nb};
            }
        }
    }
    return best;
}
} // namespace

bool rows_gemm_serves(int phase, const DraftParams &p) { return rows_k(phase, p) % kRgBK == 0; }
int rows_head_cands(const DraftParams &p, int cus) { return rows_plan(BG_LMHEAD, p, cus, 0).nb; }
void launch_rows_gemm(int phase, bool logits_only, const DraftParams &p, int step, int cus, size_t part_floats,
                      hipStream_t st) {
    const RowsPlan pl = rows_plan(phase, p, cus, part_floats);
    const int ph = phase == BG_LMHEAD && logits_only ? kHeadLogits : phase;
    const int units = pl.nb * pl.kp; // (N block, part) pairs: the M blocks of eight neighbouring ones form one group
    hipLaunchKernelGGL(rows_kernel(ph, pl.tile), dim3((units + 7) / 8 * 8 * pl.mb), dim3(kBlock), kRowsTile[pl.tile].lds, st,
                       p, step, pl.kp);
    if (pl.kp > 1) {
        const int rt = pl.mb * kRowsTile[pl.tile].bm / 16, live = (p.B + 15) / 16;
        const int groups = (rows_n(phase, p) / 16 / (phase == BG_GATEUP ? 2 : 1) + kWaves - 1) / kWaves;
        hipLaunchKernelGGL(rows_epilogue_kernel(phase), dim3(live, std::max(1, std::min(groups, 8 * cus / live))), dim3(kBlock),
                           0, st, p, step, pl.kp, rt);
    }
}

void launch_bprep(const DraftParams &p, int step, hipStream_t st) {
    hipLaunchKernelGGL(k_bprep, dim3(p.B), dim3(kBlock), 0, st, p, step);
}

} // namespace mtp
