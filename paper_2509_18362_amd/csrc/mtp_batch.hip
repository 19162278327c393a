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

// (the only phase that more than 16 rows take to the batched core with its reduction split: see rows_gemm_serves)
template <int NA>
__global__ __launch_bounds__(kBlock) void k_bepilogue_down(DraftParams p, int step) {
    __shared__ __align__(16) char smem[kWaves * kBatchMaxSeq * 8 + kBatchMaxSeq * 4];
    BgDown ph(p);
    phase_bepilogue<NA>(p, ph, p.bg_kp[BG_DOWN], smem);
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
template <int PH, class T>
__global__ __launch_bounds__(kBlock, 2) void k_rows_gemm(DraftParams p, int step, int KP) {
    extern __shared__ __align__(16) char smem[];
    with_phase<PH>(step, [&](auto make) { rows_gemm<T, decltype(make(p))>(p, make, KP, smem); });
}
template <int PH>
__global__ __launch_bounds__(kBlock) void k_rows_epilogue(DraftParams p, int step, int KP, int RT) {
    __shared__ __align__(16) float scale[16 + kWaves * 16 * 2]; // the rows' norm scales, the waves' candidates
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
// More than 16 rows take the tiled products wherever those serve: the batched core then runs the down projection of
// reduction lengths that are no multiple of 32 and heads of more rows than the tiles have candidates for.
template <int PH>
bg_kernel_t pick_na(int na) {
    if constexpr (PH == BG_DOWN || PH == BG_LMHEAD)
        return na == 1 ? k_bgemv<PH, 1> : na == 2 ? k_bgemv<PH, 2> : k_bgemv<PH, 4>;
    else
        return na == 1 ? k_bgemv<PH, 1> : nullptr;
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
    int bm, bn, bk, lds;
    double step_us; // one reduction step of a workgroup that has its CU to itself
};
template <class T>
constexpr RowsTileInfo rows_tile_info(double step_us) {
    return RowsTileInfo{T::BM, T::BN, T::BK, T::kLds, step_us};
}
typedef RowsTile<4, 4, 2, 8, 3> Rows256x256;
typedef RowsTile<4, 2, 4, 8, 3> Rows128x512;
typedef RowsTile<4, 2, 4, 6, 3> Rows128x384;
typedef RowsTile<2, 2, 4, 4, 3, 64> Rows64x256;
typedef RowsTile<2, 2, 4, 2, 4, 64> Rows64x128;
typedef RowsTile<1, 2, 4, 2, 6, 64> Rows32x128;
typedef RowsTile<1, 1, 8, 1, 7, 64> Rows16x128;
constexpr int kRowsTiles = 7;
constexpr RowsTileInfo kRowsTile[kRowsTiles] = {
    rows_tile_info<Rows256x256>(1.3), rows_tile_info<Rows128x512>(1.3), rows_tile_info<Rows128x384>(1.0),
    rows_tile_info<Rows64x256>(1.3), rows_tile_info<Rows64x128>(0.8), rows_tile_info<Rows32x128>(0.55),
    rows_tile_info<Rows16x128>(0.52)};
constexpr int kRowsMinSteps = 8;           // reduction steps a part keeps at least
constexpr double kRowsFixedUs = 6.0;       // of a workgroup besides its steps
constexpr double kRowsEpilogueUs = 7.5;    // the launch that adds the parts
constexpr double kRowsPartUs = 8.0 / 5e6;  // a float of the parts written and read
constexpr double kRowsReadUs = 1.0 / 5.5e6; // a byte of weights, per block of rows (the blocks after the first from L2)
template <int PH>
rows_kernel_t pick_rows(int tile) {
    switch (tile) {
    case 0: return k_rows_gemm<PH, Rows256x256>;
    case 1: return k_rows_gemm<PH, Rows128x512>;
    case 2: return k_rows_gemm<PH, Rows128x384>;
    case 3: return k_rows_gemm<PH, Rows64x256>;
    case 4: return k_rows_gemm<PH, Rows64x128>;
    case 5: return k_rows_gemm<PH, Rows32x128>;
    default: return k_rows_gemm<PH, Rows16x128>;
    }
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
    case BG_DOWN: return k_rows_epilogue<BG_DOWN>;
    case BG_LMHEAD: return k_rows_epilogue<BG_LMHEAD>;
    default: return k_rows_epilogue<kHeadLogits>;
    }
}
int tiles_for(int nb) { return nb <= 16 ? 1 : nb <= 32 ? 2 : 4; }

} // namespace

size_t bgemv_lds_bytes(int rows_per_group) { return batch_lds_bytes(rows_per_group); }

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
            ok = ok && (!pick(ph, na) || hipFuncSetAttribute((const void *)pick(ph, na), hipFuncAttributeMaxDynamicSharedMemorySize,
                                                             (int)lds_limit) == hipSuccess);
    return ok;
}

void launch_bgemv(int phase, const DraftParams &p, int step, int grid, size_t lds, hipStream_t st) {
    const int na = tiles_for(p.nb);
    hipLaunchKernelGGL(pick(phase, na), dim3(grid), dim3(kBlock), lds, st, p, step);
    if (p.bg_sep[phase]) // (BG_DOWN) one wave per (tile, sequence tile)
        hipLaunchKernelGGL(na == 1 ? k_bepilogue_down<1> : na == 2 ? k_bepilogue_down<2> : k_bepilogue_down<4>,
                           dim3(std::min((p.d / 16 * na + kWaves - 1) / kWaves, 1024)), dim3(kBlock), 0, st, p, step);
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
// share of the steps (or the time HBM takes for the weights, if that is longer), and the parts' sums written and read
// once.  The constants are this kernel's own times on the 7B-shaped head: a step of a workgroup in long reductions, what a
// workgroup takes from launch to first step and from last step to end, the launch that adds the parts.  Parts pay where
// a phase has few tiles: 4096 weight rows at 512 rows are 32 tiles of 256 x 256 and take 84 us in eight parts, 270 in one.
struct RowsPlan {
    int tile, kp, mb, nb;
};
RowsPlan rows_plan(int phase, const DraftParams &p, int cus, size_t part_floats) {
    const int K = rows_k(phase, p), n = rows_n(phase, p), rows = p.seq_hi - p.seq_lo;
    RowsPlan best{};
    double best_us = 1e30;
    for (int t = kRowsTiles - 1; t >= 0; --t) { // (small tiles first: they stay where HBM bounds all alike)
        const RowsTileInfo &ti = kRowsTile[t];
        if (K % ti.bk) continue;
        const int steps = K / ti.bk;
        const int mb = (rows + ti.bm - 1) / ti.bm, nb = (n + ti.bn - 1) / ti.bn;
        const double weights_us = (double)n * K * 2 * mb * kRowsReadUs;
        for (int kp = 1; kp <= 16 && (kp == 1 || K / 32 / kp >= kRowsMinSteps); ++kp) {
            const double sums = (double)kp * n * mb * ti.bm; // floats of the parts
            if (kp > 1 && sums > (double)part_floats) break;
            if (phase == BG_LMHEAD && kp == 1 && nb > kMaxHeadCands) continue; // a candidate per row and N block
            const int rounds = (mb * nb * kp + cus - 1) / cus;
            const double us = std::max(weights_us, rounds * ((steps + kp - 1) / kp * ti.step_us)) + rounds * kRowsFixedUs +
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

bool rows_gemm_serves(int phase, const DraftParams &p, int cus) {
    const int K = rows_k(phase, p);
    if (K % kRgBK) return false;
    if (phase == BG_LMHEAD && rows_n(phase, p) > Rows128x512::BN * kMaxHeadCands) return false; // no room for the candidates
    if (p.seq_hi - p.seq_lo > 16) return true;
    // Up to 16 rows the batched core's plain kernel (waves split the reduction) streams large matrices as fast, and adds its
    // parts by itself; but it takes 10 us (tiny) to 14 us before its workgroups' sums are added up, against 5 us, or 10 with
    // the launch that adds the parts.  Measured at five rows (us, this kernel / that one): 4096 x 2048 11 / 14, 2048 x 6144
    // 13 / 17, 12288 x 2048 14 / 17, 8192 x 2048 of a head 15 / 18; at sixteen rows 4096 x 4096 17 / 17.5, 6144 x 4096
    // 21 / 19.5, 4096 x 8192 23 / 21, 22016 x 4096 40 / 35; a head that fills the chip in one part, 32768 x 4096: 53 / 59
    // (a head of more blocks than candidates takes a larger tile: 151680 x 4096 at sixteen rows 260 / 247).
    const int n = rows_n(phase, p);
    return K <= 2048 || (double)n * K * 2 <= 32e6 ||
           (phase == BG_LMHEAD && n >= Rows16x128::BN * cus && n <= Rows16x128::BN * kMaxHeadCands);
}
namespace {
// workgroups per row tile of the kernel that adds the parts
int rows_epilogue_groups(int phase, const DraftParams &p, int cus) {
    const int live = (p.seq_hi - p.seq_lo + 15) / 16, per_wave = rows_n(phase, p) / 16 / (phase == BG_GATEUP ? 2 : 1);
    return std::max(1, std::min({(per_wave + kWaves - 1) / kWaves, 8 * cus / live, kMaxHeadCands}));
}
} // namespace
int rows_head_cands(const DraftParams &p, int cus, size_t part_floats) {
    const RowsPlan pl = rows_plan(BG_LMHEAD, p, cus, part_floats);
    return pl.kp > 1 ? rows_epilogue_groups(BG_LMHEAD, p, cus) : pl.nb;
}
void launch_rows_gemm(int phase, bool logits_only, const DraftParams &p, int step, int cus, size_t part_floats,
                      hipStream_t st) {
    const RowsPlan pl = rows_plan(phase, p, cus, part_floats);
    const int ph = phase == BG_LMHEAD && logits_only ? kHeadLogits : phase;
    const int units = pl.nb * pl.kp; // (N block, part) pairs: the M blocks of eight neighbouring ones form one group
    hipLaunchKernelGGL(rows_kernel(ph, pl.tile), dim3((units + 7) / 8 * 8 * pl.mb), dim3(kBlock), kRowsTile[pl.tile].lds, st,
                       p, step, pl.kp);
    if (pl.kp > 1)
        hipLaunchKernelGGL(rows_epilogue_kernel(ph), dim3((p.seq_hi - p.seq_lo + 15) / 16, rows_epilogue_groups(phase, p, cus)), dim3(kBlock),
                           0, st, p, step, pl.kp, pl.mb * kRowsTile[pl.tile].bm / 16);
}

void launch_bprep(const DraftParams &p, int step, hipStream_t st) {
    hipLaunchKernelGGL(k_bprep, dim3(p.B), dim3(kBlock), 0, st, p, step);
}

} // namespace mtp
