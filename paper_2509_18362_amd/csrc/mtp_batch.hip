// Kernels of the batched draft path (two or more sequences per call) for gfx950.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "attn_mfma.h"
#include "attn_rows.h"
#include "batch.h"
#include "batch_launch.h"
#include "rows_kernels.h"

namespace mtp {
namespace {

template <int PH, int NA>
__global__ __launch_bounds__(kBlock) void k_bgemv(DraftParams p, int step) {
    extern __shared__ __align__(16) char smem[];
    if constexpr (PH == BG_DOWN) {
        BgDown ph(p);
        bgemv_lds<NA>(p, ph, p.bg_rg[PH], p.bg_kp[PH], smem);
    } else {
        BgHead ph(p, step);
        bgemv_lds<NA>(p, ph, p.bg_rg[PH], p.bg_kp[PH], smem);
    }
}

// (the only phase that comes to the batched core with its reduction split)
template <int NA>
__global__ __launch_bounds__(kBlock) void k_bepilogue_down(DraftParams p, int step) {
    __shared__ __align__(16) char smem[kBatchMaxSeq * 4];
    BgDown ph(p);
    phase_bepilogue<NA>(p, ph, p.bg_kp[BG_DOWN], smem);
}

__global__ __launch_bounds__(kBlock) void k_bprep(DraftParams p, int step) {
    __shared__ __align__(16) char smem[256];
    phase_bprep(p, step, smem);
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

// a block of positions in small workgroups
template <int G, int HD, int W>
__global__ __launch_bounds__(W *kWave, 2) void k_attn_rows(DraftParams p) {
    extern __shared__ __align__(16) char smem[];
    attn_rows<G, HD, W>(p, smem);
}

typedef void (*bg_kernel_t)(DraftParams, int);
struct AttnRowsKernel {
    void (*fn)(DraftParams);
    size_t lds;
};
template <int W>
AttnRowsKernel attn_rows_kernel_of(int G, int HD) {
    switch (HD * 16 + G) {
    case 128 * 16 + 1: return {k_attn_rows<1, 128, W>, sizeof(AttnRowsLds<1, 128, W>)};
    case 128 * 16 + 2: return {k_attn_rows<2, 128, W>, sizeof(AttnRowsLds<2, 128, W>)};
    case 128 * 16 + 4: return {k_attn_rows<4, 128, W>, sizeof(AttnRowsLds<4, 128, W>)};
    case 128 * 16 + 8: return {k_attn_rows<8, 128, W>, sizeof(AttnRowsLds<8, 128, W>)};
    case 64 * 16 + 1: return {k_attn_rows<1, 64, W>, sizeof(AttnRowsLds<1, 64, W>)};
    case 64 * 16 + 2: return {k_attn_rows<2, 64, W>, sizeof(AttnRowsLds<2, 64, W>)};
    case 64 * 16 + 4: return {k_attn_rows<4, 64, W>, sizeof(AttnRowsLds<4, 64, W>)};
    case 64 * 16 + 8: return {k_attn_rows<8, 64, W>, sizeof(AttnRowsLds<8, 64, W>)};
    }
    return {nullptr, 0};
}
AttnRowsKernel attn_rows_kernel(int G, int HD, int waves) { return waves == 4 ? attn_rows_kernel_of<4>(G, HD) : attn_rows_kernel_of<8>(G, HD); }
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
// What the tiled products do not serve: the down projection of reduction lengths that are no multiple of 32 and heads of more
// rows than the tiles have candidates for.
constexpr int kCorePhases[] = {BG_DOWN, BG_LMHEAD};
bg_kernel_t pick(int phase, int na) {
    if (phase == BG_DOWN) return na == 2 ? k_bgemv<BG_DOWN, 2> : k_bgemv<BG_DOWN, 4>;
    return na == 2 ? k_bgemv<BG_LMHEAD, 2> : k_bgemv<BG_LMHEAD, 4>;
}
typedef RowsTile<4, 4, 2, 8, 3> Rows256x256;
typedef RowsTile<4, 2, 4, 8, 3> Rows128x512;
typedef RowsTile<4, 2, 4, 6, 3> Rows128x384;
typedef RowsTile<2, 2, 4, 4, 3, 64> Rows64x256;
typedef RowsTile<2, 2, 4, 2, 4, 64> Rows64x128;
typedef RowsTile<1, 2, 4, 2, 6, 64> Rows32x128;
typedef RowsTile<1, 1, 8, 1, 7, 64> Rows16x128;
template <class T>
constexpr bool is_tile(int t) { // the plan's entry t describes T
    return kRowsTile[t].bm == T::BM && kRowsTile[t].bn == T::BN && kRowsTile[t].bk == T::BK && kRowsTile[t].lds == T::kLds;
}
static_assert(is_tile<Rows256x256>(0) && is_tile<Rows128x512>(1) && is_tile<Rows128x384>(2) && is_tile<Rows64x256>(3) &&
                  is_tile<Rows64x128>(4) && is_tile<Rows32x128>(5) && is_tile<Rows16x128>(6),
              "the kernels below in the order of the plan's tilings");
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
rows_kernel_t rows_kernel(int phase, int tile, bool half) {
    if (half) return rows_half_kernel(phase, tile);
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
int tiles_for(int nb) { return nb <= 32 ? 2 : 4; }

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

void launch_attn_rows(const DraftParams &p, int cus, hipStream_t st) {
    const int G = p.Hq / p.Hkv, jp = 16 / G, groups = p.ext_B * ((p.B / p.ext_B + jp - 1) / jp) * p.Hkv;
    const int waves = attn_rows_waves(groups, cus);
    const AttnRowsKernel k = attn_rows_kernel(G, p.hd, waves);
    hipLaunchKernelGGL(k.fn, dim3(groups), dim3(waves * kWave), k.lds, st, p);
}

bool batch_allow_lds(size_t lds_limit, const mtp_config &c) {
    bool ok = true;
    auto allow = [&](const void *kernel) {
        ok = ok && (!kernel || hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds_limit) == hipSuccess);
    };
    const int G = c.n_q_heads / c.n_kv_heads;
    for (bool lpt : {false, true}) allow((const void *)attn_mfma_kernel(G, c.head_dim, lpt));
    allow((const void *)attn_mfma_block_kernel(G, c.head_dim));
    for (int waves : {4, 8}) allow((const void *)attn_rows_kernel(G, c.head_dim, waves).fn);
    if (c.max_batch < 2) return ok; // one sequence: the row-streaming kernels
    ok = ok && few_allow_lds(lds_limit);
    for (int ph = 0; ph <= kHeadLogits; ++ph)
        for (int t = 0; t < kRowsTiles; ++t) {
            if (c.max_batch <= kRowsFew && kRowsTile[t].bm > 64) continue; // (rows_plan)
            allow((const void *)rows_kernel(ph, t, false));
            if (c.d_model % 64 || c.d_ffn % 64) allow((const void *)rows_kernel(ph, t, true));
        }
    for (int ph : kCorePhases)
        for (int na : {2, 4}) allow((const void *)pick(ph, na));
    return ok;
}

void launch_bgemv(int phase, const DraftParams &p, int step, int grid, size_t lds, hipStream_t st) {
    const int na = tiles_for(p.nb);
    hipLaunchKernelGGL(pick(phase, na), dim3(grid), dim3(kBlock), lds, st, p, step);
    if (p.bg_sep[phase]) // (BG_DOWN) one wave per (tile, sequence tile)
        hipLaunchKernelGGL(na == 2 ? k_bepilogue_down<2> : k_bepilogue_down<4>,
                           dim3(std::min((p.d / 16 * na + kWaves - 1) / kWaves, 1024)), dim3(kBlock), 0, st, p, step);
}

namespace {
RowsCall rows_call(int phase, const DraftParams &p) {
    auto rows16 = [](int rows) { return (rows + 15) / 16 * 16; };
    RowsCall c;
    c.K = phase == BG_PROJ ? 2 * p.d : phase == BG_OPROJ ? p.qd : phase == BG_DOWN ? p.F : p.d;
    c.n = phase == BG_QKV      ? rows16(p.qkv_dim)
          : phase == BG_GATEUP ? 2 * rows16(p.F)
          : phase == BG_LMHEAD ? rows16(p.n)
                               : p.d;
    c.rows = p.seq_hi - p.seq_lo;
    c.head = phase == BG_LMHEAD;
    c.pairs = phase == BG_GATEUP;
    return c;
}
} // namespace

RowsRoute rows_route(int phase, const DraftParams &p, bool all_few, int cus) { return rows_route(rows_call(phase, p), all_few, cus); }
int rows_head_cands(const DraftParams &p, int cus, size_t part_floats) {
    const RowsCall c = rows_call(BG_LMHEAD, p);
    const RowsPlan pl = rows_plan(c, cus, part_floats);
    return pl.kp > 1 ? rows_epilogue_groups(c, cus) : pl.nb;
}
void launch_rows_gemm(int phase, bool logits_only, const DraftParams &p, int step, int cus, size_t part_floats,
                      hipStream_t st) {
    const RowsCall c = rows_call(phase, p);
    const RowsPlan pl = rows_plan(c, cus, part_floats);
    const int ph = phase == BG_LMHEAD && logits_only ? kHeadLogits : phase;
    const int units = pl.nb * pl.kp; // (N block, part) pairs: the M blocks of eight neighbouring ones form one group
    hipLaunchKernelGGL(rows_kernel(ph, pl.tile, c.K % kRowsTile[pl.tile].bk != 0), dim3((units + 7) / 8 * 8 * pl.mb), dim3(kBlock), kRowsTile[pl.tile].lds, st,
                       p, step, pl.kp);
    if (pl.kp > 1)
        hipLaunchKernelGGL(rows_epilogue_kernel(ph), dim3((c.rows + 15) / 16, rows_epilogue_groups(c, cus)), dim3(kBlock), 0, st,
                           p, step, pl.kp, pl.mb * kRowsTile[pl.tile].bm / 16);
}

void launch_bprep(const DraftParams &p, int step, hipStream_t st) {
    hipLaunchKernelGGL(k_bprep, dim3(p.B), dim3(kBlock), 0, st, p, step);
}

} // namespace mtp
