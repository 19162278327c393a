// The tiled matrix products whose reduction ends in half a step (widths of an odd number of 32s, tiles with steps of 64) for
// gfx950.  In a code object of their own they leave the place of the other kernels' code alone, which identical kernels turned out
// to depend on: with these among them three steps of a 4096-wide head took 639 us instead of 632 at forty sequences, 703 instead
// of 698 at sixty-four.
#include <hip/hip_runtime.h>

#include "batch_launch.h"
#include "rows_kernels.h"

namespace mtp {
namespace {
typedef RowsTile<2, 2, 4, 2, 4, 64, true> Rows64x128Half;
typedef RowsTile<1, 2, 4, 2, 6, 64, true> Rows32x128Half;
typedef RowsTile<1, 1, 8, 1, 7, 64, true> Rows16x128Half;
template <int PH>
rows_kernel_t pick(int tile) {
    switch (tile) { // the plan's tilings from kRowsHalf on
    case 4: return k_rows_gemm<PH, Rows64x128Half>;
    case 5: return k_rows_gemm<PH, Rows32x128Half>;
    case 6: return k_rows_gemm<PH, Rows16x128Half>;
    default: return nullptr;
    }
}
} // namespace

rows_kernel_t rows_half_kernel(int phase, int tile) {
    switch (phase) { // (never one of the projections: 2 d and Hq * hd are multiples of 64)
    case BG_QKV: return pick<BG_QKV>(tile);
    case BG_GATEUP: return pick<BG_GATEUP>(tile);
    case BG_DOWN: return pick<BG_DOWN>(tile);
    case BG_LMHEAD:
    case kHeadLogits: return pick<BG_LMHEAD>(tile);
    default: return nullptr;
    }
}

} // namespace mtp
