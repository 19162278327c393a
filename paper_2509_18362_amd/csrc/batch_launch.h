// Host-side entry points of the batched path (kernels live in mtp_batch.hip, the caller in mtp_draft.hip).
#pragma once
#include <hip/hip_runtime.h>

#include "../../include/mtp_draft.h"
#include "phases.h"
#include "rows_plan.h"

namespace mtp {

// dynamic LDS of a batched matrix phase whose row groups hold at most `rows_per_group` rows
size_t bgemv_lds_bytes(int rows_per_group);
// raises the dynamic-LDS limit of the batched and matrix-core attention kernels that calls of a handle with this configuration
// can take; false if a call failed
bool batch_allow_lds(size_t lds_limit, const mtp_config &c);
// the kernel of a matrix phase (BG_* index) over the rows p.seq_lo .. p.seq_hi - 1 (rows_plan.h)
RowsRoute rows_route(int phase, const DraftParams &p, bool all_few, int cus);
// one batched matrix phase (BG_* index) for the sequences [p.b0, p.b0 + p.nb)
void launch_bgemv(int phase, const DraftParams &p, int step, int grid, size_t lds, hipStream_t st);
// A matrix phase of the rows [p.b0, p.b0 + p.nb), at most sixteen (few_rows.h), on few_groups workgroups; the output head
// leaves as many candidates per row.
int few_groups(int phase, const DraftParams &p, int cus);
bool few_allow_lds(size_t lds_limit);
void launch_few(int phase, const DraftParams &p, int step, int cus, hipStream_t st);
// the preparation kernel before step `step` (step == K: after the last step), all sequences
void launch_bprep(const DraftParams &p, int step, hipStream_t st);

// A matrix phase (BG_* index) over the rows p.seq_lo .. p.seq_hi - 1 as one tiled matrix product (rows_gemm.h).  The output
// head leaves rows_head_cands candidates per row, or none where the caller wants logits only.  part_floats: room of the
// partial buffer.
int rows_head_cands(const DraftParams &p, int cus, size_t part_floats);
void launch_rows_gemm(int phase, bool logits_only, const DraftParams &p, int step, int cus, size_t part_floats,
                      hipStream_t st);

// the kernel of a phase and a tiling whose last reduction step is half a one (mtp_rows_half.hip); null: not needed
typedef void (*rows_kernel_t)(DraftParams, int, int);
rows_kernel_t rows_half_kernel(int phase, int tile);

// matrix-core attention (attn_mfma.h): dynamic LDS, and the launch for query-group size G and head dimension HD
size_t attn_mfma_lds_bytes(int G, int HD);
void launch_attn_mfma(int G, int HD, const DraftParams &p, int step, int grid, size_t lds, hipStream_t st);
// the same for a block of new positions per sequence whose keys and values are in the cache (p.kv_appended, p.ext_B):
// positions_per_item = 16 / G positions of a sequence share its key/value reads
size_t attn_mfma_block_lds_bytes(int G, int HD);
void launch_attn_mfma_block(int G, int HD, const DraftParams &p, int step, int grid, size_t lds, hipStream_t st);
// a block of new positions whose keys and values are in the cache: a small workgroup per KV head and 16 / G positions (attn_rows.h)
void launch_attn_rows(const DraftParams &p, int cus, hipStream_t st);

} // namespace mtp
