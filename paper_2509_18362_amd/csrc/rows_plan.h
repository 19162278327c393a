// Rules that choose a call's kernels: which kernel a matrix phase of several rows takes, which tiles, and how many reduction
// parts, a tiled matrix product (rows_gemm.h) runs with, and where one sequence takes a single launch.  Host code without HIP:
// the rules can be compiled and checked on their own.
#pragma once
#include <algorithm>
#include <cstddef>

namespace mtp {

constexpr int kMaxHeadCands = 1024; // candidates of the output head a sequence has room for
constexpr int kRgBK = 32;           // elements of the shortest reduction step

// One matrix phase over some rows of a call.
struct RowsCall {
    int K, n, rows; // reduction length, weight rows in whole tiles of sixteen, rows of activations
    bool head;      // leaves argmax candidates: one per row and block of weight rows, or per group of the adding launch
    bool pairs;     // gate/up: two tiles make one
};
struct RowsPlan {
    int tile, kp, mb, nb; // tiling, reduction parts, blocks of rows and of weight rows
    double us;            // estimated time
};

// the tilings of the many-row matrix products
struct RowsTileInfo {
    int bm, bn, bk, lds;
    double step_us; // one reduction step of a workgroup that has its CU to itself
};
constexpr int kRowsTiles = 7;
constexpr RowsTileInfo kRowsTile[kRowsTiles] = {
    {256, 256, 32, 3 * (2 * 256 + 256) * 64, 1.3}, {128, 512, 32, 3 * (2 * 128 + 512) * 64, 1.3},
    {128, 384, 32, 3 * (2 * 128 + 384) * 64, 1.0}, {64, 256, 64, 3 * (2 * 64 + 256) * 128, 1.3},
    {64, 128, 64, 4 * (2 * 64 + 128) * 128, 0.8},  {32, 128, 64, 6 * (2 * 32 + 128) * 128, 0.55},
    {16, 128, 64, 7 * (2 * 16 + 128) * 128, 0.52}};
constexpr int kRowsFew = 16;              // rows up to which few_rows.h is an alternative
constexpr int kRowsHalf = 4;               // the tilings from this one on take a last step that is half a one
constexpr int kRowsMinSteps = 8;           // reduction steps of 32 a part keeps at least
constexpr double kRowsFixedUs = 6.0;       // of a workgroup besides its steps
constexpr double kRowsEpilogueUs = 7.5;    // the launch that adds the parts
constexpr double kRowsPartUs = 8.0 / 5e6;  // a float of the parts written and read
constexpr double kRowsReadUs = 1.0 / 5.5e6; // a byte of weights, per block of rows (the blocks after the first from L2)

// The tiling and the number of reduction parts with the shortest estimated time: rounds of one workgroup per CU, each its
// share of the steps (or the time HBM takes for the weights, if that is longer), and the parts' sums written and read
// once.  The constants are this kernel's own times on the 7B-shaped head: a step of a workgroup in long reductions, what a
// workgroup takes from launch to first step and from last step to end, the launch that adds the parts.  Parts pay where
// a phase has few tiles: 4096 weight rows at 512 rows are 32 tiles of 256 x 256 and take 84 us in eight parts, 270 in one.
// part_floats: room of the partial buffer.
inline RowsPlan rows_plan(const RowsCall &c, int cus, size_t part_floats) {
    RowsPlan best{};
    best.us = 1e30;
    for (int t = kRowsTiles - 1; t >= 0; --t) { // (small tiles first: they stay where HBM bounds all alike)
        const RowsTileInfo &ti = kRowsTile[t];
        if (c.K % ti.bk && t < kRowsHalf) continue;
        // Few rows: no tiles of many times as many (their products with rows that are not there cost more than the estimate
        // says: 75841 x 3072 in tiles of 128 rows takes 18 us more than without them).  Where blocks of 128 weight rows would take a
        // second round, blocks of 256 (36000 x 4096 at sixteen rows: 12 us less than in 282 narrow blocks for 256 CUs).
        const int nb = (c.n + ti.bn - 1) / ti.bn;
        if (c.rows <= kRowsFew && (ti.bm > 64 || (ti.bn == 128 && nb > cus && c.K % 64 == 0))) continue;
        const int steps = (c.K + ti.bk - 1) / ti.bk;
        const int mb = (c.rows + ti.bm - 1) / ti.bm;
        const double weights_us = (double)c.n * c.K * 2 * mb * kRowsReadUs;
        for (int kp = 1; kp <= 16 && (kp == 1 || c.K / 32 / kp >= kRowsMinSteps); ++kp) {
            const double sums = (double)kp * c.n * mb * ti.bm; // floats of the parts
            if (kp > 1 && sums > (double)part_floats) break;
            if (c.head && kp == 1 && nb > kMaxHeadCands) continue; // a candidate per row and N block
            const int rounds = (mb * nb * kp + cus - 1) / cus;
            const double us = std::max(weights_us, rounds * ((steps + kp - 1) / kp * ti.step_us)) + rounds * kRowsFixedUs +
                              (kp > 1 ? kRowsEpilogueUs + sums * kRowsPartUs : 0.0);
            if (us < best.us) best = RowsPlan{t, kp, mb, nb, us};
        }
    }
    return best;
}

// workgroups per row tile of the kernel that adds the parts
inline int rows_epilogue_groups(const RowsCall &c, int cus) {
    const int live = (c.rows + 15) / 16, per_wave = c.n / 16 / (c.pairs ? 2 : 1);
    return std::max(1, std::min({(per_wave + 7) / 8, 8 * cus / live, kMaxHeadCands})); // (eight waves each)
}

// The tiled product serves the phase, and is the faster kernel.
inline bool rows_gemm_serves(const RowsCall &c, int cus) {
    if (c.K % kRgBK) return false;
    if (c.head && c.n > kRowsTile[1].bn * kMaxHeadCands) return false; // no room for the candidates
    if (c.rows > kRowsFew) return true;
    // Up to 16 rows (9 to 16 of narrow heads, and the lists of a larger batch: other calls take few_rows.h without asking) few_rows.h
    // with row-major activations is the alternative.  Both go in rounds of one workgroup per CU; this kernel is ahead while its
    // workgroups fit one round, the other, which deals tiles of sixteen rows evenly, beyond.  Gain of the tiled product over
    // few_rows.h, us per step, heads at 8 and 16 rows, K = 512 .. 4096:
    //   blocks of 128 in one round (up to 32768 rows): K <= 2048 or up to 32 MB -0.3 .. +4; larger heads +0.5 .. +6 where nine
    //   tenths of the round are there, -4 .. +3 below;
    //   blocks of 256: one round (33000 .. 65536 rows) +1.2 .. +6 (65536: -2 .. +6), two full ones (131072) -2.6 .. +5 up to K = 2048,
    //   -5 .. 0 from 3072 on; 0.58 of two (75841) -2.5 .. -16, 0.75 of two (98304) -2.5 .. -18, 0.77 of three (151680) -5 .. -32;
    //   reductions of an odd number of 32s, which have no blocks of 256, in two rounds and more: K = 544 and 1056 -1 .. +1, 1568 and 2016
    //   -1 .. -7 (33000 .. 65536 rows), -1 .. -36 beyond.
    // The body's phases at 9 and 16 rows, 384 .. 2048 wide: +2.5 .. +11 us per step together.
    const bool small = c.K <= 2048 || (double)c.n * c.K * 2 <= 32e6;
    if (!small && !c.head) return false;
    const int narrow = (c.n + 127) / 128, wide = (c.n + 255) / 256; // blocks of the two tiles that such calls take
    if (narrow <= cus) return small || 10 * narrow >= 9 * cus;
    if (c.K % 64 || wide > kMaxHeadCands) return false;
    return wide <= cus || (small && 10 * wide >= 9 * ((wide + cus - 1) / cus * cus));
}

// Kernels of the matrix phases of a call of `rows` rows (sequences, or positions of a block) of a head d wide.
enum RowsRoute : int { kOnFew, kOnTiles, kOnCore };
constexpr int kFewRows = 16, kFewPacked = 8; // few_rows.h: rows of a launch at most; up to eight, hi and lo halves in one operand
constexpr int kFewFrom = 384;                // 2..8 rows: widths from which on all phases take it
constexpr int kFewNarrow = 2048;             // 9..16 rows: widths up to which tiles are faster
// The whole call on few_rows.h, its activations in operand order.  Two steps against the kernels before it (batched core, tiles),
// us: 4096 wide 2 / 8 / 16 rows 336 / 355 / 365 -> 285 / 310 / 345 (16853-row head), 751 / 773 / 792 -> 658 / 690 / 737 (full); 2048
// wide 181 / 200 / 209 -> 168 / 190 / 218.  From nine rows on every workgroup reads twice its weights in activations: narrow matrices
// (few tiles, so few workgroups) are then faster in tiles, split over workgroups.  Below 384 wide a phase is one or two chunks of
// few_rows.h and the tiles are ahead: 256 wide, 2 / 8 rows 106 / 110 there and 102 / 107 in tiles (1024-row head), 109 / 115 and
// 103 / 109 (32768 rows), 122 / 128 and 113 / 120 (65536); 320 wide 113 / 120 and 108 / 116 (32768), within 1 % elsewhere; 384
// wide 106 / 113 and 108 / 116 (1024), 115 / 123 and 113 / 124 (32768).
inline bool rows_all_few(int rows, int d) {
    return rows <= kFewPacked ? d >= kFewFrom : rows <= kFewRows && d > kFewNarrow;
}
// A phase of the call (the output head: of the rows that share an id list).  What the tiles do not serve, or not as fast, takes
// few_rows.h with row-major activations up to sixteen rows, the batched core above.
inline RowsRoute rows_route(const RowsCall &c, bool all_few, int cus) {
    if (all_few) return kOnFew;
    if (rows_gemm_serves(c, cus)) return kOnTiles;
    return c.rows <= kFewRows ? kOnFew : kOnCore;
}

// Attention of a block of new positions (two or more per sequence): attn_rows.h, small workgroups that each serve 16 / G positions
// of a KV head over all their tokens, or the kernels that split a context over workgroups.  matrix_cores: the splits are long enough
// for the matrix cores there.  Shorter ones stay with the vector attention, whose query and probabilities are 32-bit (here as there they
// are pairs of bf16) and which a value that is not finite at a later position does not reach.
//
// The host knows the capacity, not the contexts, so the rule has to hold where one sequence fills its cache and the others are short: the
// chain of that one's rounds of 128 tokens then decides, as it does where there are few groups (sequence, KV head, 16 / G positions).
// sized: the splits are sized by the lengths found on the device (few groups), which shortens just that.  Splits / attn_rows.h, whole
// calls of heads 512 wide, least and mean of a set of 1863 (all contexts at the capacity; one of them, the others at 60):
//   5 and 9 rounds                               1.04, 1.12;  1.04, 1.13
//   sized:      17, 25, 33, 65 rounds            1.02, 1.11;  0.97, 1.06     0.99, 1.08;  0.93, 1.01     0.95, 1.04;  0.88, 0.95     0.82, 0.94;  0.75, 0.81
//   not sized:  25, 33, 49, 129 rounds           1.02, 1.07;  1.00, 1.10     1.11, 1.18;  1.07, 1.18     1.02, 1.14;  0.93, 1.08     0.88, 1.17;  0.67, 0.87
//               (fewer than 64 groups: 25, 33    0.98, 1.00;  0.98, 1.00     0.92;  0.93)
//   one sequence, more than 16 rounds: two groups per round or more 1.03, 1.25; fewer 0.43, 0.87
// (Those with workgroups of four waves had four sums of a column's tokens then.  With eight, 264 blocks of 5 to 40 rounds that are served:
// mean 1.18; least 0.975 with all contexts at the capacity, 17 rounds, 289 us / 296, and 0.988 with one, 40 rounds, 114 / 116.)
inline bool attn_rows_serves(int positions, bool matrix_cores, int sequences, long long groups, bool sized, int capacity) {
    const int rounds = (capacity + 127) / 128;
    if (positions < 2 || !matrix_cores) return false;
    return rounds <= 16 || (!sized && groups >= 64 && rounds <= 40) || (sequences == 1 && 2ll * rounds <= groups);
}

// waves of its workgroups: eight where there are no more groups than compute units
inline int attn_rows_waves(long long groups, int cus) { return groups <= cus ? 8 : 4; }

// One sequence of a head with a reduction below 512: the single launch on a quarter of the compute units (flow.h), or one launch
// per phase on all of them.  step_bytes: weights of a step, kv_bytes: keys and values up to the capacity (the lengths are on the
// device).  What a launch per phase loses to its gaps a quarter of the units loses to reading more.  Three steps, us, single launch
// / launch per phase: 256 wide, 3.6 MiB of weights 122 / 151, 4.6 131 / 158, 5.6 140 / 160, 7.1 155 / 169, 8.6 169 / 173, 9.6 178 / 177
// (wider ones meet later: 480 wide, 9.3 132 / 162, 18.7 185 / 185); with 4.5 MiB of weights, 16 query heads and 8 MiB of keys and values
// 149 / 180, 16 MiB 168 / 177 (6.5 MiB of weights: 185 / 183), 32 MiB 303 / 193.  Of 317 heads within the lines none is below 1.04
// times as fast so.
constexpr size_t kFlowNarrowBytes = 8 << 20, kFlowNarrowKvBytes = 16 << 20;
inline bool flow_narrow_serves(size_t step_bytes, size_t kv_bytes) {
    return step_bytes <= kFlowNarrowBytes && kv_bytes <= kFlowNarrowKvBytes;
}

} // namespace mtp
