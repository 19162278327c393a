// Prints what the rules of csrc/rows_plan.h say.  Without an argument: reads lines "K n rows head pairs cus part_floats call_rows d"
// (a matrix phase over `rows` of the call's rows), writes "route tile_rows tile_weight_rows parts microseconds" for each, route 0
// few_rows.h, 1 the tiles, 2 the batched core; -1 where the whole call takes few_rows.h.  With "narrow": reads "step_bytes
// kv_bytes", writes 1 where one sequence of a narrow head takes the single launch.  With "block": reads "positions matrix_cores
// sequences groups sized capacity", writes 1 where a block's attention takes attn_rows.h.
#include <cstdio>
#include <cstring>

#include "../../paper_2509_18362_amd/csrc/rows_plan.h"

int main(int argc, char **argv) {
    if (argc > 1 && !std::strcmp(argv[1], "narrow")) {
        unsigned long long step, kv;
        while (std::scanf("%llu %llu", &step, &kv) == 2) std::printf("%d\n", mtp::flow_narrow_serves(step, kv) ? 1 : 0);
        return 0;
    }
    if (argc > 1 && !std::strcmp(argv[1], "block")) {
        int positions, matrix_cores, sequences, sized, capacity;
        long long groups;
        while (std::scanf("%d %d %d %lld %d %d", &positions, &matrix_cores, &sequences, &groups, &sized, &capacity) == 6)
            std::printf("%d\n", mtp::attn_rows_serves(positions, matrix_cores != 0, sequences, groups, sized != 0, capacity) ? 1 : 0);
        return 0;
    }
    int K, n, rows, head, pairs, cus, call_rows, d;
    unsigned long long part_floats;
    while (std::scanf("%d %d %d %d %d %d %llu %d %d", &K, &n, &rows, &head, &pairs, &cus, &part_floats, &call_rows, &d) == 9) {
        const mtp::RowsCall c{K, n, rows, head != 0, pairs != 0};
        const mtp::RowsPlan p = mtp::rows_plan(c, cus, (size_t)part_floats);
        const mtp::RowsTileInfo &t = mtp::kRowsTile[p.tile];
        const bool all_few = mtp::rows_all_few(call_rows, d);
        std::printf("%d %d %d %d %.3f\n", all_few ? -1 : (int)mtp::rows_route(c, all_few, cus), t.bm, t.bn, p.kp, p.us);
    }
    return 0;
}
