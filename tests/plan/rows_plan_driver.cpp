// Prints what the tiled matrix products would do with a phase: reads lines "K n rows head pairs cus part_floats" from
// standard input, writes "serves tile_rows tile_weight_rows parts microseconds" for each.  With the argument "narrow": reads
// "step_bytes kv_bytes", writes 1 where one sequence of a narrow head takes the single launch.
#include <cstdio>
#include <cstring>

#include "../../paper_2509_18362_amd/csrc/rows_plan.h"

int main(int argc, char **argv) {
    if (argc > 1 && !std::strcmp(argv[1], "narrow")) {
        unsigned long long step, kv;
        while (std::scanf("%llu %llu", &step, &kv) == 2) std::printf("%d\n", mtp::flow_narrow_serves(step, kv) ? 1 : 0);
        return 0;
    }
    int K, n, rows, head, pairs, cus;
    unsigned long long part_floats;
    while (std::scanf("%d %d %d %d %d %d %llu", &K, &n, &rows, &head, &pairs, &cus, &part_floats) == 7) {
        const mtp::RowsCall c{K, n, rows, head != 0, pairs != 0};
        const mtp::RowsPlan p = mtp::rows_plan(c, cus, (size_t)part_floats);
        const mtp::RowsTileInfo &t = mtp::kRowsTile[p.tile];
        std::printf("%d %d %d %d %.3f\n", mtp::rows_gemm_serves(c, cus) ? 1 : 0, t.bm, t.bn, p.kp, p.us);
    }
    return 0;
}
