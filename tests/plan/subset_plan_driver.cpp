// Prints what the rules of csrc/subset_plan.h say.  Reads lines "vocab tokens n", writes "bits chunks chunk_ids slices lds_bytes
// stream_slices cap passes bits0 shift0 bits1 shift1 bits2 shift2 stream_slices_without_workspace".
#include <cstdio>

#include "../../paper_2509_18362_amd/csrc/subset_plan.h"

int main() {
    using namespace mtp::subset;
    int V, n;
    long long tokens;
    while (std::scanf("%d %lld %d", &V, &tokens, &n) == 3) {
        const CountPlan c = count_plan(V);
        const SelPlan s = sel_plan(tokens, n);
        std::printf("%d %d %d %d %zu %d %u %d", c.bits, c.chunks, c.chunk_ids, c.slices, hist_lds_bytes(c.chunk_ids, c.bits),
                    stream_slices(c, tokens, true), s.cap, s.passes);
        for (int p = 0; p < kSelPasses; ++p) std::printf(" %d %d", s.bits[p], s.shift[p]);
        std::printf(" %d\n", stream_slices(c, tokens, false));
    }
    return 0;
}
