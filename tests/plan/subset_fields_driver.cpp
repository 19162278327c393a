// Counts a token stream by csrc/subset_fields.h, one add after the other: "bits vocab chunk_ids" on the command line, int32 tokens
// on standard input; writes "id counted occurs" for every id that is counted wrongly.
#include <cstdio>
#include <cstdlib>
#include <vector>

#define __host__
#define __device__
#include "../../paper_2509_18362_amd/csrc/subset_fields.h"

template <int BITS>
void run(const std::vector<int> &tokens, int V, int chunk_ids) {
    using F = mtp::subset::Fields<BITS>;
    std::vector<long long> occurs(V);
    for (int t : tokens)
        if (t >= 0 && t < V) ++occurs[t];
    for (int c0 = 0; c0 < V; c0 += chunk_ids) {
        const int nb = V - c0 < chunk_ids ? V - c0 : chunk_ids;
        std::vector<unsigned> bins(nb / F::kPerWord + 1), spare(64);
        std::vector<long long> wraps(nb + F::kPerWord);
        constexpr int N = 16;
        for (size_t i = 0; i < tokens.size(); i += N) {
            int t[N];
            for (int k = 0; k < N; ++k) t[k] = i + k < tokens.size() ? tokens[i + k] : -1;
            unsigned &mine = spare[i / N % 64]; // (a lane's)
            F::template count<N>(
                t, c0, (unsigned)nb,
                [&](unsigned rel, bool inside, unsigned by) {
                    unsigned &w = inside ? bins[rel / F::kPerWord] : mine;
                    const unsigned was = w;
                    w += by;
                    return was;
                },
                [&](int id) { ++wraps[id]; });
        }
        for (int j = 0; j < nb; ++j) {
            const long long below = j % F::kPerWord ? wraps[j - 1] : 0;
            const long long got = F::field(bins[j / F::kPerWord], (unsigned)j) + (wraps[j] << BITS) - below;
            if (got != occurs[c0 + j]) std::printf("%d %lld %lld\n", c0 + j, got, occurs[c0 + j]);
        }
    }
}

int main(int, char **argv) {
    const int bits = std::atoi(argv[1]), V = std::atoi(argv[2]), chunk_ids = std::atoi(argv[3]);
    std::vector<int> tokens;
    int buffer[4096];
    for (size_t n; (n = std::fread(buffer, 4, 4096, stdin)) > 0;) tokens.insert(tokens.end(), buffer, buffer + n);
    if (bits == 16) run<16>(tokens, V, chunk_ids);
    if (bits == 8) run<8>(tokens, V, chunk_ids);
    if (bits == 6) run<6>(tokens, V, chunk_ids);
    return 0;
}
