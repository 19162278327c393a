// Sums of csrc/exp_term.h over a vocabulary: reads lines "seed spread", writes the sum's relative error (terms as the kernel forms
// them, added up in double) for normally distributed logits.  With "weight": writes the largest relative error of a single weight
// with an exponent of -80 to 0, and what it makes of 0 and -inf.
#include <algorithm>
#include <cmath>
#include <cstdio>
#include <random>
#include <vector>

#define __device__
#define __forceinline__ inline
#define __builtin_amdgcn_exp2f std::exp2
using std::fmaf;
#include "../../paper_2509_18362_amd/csrc/exp_term.h"

int main(int argc, char **) {
    if (argc > 1) {
        double worst = 0;
        for (int i = 0; i <= 800000; ++i) {
            const float t = -1e-4f * i;
            worst = std::max(worst, std::fabs(mtp::exp_weight(t) / std::exp((double)t) - 1));
        }
        std::printf("%.6g %g %g\n", worst, mtp::exp_weight(0.f), mtp::exp_weight(-INFINITY));
        return 0;
    }
    unsigned seed;
    double spread;
    while (std::scanf("%u %lf", &seed, &spread) == 2) {
        std::mt19937 gen(seed);
        std::normal_distribution<float> normal(0.f, (float)spread);
        std::vector<float> z(151680);
        for (float &v : z) v = normal(gen);
        const float m = *std::max_element(z.begin(), z.end());
        double got = 0, want = 0;
        for (float v : z) {
            got += mtp::exp_term(v - m);
            want += std::exp((double)v - m);
        }
        std::printf("%.6g\n", got / want - 1);
    }
    std::printf("%g %g\n", mtp::exp_term(0.f), mtp::exp_term(-INFINITY));
    return 0;
}
