// Prints the rotary factors of csrc/rope.h: reads lines "pos inv_freq" from standard input, writes "cos sin cos sin" for each
// (the launch-per-phase kernels' function, then the single-launch kernel's).
#include <cmath>
#include <cstdio>

#define __device__
#define __forceinline__ inline
using std::floor;
using std::fma;
using std::rint;
#include "../../paper_2509_18362_amd/csrc/rope.h"

int main() {
    int pos;
    double inv;
    while (std::scanf("%d %lf", &pos, &inv) == 2) {
        float c, s, cl, sl;
        mtp::rope_cos_sin(pos, inv, c, s);
        mtp::rope_cos_sin_lib(pos, inv, cl, sl);
        std::printf("%.13g %.13g %.13g %.13g\n", c, s, cl, sl);
    }
    return 0;
}
