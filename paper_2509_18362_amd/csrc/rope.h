// Rotary factors (Sec. 2.1: the head is an ordinary decoder layer).  No HIP in here: the functions can be compiled and checked
// on their own, with __device__ and __forceinline__ defined away.
#pragma once

namespace mtp {

// Cosine and sine of pos * inv_freq, for the kernels that run once per phase.  The angle is brought into [-pi/4, pi/4] around a
// multiple n of pi/2 in double precision (two-part constant); sine and cosine of the rest are their Taylor polynomials there
// (remainders below 1e-11), also in double, and rounded once: half a unit in the last place, and 1e-11, of the exact factors
// of the rounded angle.  cosf and sinf took 2-3 us of every attention launch: two functions with argument reductions of their
// own, code that is fetched from memory in every launch (matrix-core attention of 5 sequences, with the query split once per
// workgroup instead of by every wave: 19.3 -> 15.7 us).
__device__ __forceinline__ void rope_cos_sin(int pos, double inv_freq, float &cs, float &sn) {
    const double half_pi_hi = 1.5707963267948966, half_pi_lo = 6.123233995736766e-17, two_over_pi = 0.6366197723675814;
    const double ang = (double)pos * inv_freq, n = rint(ang * two_over_pi);
    const double r = fma(-n, half_pi_lo, fma(-n, half_pi_hi, ang)), r2 = r * r;
    double s = fma(r2, -1.0 / 39916800, 1.0 / 362880), c = fma(r2, 1.0 / 479001600, -1.0 / 3628800);
    s = fma(r2, s, -1.0 / 5040);
    c = fma(r2, c, 1.0 / 40320);
    s = fma(r2, s, 1.0 / 120);
    c = fma(r2, c, -1.0 / 720);
    s = fma(r2, s, -1.0 / 6);
    c = fma(r2, c, 1.0 / 24);
    s = fma(r * r2, s, r);
    c = fma(r2, fma(r2, c, -0.5), 1.0);
    const int q = (int)fma(-4.0, floor(n * 0.25), n); // quadrant (a theta below one gives more quarter turns than an int holds)
    const float fs = (float)s, fc = (float)c, a = (q & 1) ? fs : fc, b = (q & 1) ? fc : fs;
    cs = (q == 1 || q == 2) ? -a : a;
    sn = q >= 2 ? -b : b;
}

// The same with the library's functions, for the single-launch kernel: there the factors are formed while q/k/v travel, its code
// stays in the instruction cache over the steps, and the chain above, in its place, took 4 us more per three steps (420.7
// against 416.4).
__device__ __forceinline__ void rope_cos_sin_lib(int pos, double inv_freq, float &cs, float &sn) {
    const double two_pi_hi = 6.283185307179586232, two_pi_lo = 2.4492935982947064e-16, inv_two_pi = 0.15915494309189535;
    const double ang = (double)pos * inv_freq;
    const double n = rint(ang * inv_two_pi);
    const float r = (float)fma(-n, two_pi_lo, fma(-n, two_pi_hi, ang));
    cs = cosf(r);
    sn = sinf(r);
}

} // namespace mtp
