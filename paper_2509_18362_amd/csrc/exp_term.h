// A term of a softmax's sum.  No HIP in here but the hardware's exp2 and __device__: a CPU test compiles it with both defined away.
#pragma once

namespace mtp {

// exp(t), t <= 0: a product with log2(e) and the hardware's exp2.  The product is rounded once, with the constant in two parts: what
// a term is off by that way, 2^-24 of its exponent, is at random over the terms and next to nothing of it is left in their sum (with
// the constant in one part all terms are off the same way: 6e-8 of the sum at a spread of the logits of 1 to 3).
__device__ __forceinline__ float exp_term(float t) { return __builtin_amdgcn_exp2f(fmaf(t, 1.44269502f, t * 1.92596303e-8f)); }

} // namespace mtp
