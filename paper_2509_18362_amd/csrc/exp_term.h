// Terms of a softmax.  No HIP in here but the hardware's exp2 and __device__: a CPU test compiles it with both defined away.
#pragma once

namespace mtp {

// A term of a sum of very many (a vocabulary's): exp(t), t <= 0, as a product with log2(e) and the hardware's exp2.  The product is
// rounded once, with the constant in two parts: what a term is off by that way, 2^-24 of its exponent, is at random over the terms and
// next to nothing of it is left in their sum (with the constant in one part all terms are off the same way: 6e-8 of the sum at a
// spread of the logits of 1 to 3).
__device__ __forceinline__ float exp_term(float t) { return __builtin_amdgcn_exp2f(fmaf(t, 1.44269502f, t * 1.92596303e-8f)); }

// The weight of a token, or of one of the few partial results that a merge puts together: one or two may carry the sum, so each has
// to be right to an ulp whatever its exponent (exp_term is off by up to 2^-24 |t|; with it three steps took 107.5 us instead of 109.5 at
// d = 256, 837 instead of 842 at 8 Ki of context, d = 4096).
__device__ __forceinline__ float exp_weight(float t) { return expf(t); }

} // namespace mtp
