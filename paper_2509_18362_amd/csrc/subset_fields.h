// The list builder's counting fields (subset_build.hip): several to a word, so narrow that they wrap.  No HIP in here but
// __host__ __device__: a CPU test compiles it with both defined away.
#pragma once

namespace mtp {
namespace subset {

template <int BITS>
struct Fields {
    static constexpr int kPerWord = 32 / BITS;
    static constexpr unsigned kFull = (1u << BITS) - 1u; // a field that the next add wraps
    // place of an id's field in its word (the hardware takes the low five bits of a shift)
    static __host__ __device__ unsigned shift_of(unsigned rel) { return 32 % BITS == 0 ? rel * BITS & 31u : rel % kPerWord * BITS; }
    static __host__ __device__ unsigned field(unsigned word, unsigned rel) { return word >> shift_of(rel) & kFull; }

    // Counts N tokens of one thread.  Local ids begin at c0, nb of them are counted; add(rel, inside, increment) adds to the id's
    // word - or, where the token is not one of them (inside false: rel may be any number), to a word that nobody reads - and returns
    // it as it was.  All adds first, then (rare) wrapped(id) for every field that they wrap: the added one, if it was full, and those
    // above it in the word as far as they were full too.  An add to the word that nobody reads wraps nothing: rel is then no id, and
    // what follows it in the word may seem to be one (-1 before c0 = 0 is 0xffffffff, and the number after that is 0).
    template <int N, class Add, class Wrapped>
    static __host__ __device__ void count(const int *t, int c0, unsigned nb, const Add &add, const Wrapped &wrapped) {
        unsigned rel[N], old[N], most = 0u, full = 0u;
#pragma unroll
        for (int i = 0; i < N; ++i) {
            rel[i] = (unsigned)t[i] - (unsigned)c0;
            old[i] = add(rel[i], rel[i] < nb, 1u << shift_of(rel[i]));
        }
#pragma unroll
        for (int i = 0; i < N; ++i) {
            const unsigned f = field(old[i], rel[i]);
            most = most > f ? most : f;
        }
        if (most != kFull) return;
#pragma unroll
        for (int i = 0; i < N; ++i) full |= rel[i] < nb && field(old[i], rel[i]) == kFull ? 1u << i : 0u;
        while (full) {
            unsigned id = rel[0], word = old[0], last = 1u;
#pragma unroll
            for (int i = 1; i < N; ++i)
                if (full & 1u << i) {
                    id = rel[i];
                    word = old[i];
                    last = 1u << i;
                }
            full &= ~last;
            word >>= shift_of(id);
            int f = (int)(id % kPerWord);
            do {
                if (id < nb) wrapped((int)id); // (carried into a field of the last word that has no id: nothing)
                ++id;
                ++f;
                word >>= BITS;
            } while (f < kPerWord && (word & kFull) == kFull);
        }
    }
};

} // namespace subset
} // namespace mtp
