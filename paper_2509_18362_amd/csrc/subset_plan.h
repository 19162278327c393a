// Rules of the list builder (subset_build.hip): how wide the counting kernel's fields are, in how many chunks and slices it
// counts, and over which bits of the counts the selection goes.  Host code without HIP: the rules can be compiled and
// checked on their own.
#pragma once
#include <algorithm>
#include <cstddef>
#include <cstdint>

namespace mtp {
namespace subset {

constexpr int kLdsWords = 160 * 1024 / 4; // of a CU, all of them the counting workgroup's
constexpr int kSpareWords = 64;

// entries of the table of wraps: ids that occur more often in a slice than a field can hold (256 times in 2^18 tokens is
// one in 1024: a few hundred ids of a long tail)
constexpr int table_bits(int bits) { return bits == 8 ? 10 : 8; }
constexpr int table_entries(int bits) { return 1 << table_bits(bits); }
// words of the bins of `ids` ids, whole 16-byte pieces
constexpr int bin_words(int ids, int bits) { return ((ids + 32 / bits - 1) / (32 / bits) + 3) / 4 * 4; }
// ids that fit a workgroup's LDS
constexpr int chunk_capacity(int bits) { return (kLdsWords - 2 * table_entries(bits) - kSpareWords) / 4 * 4 * (32 / bits); }
constexpr size_t hist_lds_bytes(int ids, int bits) {
    return ((size_t)bin_words(ids, bits) + 2 * table_entries(bits) + kSpareWords) * 4;
}
static_assert(chunk_capacity(16) == 80768 && chunk_capacity(8) == 155392, "said elsewhere");

struct CountPlan {
    int bits, chunks, chunk_ids, slices; // width of a field, passes over the stream, ids of each, workgroups of each
};

// The wider fields unless the narrower ones read the stream fewer times (wide fields wrap less often, narrow ones hold more
// ids).  256 workgroups in all, one per CU of the device this is written for, a multiple of eight per chunk: the chunks' workgroups of
// a slice then share a compute die.  (Fields of 6 bits would hold 201 920 ids in one chunk, but leave no room for the wraps of a stream of
// a few hundred ids: 2^26 tokens of 200 001 ids, 600 of which occur, side by side / a long tail: 418 / 103 us, in two chunks of
// 8 bits 135 / 113, in three of 16 bits 151 / 165.)
inline CountPlan count_plan(int V) {
    CountPlan p{};
    for (int bits : {16, 8}) {
        const int chunks = (V - 1) / chunk_capacity(bits) + 1;
        if (p.bits && chunks >= p.chunks) continue;
        p.bits = bits;
        p.chunks = chunks;
    }
    const int per_word = 32 / p.bits, piece = 4 * per_word; // chunks begin at whole 16-byte pieces of words
    p.chunk_ids = ((V - 1) / p.chunks / piece + 1) * piece;
    p.chunks = (V - 1) / p.chunk_ids + 1; // (rounding up may have emptied the last of very many)
    const int s = 256 / p.chunks;
    p.slices = s >= 8 ? s / 8 * 8 : std::max(1, s);
    return p;
}
inline size_t partial_words(const CountPlan &p) { return (size_t)p.slices * p.chunks * bin_words(p.chunk_ids, p.bits); }
// Slices of a stream of n_tokens: a workgroup clears and stores its bins however few tokens it counts, and the kernel after
// it reads them all (151 680 ids, 2^22 tokens: 50 us in 256 slices, 41 in 128; 2^18: 52 and 30 in 8).
// Without the copies of the bins (stored: false) only ids that occur cost anything afterwards: an add of every slice that has one,
// and those of one id go one by one.  Half as many slices are ahead until the reading counts for more (151 680 ids, 256 slices
// / 128: 2^23 tokens of a long tail 108 us / 93, of 2500 ids 70 / 55).
constexpr int kSliceTokens = 32768, kSliceTokensAdded = 4096, kSliceTokensAll = 65536;
inline int stream_slices(const CountPlan &p, int64_t n_tokens, bool stored) {
    const int per = stored ? kSliceTokens : kSliceTokensAdded;
    const int most = stored || n_tokens >= (int64_t)kSliceTokensAll * p.slices ? p.slices : (p.slices + 1) / 2;
    const int64_t want = (n_tokens + per - 1) / per;
    return (int)std::min<int64_t>(most, std::max<int64_t>(8, (want + 7) / 8 * 8));
}

// The selection's digits, most significant first.  The n-th largest count T is at most n_tokens / n, so the keys are the
// counts cut off at that + 1: order and ties up to T stay as they are.
constexpr int kSelPasses = 3, kSelBuckets = 4096;
struct SelPlan {
    unsigned cap; // keys: min(count, cap)
    int passes, bits[kSelPasses], shift[kSelPasses];
};
constexpr unsigned sel_key(const SelPlan &p, unsigned count) { return count < p.cap ? count : p.cap; }
constexpr int sel_buckets(const SelPlan &p, int pass) { // (the top digit of no key is larger than the cap's)
    return pass == 0 ? (int)(p.cap >> p.shift[0]) + 1 : 1 << p.bits[pass];
}
inline SelPlan sel_plan(int64_t n_tokens, int n) {
    SelPlan p{};
    if (n < 1) return p; // nothing to select
    p.cap = (unsigned)(n_tokens / n) + 1u; // (n_tokens < 2^31)
    int left = 32 - __builtin_clz(p.cap);
    p.passes = (left + 11) / 12;
    for (int i = 0; i < p.passes; ++i) {
        p.bits[i] = (left + p.passes - i - 1) / (p.passes - i);
        p.shift[i] = left -= p.bits[i];
    }
    return p;
}

} // namespace subset
} // namespace mtp
