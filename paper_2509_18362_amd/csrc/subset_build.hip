// High-frequency vocabulary list from a token stream (gfx950): occurrence counts per id, the n most frequent ids
// (equal counts: lower id first), written in ascending id order - the list the compressed output head is gathered
// with (Sec. 2.2, which takes the frequent tokens of a language from statistics over a corpus; Eq. (3)).
//
// Counting is the only part that touches much memory.  Global atomics on a long-tailed stream would pile up on the
// few hottest ids (same-address device atomics serialize at ~40 ns each), so every workgroup counts in LDS, in fields so
// narrow that the 160 KB of a CU hold the whole vocabulary and the stream is read once: 16 bits up to 80 768 ids, 8 up to
// 155 392; beyond that the vocabulary is counted in chunks.  Narrow fields wrap, and a
// wrap carries into the next field of its word.  Both are accounted for exactly: the atomic that adds returns the word as it
// was, which tells which fields this add wraps, and the number W[j] of wraps of field j is kept in a small table in LDS
// (hashed by id: only ids that occur more often than a field can hold get there).  A field has had as many increments as it
// holds plus 2^bits W[j], and W[j-1] of them were carries of the field below, so count[j] = field[j] + 2^bits W[j] - W[j-1],
// whatever the order of the adds.  (Fields of 16 bits, two passes over the stream and sweeps that moved full fields away in
// time: 99 us for 2^26 tokens of 151 680 ids; this: 58.)
// At the end a workgroup stores its bins as they are and a second kernel adds the workgroups' copies up (every workgroup
// adding its non-zero fields to the global counts with atomics took longer than the counting; the entry point without a
// workspace still does that).  Every thread keeps the four 16-byte loads of the next round in flight while it counts.
// Selection: the n-th largest of the counts is at most n_tokens / n, so larger ones are as good as that + 1, and a radix
// select over the few bits that leaves (digits of up to 12 bits: 2^26 tokens and n = 32 768 take one pass) finds the count T
// of the n-th most frequent id and how many ids with exactly that count belong to the list; the compaction then walks the
// ids in ascending order and keeps those with count > T plus the first ties, placing them by prefix sums - the output is
// born sorted, nothing is sorted.  Both are spread over many workgroups (a single compute unit reads memory at
// ~20 GB/s: as one workgroup these steps took 0.5 ms, more than the counting); the walk over a pass's buckets is done by
// every workgroup of the kernel that follows, as a scan (as a kernel of its own with a serial loop it took 13 us a pass).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>
#include <cstdio>
#include <mutex>
#include <type_traits>

#include "../../include/mtp_draft.h"
#include "subset_fields.h"
#include "subset_plan.h"

namespace {

using namespace mtp::subset;

constexpr int kHistBlock = 1024;
// Copies of the global counts that the counting kernel's workgroups give the wraps to (where the copies of the bins are there
// too): in streams of a few hundred ids every workgroup has all of them, and atomics to one cache line go one by one (600
// scattered ids of 151 680, 2^26 tokens: 93 us with one copy, 86 with four; a long-tailed stream 86 and 85).
constexpr int kCountCopies = 4;
__host__ __device__ constexpr size_t round4(size_t words) { return (words + 3) / 4 * 4; }
constexpr int kSelBlock = 1024;

// clears `words` words (whole 16-byte pieces), the state among them, and leaves n in the state
__global__ void k_subset_clear(unsigned *work, size_t words, unsigned *state, int n) {
    const size_t i = ((size_t)blockIdx.x * blockDim.x + threadIdx.x) * 4;
    if (i >= words) return;
    uint4 zero{0u, 0u, 0u, 0u};
    if (work + i == state) zero.z = (unsigned)n; // [2]: ids still to be found by the selection
    *reinterpret_cast<uint4 *>(work + i) = zero;
}

// The table of wraps: keys (local id, or kNoKey), then as many counts.  Ids that differ in their last four bits only are neighbours in
// it, so that the wave that hands them to the global counts has few cache lines to go to, each once (an atomic per id, what the
// field below carried in taken off: 600 ids side by side of 151 680, 2^26 tokens: places scattered by id and two atomics per id 128 us,
// without a workspace 190; so 80 and 78).
constexpr unsigned kNoKey = 0xffffffffu;

// grid (slices, chunks): workgroup (s, c) counts the ids of chunk c in every (slices)-th piece of the stream, from the s-th on.
// What bounds it: reading the stream and writing the bins (268 + 39 MB at 2^26 tokens and 151 680 ids: 58 us, 52 with the adds
// taken out; a stream read twice took 99).
// The loop over whole rounds has no check for the slice's end, no count of ids outside the vocabulary (that is what is
// missing from the sum of all counts) and no branch around a load or an add: an id that is not of this chunk adds to a
// word that its lane alone uses.
template <int BITS>
__global__ __launch_bounds__(kHistBlock) void k_subset_hist(const int *__restrict__ tokens, long long n_tokens, int V,
                                                            int chunk_ids, unsigned *counts, int copies, unsigned *partials) {
    constexpr int FPW = Fields<BITS>::kPerWord;
    constexpr unsigned kFull = Fields<BITS>::kFull;
    constexpr int kTable = table_entries(BITS);
    extern __shared__ unsigned bins[]; // word w: local ids FPW w (lowest bits) .. FPW w + FPW - 1
    const int c0 = blockIdx.y * chunk_ids;
    const int nb = min(chunk_ids, V - c0), nw4 = bin_words(chunk_ids, BITS);
    unsigned *keys = bins + nw4, *wraps = keys + kTable, *spare = wraps + kTable; // spare: 64 words, one per lane
    for (int i4 = threadIdx.x * 4; i4 < nw4; i4 += kHistBlock * 4)
        *reinterpret_cast<uint4 *>(bins + i4) = uint4{0u, 0u, 0u, 0u};
    for (int i = threadIdx.x; i < kTable; i += kHistBlock) {
        keys[i] = kNoKey;
        wraps[i] = 0u;
    }
    if (threadIdx.x < 64) spare[threadIdx.x] = 0u;
    __syncthreads();
    counts += (size_t)(blockIdx.x % copies) * round4(V);
    // `by` wraps of the field of local id `id`: that many carries went into the next field of the word, if there is one
    auto give = [&](int id, unsigned by) {
        atomicAdd(&counts[c0 + id], by << BITS);
        if (id % FPW + 1 < FPW && id + 1 < nb) atomicAdd(&counts[c0 + id + 1], 0u - by);
    };
    // the first place of an id; the others it can have are sixteen apart
    auto slot_of = [](int id) {
        return ((unsigned)(id >> 4) * 2654435761u >> (36 - table_bits(BITS))) * 16 + (unsigned)(id & 15);
    };
    auto wrapped = [&](int id) {
        unsigned slot = slot_of(id);
        for (int tries = 0; tries < 4; ++tries) {
            const unsigned key = atomicCAS(&keys[slot], kNoKey, (unsigned)id);
            if (key == kNoKey || key == (unsigned)id) {
                atomicAdd(&wraps[slot], 1u);
                return;
            }
            slot = (slot + 16) % kTable;
        }
        give(id, 1u); // no room: straight to the global counts
    };
    // an id's wraps in the table (an id in it always has some), once no more are added
    auto booked = [&](int id) {
        unsigned slot = slot_of(id);
        for (int tries = 0; tries < 4; ++tries) {
            if (keys[slot] == (unsigned)id) return wraps[slot];
            slot = (slot + 16) % kTable;
        }
        return 0u;
    };
    // (an id that is not of this chunk adds to a word that its lane alone uses)
    auto count = [&](auto n, const int *t) {
        Fields<BITS>::template count<decltype(n)::value>(
            t, c0, (unsigned)nb,
            [&](unsigned rel, bool inside, unsigned by) { return atomicAdd(inside ? bins + rel / FPW : spare + (threadIdx.x & 63), by); },
            wrapped);
    };
    typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
    typedef int i32x4 __attribute__((ext_vector_type(4)));
    const i32x4 *t4 = reinterpret_cast<const i32x4 *>(tokens);
    constexpr int kUnroll = 4; // 16-byte loads per thread and round
    // Pieces of 16 KB go round the workgroups, so that together they sweep the stream (contiguous slices lie a power of two
    // apart for such streams, and their reads meet in the same memory channels).
    const long long groups = n_tokens / 4, stride = (long long)gridDim.x * kHistBlock;
    const long long first = (long long)blockIdx.x * kHistBlock + threadIdx.x;
    if (blockIdx.x == gridDim.x - 1) { // the stream's last one to three tokens
        const long long i = groups * 4 + threadIdx.x;
        if (i < n_tokens) count(std::integral_constant<int, 1>(), tokens + i);
    }
    if (groups > 0) {
        // the loads of round i + 1 are requested before round i is counted; past the end the last group is read again
        auto fetch = [&](long long r, i32x4(&v)[kUnroll]) {
#pragma unroll
            for (int u = 0; u < kUnroll; ++u) v[u] = t4[min(first + (r * kUnroll + u) * stride, groups - 1)];
        };
        auto count_all = [&](const i32x4(&v)[kUnroll]) {
            int t[4 * kUnroll];
#pragma unroll
            for (int i = 0; i < 4 * kUnroll; ++i) t[i] = v[i / 4][i % 4];
            count(std::integral_constant<int, 4 * kUnroll>(), t);
        };
        const long long rounds = groups / (kUnroll * stride); // whole ones, of all workgroups alike
        i32x4 va[kUnroll], vb[kUnroll];
        fetch(0, va);
        long long r = 0;
        for (; r + 1 < rounds; r += 2) {
            fetch(r + 1, vb);
            count_all(va);
            fetch(r + 2, va);
            count_all(vb);
        }
        if (r < rounds) {
            fetch(r + 1, vb);
            count_all(va);
#pragma unroll
            for (int u = 0; u < kUnroll; ++u) va[u] = vb[u];
        }
        // what is left: less than a round
#pragma unroll
        for (int u = 0; u < kUnroll; ++u)
            if (first + (rounds * kUnroll + u) * stride >= groups) va[u] = i32x4{-1, -1, -1, -1};
        count_all(va);
    }
    __syncthreads();
    for (int i = threadIdx.x; i < kTable; i += kHistBlock) {
        if (keys[i] == kNoKey) continue;
        const int id = (int)keys[i];
        const unsigned w = wraps[i], below = id % FPW ? booked(id - 1) : 0u;
        atomicAdd(&counts[c0 + id], (w << BITS) - below);
        if (id % FPW + 1 < FPW && id + 1 < nb && booked(id + 1) == 0u) atomicAdd(&counts[c0 + id + 1], 0u - w);
    }
    // What is in the bins: with room for it, the workgroup's bins go to memory as they are (k_subset_reduce adds
    // the workgroups' copies up); without, every non-zero field is added to the global counts (up to a vocabulary of
    // atomics per workgroup, 39 M over the grid when every id occurs: slower than the counting itself).
    if (partials) {
        unsigned *dst = partials + ((size_t)blockIdx.y * gridDim.x + blockIdx.x) * nw4;
        for (int i4 = threadIdx.x * 4; i4 < nw4; i4 += kHistBlock * 4)
            *reinterpret_cast<u32x4 *>(dst + i4) = *reinterpret_cast<const u32x4 *>(bins + i4);
    } else {
        for (int i = threadIdx.x; i < nb; i += kHistBlock) { // (consecutive lanes, consecutive ids: few cache lines)
            const unsigned x = bins[i / FPW] >> (i % FPW * BITS) & kFull;
            if (x) atomicAdd(&counts[c0 + i], x);
        }
    }
}

// state: [0] unused, [1] T, [2] n, then r at [3]; [4 + 2 p], [5 + 2 p]: prefix and ids still needed after the walk
// of pass p; then the bucket counts of the passes, then per-workgroup (above, ties) totals of the compaction, then
// the slots of the sum of all counts
constexpr int kCmpGroups = 160; // workgroups of the compaction: one round of 1024 ids each at 151 680 ids
static_assert(kCmpGroups <= kSelBlock, "a thread for each workgroup's totals");
constexpr int kSumSlots = 64;   // words the sum of all counts is spread over
constexpr int kHistCopies = 2;  // and the bucket counts of a pass: a few dozen buckets hold most ids
constexpr int kStateAfter = 4, kStateHist = 16, kStateTotals = kStateHist + kSelPasses * kSelBuckets * kHistCopies,
              kStateSums = kStateTotals + 2 * kCmpGroups, kStateWordsFull = kStateSums + kSumSlots;
static_assert(kStateAfter + 2 * kSelPasses <= kStateHist, "state layout");

// The sum over the workgroup's threads, added to one of the slots: one atomic per workgroup (same-address device atomics
// take ~40 ns each and those to one cache line little less: one per wave, 4752 of them, took 7 of 19 us).  scratch: a word
// per wave.
__device__ __forceinline__ void add_to_sum(unsigned x, unsigned *scratch, unsigned *sums) {
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) x += __shfl_xor(x, off, 64);
    if ((threadIdx.x & 63) == 0) scratch[threadIdx.x >> 6] = x;
    __syncthreads();
    if (threadIdx.x >= 64) return;
    x = threadIdx.x < blockDim.x / 64 ? scratch[threadIdx.x] : 0u;
#pragma unroll
    for (int off = 1; off < 16; off <<= 1) x += __shfl_xor(x, off, 64);
    if (threadIdx.x == 0 && x) atomicAdd(&sums[blockIdx.x % kSumSlots], x);
}

// the workgroup's bucket counts of a pass, from LDS to one of the copies in the state
__device__ __forceinline__ void put_hist(const unsigned *hist, int buckets, int pass, unsigned *state) {
    unsigned *dst = state + kStateHist + (pass * kHistCopies + (int)(blockIdx.x % kHistCopies)) * kSelBuckets;
    for (int i = threadIdx.x; i < buckets; i += blockDim.x)
        if (hist[i]) atomicAdd(&dst[i], hist[i]);
}

// counts[id] += the sum over the slices' workgroups of the id's field.  Workgroup: 128 words of one chunk, two waves for
// each eighth of the slices (all of whose loads are in flight at once: the kernel is a chain of strided reads, 12 us for 256 copies of 152 KB).  The final
// counts pass through here, so the first histogram pass of the selection, their sum and the copy for the caller are taken along.
constexpr int kReduceWords = 128;
template <int BITS>
__global__ __launch_bounds__(kSelBlock) void k_subset_reduce(const unsigned *__restrict__ partials, int slices, int V,
                                                             int chunk_ids, SelPlan plan, unsigned *counts,
                                                             unsigned *state, int *counts_out) {
    constexpr int FPW = 32 / BITS, kParts = kSelBlock / kReduceWords;
    __shared__ unsigned hist[kSelBuckets];
    __shared__ unsigned sums[kParts][kReduceWords * FPW], scratch[kSelBlock / 64];
    const int buckets = sel_buckets(plan, 0);
    for (int i = threadIdx.x; i < buckets; i += kSelBlock) hist[i] = 0u;
    const int c0 = blockIdx.y * chunk_ids, nb = min(chunk_ids, V - c0), nw = bin_words(chunk_ids, BITS);
    const int part = threadIdx.x / kReduceWords, lw = threadIdx.x % kReduceWords;
    const int w0 = blockIdx.x * kReduceWords, w = min(w0 + lw, nw - 1);
    unsigned s[FPW];
#pragma unroll
    for (int f = 0; f < FPW; ++f) s[f] = 0u;
    const unsigned *src = partials + (size_t)blockIdx.y * slices * nw + w;
    auto take = [&](unsigned x) {
#pragma unroll
        for (int f = 0; f < FPW; ++f) s[f] += x >> (f * BITS) & ((1u << BITS) - 1u);
    };
    int sl = part * slices / kParts;
    const int end = (part + 1) * slices / kParts;
    for (; sl + 32 <= end; sl += 32) {
        unsigned x[32];
#pragma unroll
        for (int u = 0; u < 32; ++u) x[u] = src[(size_t)(sl + u) * nw];
#pragma unroll
        for (int u = 0; u < 32; ++u) take(x[u]);
    }
    for (; sl + 8 <= end; sl += 8) {
        unsigned x[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) x[u] = src[(size_t)(sl + u) * nw];
#pragma unroll
        for (int u = 0; u < 8; ++u) take(x[u]);
    }
    for (; sl < end; ++sl) take(src[(size_t)sl * nw]);
#pragma unroll
    for (int f = 0; f < FPW; ++f) sums[part][lw * FPW + f] = s[f];
    __syncthreads();
    unsigned total = 0u;
    for (int base = 0; base < kReduceWords * FPW; base += kSelBlock) { // (whole waves go round together)
        const int i = base + (int)threadIdx.x, id = w0 * FPW + i;
        const bool has = i < kReduceWords * FPW && id < nb;
        unsigned c = 0u;
        if (has) {
#pragma unroll
            for (int q = 0; q < kCountCopies; ++q) c += counts[q * round4(V) + c0 + id]; // (what the counting kernel has given here)
#pragma unroll
            for (int q = 0; q < kParts; ++q) c += sums[q][i];
            counts[c0 + id] = c;
            if (counts_out) counts_out[c0 + id] = (int)c;
            total += c;
        }
        // ids that do not occur are counted per wave (one LDS atomic instead of up to 64 on the same word)
        const unsigned digit = sel_key(plan, c) >> plan.shift[0];
        const unsigned zeros = (unsigned)__popcll(__builtin_amdgcn_ballot_w64(has && digit == 0u));
        if ((threadIdx.x & 63) == 0 && zeros) atomicAdd(&hist[0], zeros);
        if (has && digit) atomicAdd(&hist[digit], 1u);
    }
    add_to_sum(total, scratch, state + kStateSums); // (a barrier: the bucket counts are complete)
    if (plan.passes) put_hist(hist, buckets, 0, state);
}

// ---- selection: T = the n-th largest count, r = how many ids with count == T belong to the n most frequent ----
// (1 <= r when n >= 1; #(count > T) = n - r).  A radix select, most significant digit first: pass p histograms digit
// p of the keys that agree with the prefix found so far (kSelGroups workgroups, each in LDS first); the kernel that
// follows walks the buckets from the top to the one that holds the n-th largest, every workgroup for itself.
constexpr int kSelGroups = 64; // workgroups of a histogram pass of the selection

// inclusive scan of one value per thread over the workgroup; scratch holds one word per wave; returns the total too
__device__ __forceinline__ unsigned block_scan(unsigned v, unsigned *scratch, unsigned &total) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const unsigned o = __shfl_up(v, off, 64);
        if (lane >= off) v += o;
    }
    __syncthreads(); // scratch of the previous scan has been read
    if (lane == 63) scratch[wave] = v;
    __syncthreads();
    unsigned base = 0u, tot = 0u;
    for (int w = 0; w < kSelBlock / 64; ++w) {
        const unsigned s = scratch[w];
        if (w < wave) base += s;
        tot += s;
    }
    total = tot;
    return v + base;
}

// The walk over the buckets of pass `pass`, by the whole workgroup: from the largest digit down to the bucket that
// holds the need-th largest of the keys that agree with the prefix.  Returns the prefix extended by that digit and
// the ids still needed from inside the bucket.  Every workgroup of a kernel computes the same values; workgroup 0
// leaves them in the state for the kernels after this one (kStateAfter).
__device__ __forceinline__ void sel_walk(unsigned *state, const SelPlan &plan, int pass, unsigned *scratch, unsigned *found,
                                         unsigned &prefix, unsigned &need) {
    const unsigned prefix_in = pass == 0 ? 0u : state[kStateAfter + 2 * (pass - 1)];
    const unsigned need_in = pass == 0 ? state[2] : state[kStateAfter + 2 * (pass - 1) + 1];
    const unsigned *hist = state + kStateHist + pass * kHistCopies * kSelBuckets;
    typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
    constexpr int kMine = kSelBuckets / kSelBlock; // buckets of a thread, the scan runs from the top
    static_assert(kMine == 4, "one 16-byte load per copy");
    const int top = (sel_buckets(plan, pass) + kMine - 1) / kMine * kMine - 1 - kMine * (int)threadIdx.x; // its highest
    unsigned a[kMine] = {0u, 0u, 0u, 0u};
    if (top >= 0) {
        u32x4 x[kHistCopies];
#pragma unroll
        for (int c = 0; c < kHistCopies; ++c) x[c] = *reinterpret_cast<const u32x4 *>(hist + c * kSelBuckets + top - (kMine - 1));
#pragma unroll
        for (int q = 0; q < kMine; ++q)
#pragma unroll
            for (int c = 0; c < kHistCopies; ++c) a[q] += x[c][kMine - 1 - q];
    }
    const unsigned mine = a[0] + a[1] + a[2] + a[3];
    unsigned total;
    const unsigned incl = block_scan(mine, scratch, total);
    if (threadIdx.x == 0) { // fewer candidates than needed cannot happen (need <= their number); bucket 0 if it did
        found[0] = 0u;
        found[1] = need_in > total ? 0u : need_in;
    }
    __syncthreads();
    unsigned above = incl - mine;
#pragma unroll
    for (int q = 0; q < kMine; ++q) {
        if (above < need_in && need_in <= above + a[q]) { // (an empty bucket never)
            found[0] = (unsigned)(top - q);
            found[1] = need_in - above;
        }
        above += a[q];
    }
    __syncthreads();
    prefix = prefix_in | (found[0] << plan.shift[pass]);
    need = found[1];
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        state[kStateAfter + 2 * pass] = prefix;
        state[kStateAfter + 2 * pass + 1] = need;
    }
    __syncthreads(); // found and scratch may be reused
}

__global__ __launch_bounds__(kSelBlock) void k_subset_sel_hist(const unsigned *__restrict__ counts, int V, SelPlan plan,
                                                               int pass, unsigned *state) {
    __shared__ unsigned hist[kSelBuckets];
    __shared__ unsigned scratch[kSelBlock / 64], found[2];
    const int buckets = sel_buckets(plan, pass);
    for (int i = threadIdx.x; i < buckets; i += kSelBlock) hist[i] = 0u;
    unsigned prefix = 0u, need = 0u;
    if (pass > 0) sel_walk(state, plan, pass - 1, scratch, found, prefix, need);
    __syncthreads();
    const int shift = plan.shift[pass];
    const unsigned digit = (1u << plan.bits[pass]) - 1u;
    const unsigned mask = pass == 0 ? 0u : 0xffffffffu << plan.shift[pass - 1];
    const int per = (V + gridDim.x - 1) / gridDim.x, v0 = blockIdx.x * per, v1 = min(V, v0 + per);
    for (int v = v0 + threadIdx.x; v < v1; v += kSelBlock) {
        const unsigned key = sel_key(plan, counts[v]);
        if ((key & mask) == prefix) atomicAdd(&hist[(key >> shift) & digit], 1u);
    }
    __syncthreads();
    put_hist(hist, buckets, pass, state);
}

// ---- compaction: the ids in ascending order, those with count > T plus the first r ties ----
// Workgroup g owns a contiguous range of ids.  First every workgroup counts its (above, ties); then it adds up what the
// workgroups before it hold (one pair per thread) and places its own ids by two workgroup scans.
__global__ __launch_bounds__(kSelBlock) void k_subset_cmp_count(const unsigned *__restrict__ counts, int V, SelPlan plan,
                                                                unsigned *state) {
    __shared__ unsigned scratch[kSelBlock / 64], found[2];
    unsigned T, r; // the last walk: the prefix is now the whole key, and T, being a count of a listed id, is its own key
    sel_walk(state, plan, plan.passes - 1, scratch, found, T, r);
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        state[1] = T;
        state[3] = r;
    }
    const int per = (V + gridDim.x - 1) / gridDim.x, v0 = blockIdx.x * per, v1 = min(V, v0 + per);
    unsigned above = 0u, ties = 0u;
    for (int v = v0 + threadIdx.x; v < v1; v += kSelBlock) {
        const unsigned c = counts[v];
        above += c > T ? 1u : 0u;
        ties += c == T ? 1u : 0u;
    }
    unsigned ta, tt;
    (void)block_scan(above, scratch, ta);
    (void)block_scan(ties, scratch, tt);
    if (threadIdx.x == 0) {
        state[kStateTotals + 2 * blockIdx.x] = ta;
        state[kStateTotals + 2 * blockIdx.x + 1] = tt;
    }
}

// ids outside the vocabulary: the tokens that no count has (whole workgroups; wave 0 works)
__device__ __forceinline__ void put_invalid(const unsigned *state, long long n_tokens, int *invalid_out) {
    static_assert(kSumSlots == 64, "one slot per lane");
    if (!invalid_out || threadIdx.x >= 64) return;
    unsigned x = state[kStateSums + threadIdx.x];
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) x += __shfl_xor(x, off, 64);
    if (threadIdx.x == 0) invalid_out[0] = (int)(n_tokens - (long long)x);
}

__global__ __launch_bounds__(kSelBlock) void k_subset_cmp_write(const unsigned *__restrict__ counts, int V, int n,
                                                                const unsigned *__restrict__ state, int *ids_out,
                                                                long long n_tokens, int *invalid_out) {
    __shared__ unsigned scratch[kSelBlock / 64];
    if (blockIdx.x == gridDim.x - 1) put_invalid(state, n_tokens, invalid_out);
    const unsigned T = state[1], r = state[3];
    // what the workgroups before this one hold: summed by the whole workgroup
    unsigned above_before, ties_before;
    {
        const bool mine = threadIdx.x < blockIdx.x;
        (void)block_scan(mine ? state[kStateTotals + 2 * threadIdx.x] : 0u, scratch, above_before);
        (void)block_scan(mine ? state[kStateTotals + 2 * threadIdx.x + 1] : 0u, scratch, ties_before);
    }
    unsigned out_before = above_before + min(ties_before, r); // the first r ties in id order are kept
    const int per = (V + gridDim.x - 1) / gridDim.x, v0 = blockIdx.x * per, v1 = min(V, v0 + per);
    for (int vb = v0; vb < v1; vb += kSelBlock) {
        const int v = vb + threadIdx.x;
        const unsigned c = v < v1 ? counts[v] : 0u;
        const bool tie = v < v1 && c == T, above = v < v1 && c > T;
        unsigned tie_total, sel_total;
        const unsigned tie_incl = block_scan(tie ? 1u : 0u, scratch, tie_total);
        const bool take = above || (tie && ties_before + tie_incl <= r);
        const unsigned sel_incl = block_scan(take ? 1u : 0u, scratch, sel_total);
        if (take) {
            const unsigned pos = out_before + sel_incl - 1u;
            if (pos < (unsigned)n) ids_out[pos] = v;
        }
        ties_before += tie_total;
        out_before += sel_total;
    }
}

// the sum of all counts, where k_subset_reduce has not formed it
__global__ __launch_bounds__(256) void k_subset_sum(const unsigned *__restrict__ counts, int V, unsigned *sums) {
    __shared__ unsigned scratch[256 / 64];
    unsigned x = 0u;
    for (int v = blockIdx.x * 256 + threadIdx.x; v < V; v += gridDim.x * 256) x += counts[v];
    add_to_sum(x, scratch, sums);
}
__global__ void k_subset_export(const unsigned *counts, int V, const unsigned *state, long long n_tokens, int *counts_out,
                                int *invalid_out) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (counts_out && i < V) counts_out[i] = (int)counts[i];
    if (blockIdx.x == 0) put_invalid(state, n_tokens, invalid_out);
}

bool aligned16(const void *p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }

// ---- scratch of the entry point that allocates nothing ----------------------------------------------------------
// Counts and selection state of mtp_subset_build_static live in this array instead of a caller's workspace.  Each GPU
// the library runs on holds its own copy at its own address until the process ends; host code reaches it only through
// the per-device pointer below (the array's name is a host-side stand-in, not a device address).
constexpr int kStaticMaxVocab = 262144;
constexpr int kStateWordsFullStatic = 16 + 3 * 4096 * 2 + 2 * 160 + 64; // = kStateWordsFull (spelled out: used in the array bound)
__device__ __align__(256) unsigned scratch[kStaticMaxVocab + kStateWordsFullStatic];
static_assert(kStateWordsFullStatic == kStateWordsFull, "scratch layout");
constexpr int kMaxDevices = 64;
unsigned *g_scratch_ptr[kMaxDevices]; // per device: address of that device's copy of `scratch`, null until looked up
bool g_lds_allowed[kMaxDevices];      // per device: the counting kernel may use all the LDS of a CU
std::mutex g_setup_mutex;

typedef void (*hist_kernel_t)(const int *, long long, int, int, unsigned *, int, unsigned *);
hist_kernel_t hist_kernel(int bits) { return bits == 16 ? k_subset_hist<16> : k_subset_hist<8>; }
typedef void (*reduce_kernel_t)(const unsigned *, int, int, int, SelPlan, unsigned *, unsigned *, int *);
reduce_kernel_t reduce_kernel(int bits) { return bits == 16 ? k_subset_reduce<16> : k_subset_reduce<8>; }

// once per device, with that device current: raise the LDS limit of the counting kernel and (for the static entry
// point) look up the device's copy of the scratch array
int32_t subset_setup(int dev, bool want_scratch, unsigned **scratch_out) {
    if (dev < 0 || dev >= kMaxDevices) return MTP_ERR_CONFIG;
    std::lock_guard<std::mutex> lock(g_setup_mutex);
    if (!g_lds_allowed[dev]) {
        for (int bits : {16, 8})
            if (hipFuncSetAttribute((const void *)hist_kernel(bits), hipFuncAttributeMaxDynamicSharedMemorySize,
                                    (int)hist_lds_bytes(chunk_capacity(bits), bits)) != hipSuccess) {
                (void)hipGetLastError();
                return MTP_ERR_HIP;
            }
        g_lds_allowed[dev] = true;
    }
    if (want_scratch) {
        if (!g_scratch_ptr[dev]) {
            unsigned *ptr = nullptr;
            if (hipGetSymbolAddress((void **)&ptr, HIP_SYMBOL(scratch)) != hipSuccess || !ptr) {
                (void)hipGetLastError();
                return MTP_ERR_HIP;
            }
            g_scratch_ptr[dev] = ptr;
        }
        *scratch_out = g_scratch_ptr[dev];
    }
    return MTP_OK;
}

// everything after the argument checks: `work` holds V counts (with_partials: kCountCopies of them) followed by the selection
// state and, with_partials, by one copy of the bins per workgroup of the counting kernel
int32_t subset_build_on(const int32_t *tokens, int64_t n_tokens, int32_t V, int32_t n, unsigned *work, bool with_partials,
                        int32_t *ids_out, int32_t *counts_out, int32_t *invalid_out, hipStream_t st) {
    unsigned *counts = work;
    const int copies = with_partials ? kCountCopies : 1;
    unsigned *state = counts + copies * round4(V);
    unsigned *partials = with_partials ? state + round4(kStateWordsFull) : nullptr; // (all at multiples of 16 bytes)
    const size_t clear = copies * round4(V) + round4(kStateWordsFull);
    hipLaunchKernelGGL(k_subset_clear, dim3((unsigned)((clear / 4 + 255) / 256)), dim3(256), 0, st, work, clear, state, n);
    const CountPlan cp = count_plan(V);
    const SelPlan sp = sel_plan(n_tokens, n);
    const int slices = stream_slices(cp, n_tokens, with_partials);
    hipLaunchKernelGGL(hist_kernel(cp.bits), dim3(slices, cp.chunks), dim3(kHistBlock), hist_lds_bytes(cp.chunk_ids, cp.bits),
                       st, tokens, (long long)n_tokens, V, cp.chunk_ids, counts, copies, partials);
    if (partials)
        hipLaunchKernelGGL(reduce_kernel(cp.bits), dim3((bin_words(cp.chunk_ids, cp.bits) + kReduceWords - 1) / kReduceWords, cp.chunks),
                           dim3(kSelBlock), 0, st, partials, slices, V, cp.chunk_ids, sp, counts, state, counts_out);
    else if (invalid_out)
        hipLaunchKernelGGL(k_subset_sum, dim3(64), dim3(256), 0, st, counts, V, state + kStateSums);
    if (n > 0) {
        for (int pass = partials ? 1 : 0; pass < sp.passes; ++pass) // (with partials, pass 0 was taken along above)
            hipLaunchKernelGGL(k_subset_sel_hist, dim3(kSelGroups), dim3(kSelBlock), 0, st, counts, V, sp, pass, state);
        hipLaunchKernelGGL(k_subset_cmp_count, dim3(kCmpGroups), dim3(kSelBlock), 0, st, counts, V, sp, state);
        hipLaunchKernelGGL(k_subset_cmp_write, dim3(kCmpGroups), dim3(kSelBlock), 0, st, counts, V, n, state, ids_out,
                           (long long)n_tokens, invalid_out);
    }
    // what the kernels above have not handed out already
    int32_t *counts_left = partials ? nullptr : counts_out, *invalid_left = n > 0 ? nullptr : invalid_out;
    if (counts_left || invalid_left)
        hipLaunchKernelGGL(k_subset_export, dim3(counts_left ? (V + 255) / 256 : 1), dim3(256), 0, st, counts, V, state,
                           (long long)n_tokens, counts_left, invalid_left);
    if (hipGetLastError() != hipSuccess) return MTP_ERR_HIP;
    return MTP_OK;
}

int32_t subset_check_args(const int32_t *tokens, int64_t n_tokens, int32_t vocab_size, int32_t n, const int32_t *ids_out,
                          const int32_t *counts_out, const int32_t *invalid_out) {
    if ((!tokens && n_tokens > 0) || (!ids_out && n > 0)) return MTP_ERR_NULL;
    if (!aligned16(tokens) || !aligned16(ids_out) || !aligned16(counts_out) || !aligned16(invalid_out))
        return MTP_ERR_ALIGN;
    if (vocab_size < 1 || n < 0 || n > vocab_size || n_tokens < 0 || n_tokens >= ((int64_t)1 << 31))
        return MTP_ERR_CONFIG;
    return MTP_OK;
}

} // namespace

extern "C" {

size_t mtp_subset_workspace_bytes(int32_t vocab_size) {
    if (vocab_size < 1) return 0;
    return (kCountCopies * round4(vocab_size) + round4(kStateWordsFull) + partial_words(count_plan(vocab_size))) * 4;
}

int32_t mtp_subset_build(const int32_t *tokens, int64_t n_tokens, int32_t vocab_size, int32_t n, void *workspace,
                         size_t workspace_bytes, int32_t *ids_out, int32_t *counts_out, int32_t *invalid_out,
                         void *hip_stream) {
    if (!workspace) return MTP_ERR_NULL;
    if (!aligned16(workspace)) return MTP_ERR_ALIGN;
    const int32_t rc = subset_check_args(tokens, n_tokens, vocab_size, n, ids_out, counts_out, invalid_out);
    if (rc != MTP_OK) return rc;
    if (workspace_bytes < mtp_subset_workspace_bytes(vocab_size)) return MTP_ERR_WORKSPACE;
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess) return MTP_ERR_HIP;
    const int32_t rs = subset_setup(dev, false, nullptr);
    if (rs != MTP_OK) return rs;
    return subset_build_on(tokens, n_tokens, vocab_size, n, static_cast<unsigned *>(workspace), true, ids_out, counts_out,
                           invalid_out, static_cast<hipStream_t>(hip_stream));
}

int32_t mtp_subset_static_max_vocab(void) { return kStaticMaxVocab; }

int32_t mtp_subset_build_static(const int32_t *tokens, int64_t n_tokens, int32_t vocab_size, int32_t n,
                                int32_t *ids_out, int32_t *counts_out, int32_t *invalid_out, void *hip_stream) {
    const int32_t rc = subset_check_args(tokens, n_tokens, vocab_size, n, ids_out, counts_out, invalid_out);
    if (rc != MTP_OK) return rc;
    if (vocab_size > kStaticMaxVocab) {
        fprintf(stderr, "mtp_subset_build_static: vocab_size %d exceeds the built-in scratch (%d ids); use "
                        "mtp_subset_build with a workspace\n", (int)vocab_size, kStaticMaxVocab);
        return MTP_ERR_WORKSPACE;
    }
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess) return MTP_ERR_HIP;
    unsigned *work = nullptr;
    const int32_t rs = subset_setup(dev, true, &work); // first call on a device: symbol lookup; later: a table read
    if (rs != MTP_OK) return rs;
    return subset_build_on(tokens, n_tokens, vocab_size, n, work, false, ids_out, counts_out, invalid_out,
                           static_cast<hipStream_t>(hip_stream));
}

} // extern "C"
