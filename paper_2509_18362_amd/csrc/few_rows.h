// Matrix phases of 2..16 rows (sequences, or positions of a block), gfx950: one pass over the weights, no split of the
// reduction over workgroups.
//
// A workgroup owns whole tiles of sixteen weight rows; its eight waves split the reduction in chunks of 256 elements (chunk
// c to wave c mod 8) and meet in LDS at the end.  With one 16-row tile per workgroup (4096 weight rows: one per CU) every
// workgroup reads all activations, four bytes per element and row from L2 against two from HBM per weight: 2 x the
// weights at sixteen rows, which L2 delivers beside the HBM stream.  In exchange nothing crosses workgroups.
// Weights: a wave's item is 16 rows x 512 bytes, eight direct-to-LDS loads of two half-KB runs, two items in flight per
// wave.  Runs of 512 bytes instead of one 128-byte line per row and step keep the memory's pages open.  Load u of an item
// brings rows u and u + 8; the landing places of the loads lie 1040 bytes apart, and rows 8..15 are stored with their
// 16-byte pieces exchanged eight places apart, so that the sixteen rows of an operand read fall into different banks.
// Activations: the phase before leaves them in operand order ([element / 8][row][8], act_index), so an operand is one
// contiguous KB (0.25 KB per eight elements); lanes of rows that do not exist ask for nothing.  The operands of a chunk stay
// in registers for all tiles of the workgroup, the next chunk's are requested two chunks ahead.
#pragma once
#include "batch.h"

namespace mtp {

// PACKED: up to eight rows, whose hi and lo halves share one operand (rows 0..7 hi, 8..15 lo): half the activation loads,
// registers and matrix instructions; the two halves of a result are added at the end.
template <bool PACKED>
struct FewShape {
    static constexpr int HL = PACKED ? 1 : 2; // operands per tile of sixteen rows
    static constexpr int KB = 8;              // 32-element blocks of a chunk
    static constexpr int CK = 32 * KB;        // elements of a chunk
    static constexpr int L = 8;               // loads of an item (1 KB each: two rows)
    static constexpr int S = 2;               // items in flight per wave
    static constexpr int LPR = 32;            // lanes per row of a load
    static constexpr int kStep = 1040;        // bytes between the landing places of an item's loads
    static constexpr int kSlot = L * kStep;
    static constexpr int kRing = kWaves * S * kSlot;
    static constexpr int AL = KB * HL;        // activation loads of a chunk
};
// A listed row that does not exist: behind the end of any matrix (but one within 64 KB of 2 GiB, where it may read what is
// there: the row's results go nowhere).  Added to the mark of a missing piece it still does not wrap around.
constexpr uint32_t kFewNoRow = 0x7fff0000u;
constexpr int kFewMaxTiles = 8;
__host__ __device__ inline size_t few_lds_bytes() {
    return (size_t)FewShape<false>::kRing + kBatchMaxSeq * 4 + kFewMaxTiles * 16 * 4;
}

// keeps requests in the order they are written in: the waits below count them
__device__ __forceinline__ void few_order() { asm volatile("" ::: "memory"); }
template <int N>
__device__ __forceinline__ void few_wait() { asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory"); }

// The norm scales s_b = 1/sqrt(mean(u_b^2) + eps) of the pass's rows from the producers' per-tile sums of squares, in two
// parts: the sums are requested behind the first weights and added up when the rest is on its way.
struct FewScales {
    static constexpr int LR = 32, N = 16; // lanes per row, values per lane (8192 wide: 512 tiles)
    float v[N];
    __device__ __forceinline__ void request(const DraftParams &p, int kind) { // (no branch around a load)
        const int row = threadIdx.x / LR, i0 = threadIdx.x % LR, n = row < p.nb ? p.d / 16 : 0;
        const float *src = p.ssq + ((size_t)kind * p.max_batch + p.b0) * (p.d / 16);
        const row_rsrc r = make_row_rsrc(reinterpret_cast<const uint16_t *>(src), p.nb * (p.d / 16) * 4);
#pragma unroll
        for (int u = 0; u < N; ++u) {
            const int i = i0 + LR * u;
            v[u] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(
                r, i < n ? (row * (p.d / 16) + i) * 4 : (int)kOobOffset, 0, 0));
        }
    }
    __device__ __forceinline__ void finish(const DraftParams &p, float *scale_lds) {
        const int row = threadIdx.x / LR;
        float s = 0.f;
#pragma unroll
        for (int u = 0; u < N; ++u) s += v[u];
        s = sum16(row16_sum(s));
        if (threadIdx.x % LR == 0) scale_lds[row] = row < p.nb ? 1.0f / sqrtf(s / (float)p.d + p.eps) : 0.f;
    }
};

// T weight tiles per group (accumulators per wave).  Ph: as for bgemv_lds.
// Workgroup b of the launch owns `per` units (tiles, or gate/up pairs), the first `rem` workgroups one more.
template <bool PACKED, int T, class Ph>
__device__ __forceinline__ void few_rows(const DraftParams &p, Ph &ph, int per, int rem, char *smem) {
    using S_ = FewShape<PACKED>;
    constexpr int HL = S_::HL;
    constexpr int NMAT = Ph::NMAT, KB = S_::KB, CK = S_::CK, L = S_::L, S = S_::S, LPR = S_::LPR;
    static_assert(T % NMAT == 0 && (size_t)T * kWaves * kWave * 16 <= (size_t)S_::kRing, "tiles of a group");
    const int rg = blockIdx.x;
    const int lane = threadIdx.x & (kWave - 1), j = lane & 15, g = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x / kWave));
    const int K = ph.K;
    const int u0 = rg * per + min(rg, rem), u1 = u0 + per + (rg < rem);
    const int vt0 = u0 * NMAT, nvt = (u1 - u0) * NMAT;
    const int ngroups = (nvt + T - 1) / T;

    char *ring = smem + (size_t)wave * S * S_::kSlot;
    f32x4 *red = reinterpret_cast<f32x4 *>(smem); // [kWaves][T][kWave], once the ring is idle
    float *scale_lds = reinterpret_cast<float *>(smem + S_::kRing);
    uint32_t *row_off = reinterpret_cast<uint32_t *>(scale_lds + kBatchMaxSeq); // gathered rows of the group: byte offsets

    // Chunks of this wave, rotated by the workgroup's place on its die (dies take the workgroups in turn): rows lie KB apart, and
    // what one die asks for at a time must not lie at the same place of its rows, nor its workgroups ask for the same
    // activations at once.  33.5 MB of weights alone, 256 workgroups: 7.2 us; rotated by the workgroup's number, which is
    // two places per die, 10.0.
    const int nck = (K + CK - 1) / CK;
    const int nc = wave < nck ? (nck - wave + kWaves - 1) / kWaves : 0;
    const int rot = (((rg >> 3) & 31) * nck) >> 5;
    auto chunk_of = [&](int c) {
        int ck = wave + c * kWaves + rot;
        return ck >= nck ? ck - nck : ck;
    };

    // activations
    const row_rsrc ar = make_row_rsrc(ph.in, p.act_bytes);
    const int lo_bytes = (int)(p.a_lo * 2);
    const int a_step = p.act_frag ? p.act_frag * 64 : 64; // bytes per 32 elements
    int a_lane;
    { // (a mask instead of a branch, which the compiler would put in front of everything: the first requests waited for it)
        const int r = PACKED ? j & 7 : j, row = p.b0 + r;
        const int frag = -(int)(p.act_frag != 0);
        int off = (((g * p.act_frag + row) * 16) & frag) | ((row * p.a_stride * 2 + g * 16) & ~frag);
        if (PACKED && j >= 8) off += lo_bytes;
        a_lane = r < p.nb ? off : (int)kOobOffset;
    }
    // Two chunks' operands in registers where a chunk is one item long; with more tiles one, refilled block by block while the
    // chunk's last item is multiplied.
    constexpr int AB = T == 1 ? 2 : 1;
    u32x4 act[AB][KB][HL];
    auto issue_block = [&](u32x4(&dst)[KB][HL], int c, int kb) {
        const int k = chunk_of(c) * CK + kb * 32, end = c < nc ? K : 0;
        const bool in = k + g * 8 < end;
        const int off = in ? a_lane + k / 32 * a_step : (int)kOobOffset;
        dst[kb][0] = row_load16<false>(ar, off, 0);
        if (HL == 2) dst[kb][HL - 1] = row_load16<false>(ar, off, lo_bytes);
    };
    auto issue_act = [&](u32x4(&dst)[KB][HL], int c) {
#pragma unroll
        for (int kb = 0; kb < KB; ++kb) issue_block(dst, c, kb);
    };

    // weights: lane -> row q L + u of load u, 16-byte piece `piece` of the chunk
    const int q = lane / LPR, piece = (lane % LPR) ^ (q * 8);
    auto issue_w = [&](int grp, int c, int t, int slot) {
        const uint16_t *base;
        int mat_rows, row0, row_end;
        const int tv = grp * T + t;
        ph.tile(vt0 + min(tv, nvt - 1), base, mat_rows, row0, row_end);
        // (plain rows: the descriptor starts at the tile, so the lanes' offsets are the same for every tile)
        const row_rsrc wr = Ph::GATHER ? make_row_rsrc(base, tv < nvt ? (int)((size_t)mat_rows * K * 2) : 0)
                                       : make_row_rsrc(base + (size_t)row0 * K,
                                                       tv < nvt ? (int)((size_t)(mat_rows - row0) * K * 2) : 0);
        const int kel = chunk_of(c) * CK + piece * 8;
        const int end = c < nc ? K : 0;
        const uint32_t koff = kel < end ? (uint32_t)kel * 2 : kOobOffset;
        u32x4 rows[L / 4];
        if (Ph::GATHER)
#pragma unroll
            for (int u = 0; u < L / 4; ++u) rows[u] = *reinterpret_cast<const u32x4 *>(row_off + t * 16 + q * L + u * 4);
        few_order();
#pragma unroll
        for (int u = 0; u < L; ++u) {
            const uint32_t off = Ph::GATHER ? rows[u / 4][u % 4] : (uint32_t)(q * L + u) * (uint32_t)(K * 2);
            __builtin_amdgcn_raw_ptr_buffer_load_lds(
                wr, (__attribute__((address_space(3))) void *)(ring + slot * S_::kSlot + u * S_::kStep), 16,
                (int)(off + koff), 0, 0, Ph::STREAM ? 2 : 0);
        }
        few_order();
    };
    int w_lane[KB]; // where this lane's operand pieces of an item lie
#pragma unroll
    for (int kb = 0; kb < KB; ++kb)
        w_lane[kb] = (j % L) * S_::kStep + (j / L) * (LPR * 16) + (((kb * 4 + g) ^ ((j / L) * 8)) * 16);

    f32x4 acc[T][HL]; // hi and lo products apart: two chains, and the lo sums keep their low bits
#pragma unroll
    for (int t = 0; t < T; ++t) acc[t][0] = acc[t][HL - 1] = f32x4{0.f, 0.f, 0.f, 0.f};

    auto set_rows = [&](int grp) { // a group's gathered rows
        if (!Ph::GATHER) return;
        if (grp > 0) __syncthreads(); // (the group before has requested its last item)
        if ((int)threadIdx.x < T * 16) {
            const int pos = (u0 + grp * T) * 16 + (int)threadIdx.x; // (NMAT = 1)
            const bool ok = pos < min(ph.rows, u1 * 16);
            row_off[threadIdx.x] = ok ? (uint32_t)((ph.ids ? ph.ids[pos] : pos)) * (uint32_t)(K * 2) : kFewNoRow;
        }
        __syncthreads();
    };
    // refill: also ask for the blocks of chunk `next` as this chunk's are used up
    auto consume = [&](u32x4(&a)[KB][HL], int t, int slot, bool refill, int next) {
        const char *src = ring + slot * S_::kSlot;
#pragma unroll
        for (int k4 = 0; k4 < KB; k4 += 4) { // four operand reads at a time
            u32x4 w[4];
#pragma unroll
            for (int kb = 0; kb < 4; ++kb) w[kb] = *reinterpret_cast<const u32x4 *>(src + w_lane[k4 + kb]);
#pragma unroll
            for (int kb = 0; kb < 4; ++kb) {
                acc[t][0] = mfma16(a[k4 + kb][0], w[kb], acc[t][0]);
                if (HL == 2) acc[t][HL - 1] = mfma16(a[k4 + kb][HL - 1], w[kb], acc[t][HL - 1]);
                if (refill) issue_block(a, next, k4 + kb);
            }
        }
    };

    for (int grp = 0; grp < ngroups; ++grp) {
        set_rows(grp);
        int slot = 0; // of the next item to be multiplied
        issue_w(grp, 0, 0, 0);
        FewScales scales;
        if (grp == 0 && Ph::SCALE >= 0) scales.request(p, Ph::SCALE);
        issue_act(act[0], 0);
#pragma unroll
        for (int i = 1; i < S; ++i) issue_w(grp, i / T, i % T, i);
        if (AB == 2) issue_act(act[AB - 1], 1);
        if (grp == 0 && Ph::SCALE >= 0) scales.finish(p, scale_lds);
        // what the epilogue of this wave's (first) slot reads, asked for now
        constexpr int NS = T / NMAT;
        const int t0 = min(grp * T + min(wave, NS - 1) * NMAT, nvt - 1);
        const typename Ph::Pre pre = ph.pre(g * 4, vt0 + t0, j);
        auto chunk = [&](u32x4(&a)[KB][HL], int c) {
#pragma unroll
            for (int t = 0; t < T; ++t) {
                // Newer requests than this item's: the other items in flight and, near the start of a chunk, one chunk's
                // activations (which one buffer's refill asks for one item earlier)
                if (t < S - (AB == 1))
                    few_wait<(S - 1) * L + S_::AL>();
                else
                    few_wait<(S - 1) * L>();
                consume(a, t, slot, AB == 1 && t == T - 1, c + 1);
                asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory"); // the slot has been read
                issue_w(grp, c + (t + S) / T, (t + S) % T, slot);
                slot = (slot + 1) % S;
            }
            if (AB == 2) issue_act(a, c + 2);
        };
        // (one exit per loop: behind a break the compiler no longer knows how many loads are in flight; an odd last chunk of the
        // two-buffer form is followed by one of zeros)
        for (int c = 0; c < nc; c += AB) {
            chunk(act[0], c);
            if (AB == 2) chunk(act[AB - 1], c + 1);
        }
        few_wait<0>(); // (requests past the end: zeros on their way to the ring)
        __syncthreads();
#pragma unroll
        for (int t = 0; t < T; ++t) {
            red[((size_t)wave * T + t) * kWave + lane] = HL == 2 ? acc[t][0] + acc[t][HL - 1] : acc[t][0];
            acc[t][0] = acc[t][HL - 1] = f32x4{0.f, 0.f, 0.f, 0.f};
        }
        __syncthreads();
        static_assert(NS <= kWaves, "one slot per wave");
        if (wave < NS) {
            const int t = wave * NMAT;
            f32x4 sums[NMAT];
#pragma unroll
            for (int m = 0; m < NMAT; ++m) {
                f32x4 v = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int w = 0; w < kWaves; ++w) v += red[((size_t)w * T + t + m) * kWave + lane];
                if (PACKED) // rows 8..15 hold the lo products of rows 0..7
#pragma unroll
                    for (int e = 0; e < 4; ++e) v[e] = sum32(v[e]);
                sums[m] = v;
            }
            if (grp * T + t < nvt) ph.epi(g * 4, vt0 + grp * T + t, j, sums, scale_lds, pre);
        }
        if (grp + 1 < ngroups) __syncthreads(); // the ring is free again
    }
    ph.finish(rg, smem);
}

} // namespace mtp
