// The matrix phases as LDS-tiled matrix products on the matrix cores (gfx950), one per phase: every call of more than 16 rows
// (a batch, the confirmed positions of one, a prompt, the teacher-forced forward of Sec. 2.1, Eq. (1)) and, from two rows
// on, phases of narrow heads and lists (rows_route in rows_plan.h).  The batched core (batch.h)
// streams every weight once per 64 rows; here a weight tile is read once per block of BM rows (16 to 256) and the blocks of one
// weight tile share an L2.
//
// A workgroup owns BM rows x BN weight rows of the result and walks the reduction in steps of 32 or 64 elements.  Activations
// are the bf16 hi + lo halves the producing phase left (the float value to 16 bits of mantissa): two MFMAs per weight
// fragment.  Eight waves, each with a (16 TI) x (16 TJ) piece in accumulators.
// What bounds it: at few rows reading the weights, at many (pieces of 64 rows) LDS reads.  A step of a wave's piece reads 2 x
// 64 rows of activations (both halves) and 16 TJ weight rows of 64 bytes for 8 TJ MFMAs, so a CU needs
// 2048 (2 x 64 + 16 TJ) / (64 x 16 TJ) bytes per clock at the matrix cores' full rate: 64 with TJ = 8, 160 with TJ = 2, of
// the 128 the LDS delivers; and from L2 (2 BM + BN) x 64 bytes per step, 24 bytes per clock and CU with 256 x 256 against 48
// with 128 x 128.  Hence the largest pieces the registers hold (128 accumulator registers), and where a phase has too few
// such tiles to fill the chip the reduction is split over KP workgroups instead of making the tiles smaller.
// Both operands go from memory straight into LDS (no registers, no store instructions): a ring of stages, three with the
// large tiles, a stage requested two steps (with more stages, earlier) before it is multiplied.  Such a load fills 1 KB of LDS
// in lane order, so rows cannot be padded; the 16-byte
// chunks of a 64-byte row are stored at position chunk ^ ((row >> 1) & 3) instead (the lane that fills a position
// fetches the chunk that belongs there), which puts the eight rows a quarter of a read covers on different banks.
// With large tiles the two halves of the workgroup take turns, one reading its operands from LDS while the other multiplies.
// Measured at 512 rows of the 7B-shaped head (us; in brackets with all eight waves in step): 2d -> d 61 [66], q/k/v 48 [52],
// output projection 39 [43], gate/up 161 [181], down 76 [84], head of 151680 rows 1097 [1222], each split phase + 14 to 19 for
// the sum of its parts; the head of 32768 rows with candidates at 509 rows 252 [280].  The large ones now run at 1.16 PFLOP/s of
// MFMAs, 1.25 while every CU has a tile (1186 tiles of 256 x 256 are 4.6 rounds); a plain library product of 8192 cubed
// reaches 1.22.
// The phases and their epilogues are the batched core's (the Bg* structs: same operands, same result layout of a
// 16 x 16 tile).
#pragma once
#include "batch.h"
#include "rows_plan.h"

namespace mtp {

// WM x WN waves (8 in all), each with TI row tiles x TJ weight-row tiles of sixteen; ST stages of the LDS ring of BK elements
// of the reduction (HALF: the last step is half a one).
template <int TI_, int WM_, int WN_, int TJ_, int ST_, int BK_ = kRgBK, bool HALF_ = false>
struct RowsTile {
    static_assert(WM_ * WN_ == kWaves, "eight waves");
    static constexpr int TI = TI_, WM = WM_, WN = WN_, TJ = TJ_, ST = ST_, BK = BK_;
    static constexpr int kRow = BK * 2, kPieceRows = 1024 / kRow, kChunks = kRow / 16; // a row's bytes, rows of a piece
    static constexpr int BM = 16 * TI * WM, BN = 16 * TJ * WN;
    // 1 KB pieces (whole rows) of a stage: the hi rows, the lo rows, the weight rows; a wave fetches NA of the
    // activations' (with fewer pieces than waves some are fetched twice) and NW of the weights'
    static constexpr int AP = 2 * BM / kPieceRows, NA = (AP + kWaves - 1) / kWaves, NW = BN / kPieceRows / kWaves, NL = NA + NW;
    static constexpr int kStage = (2 * BM + BN) * kRow;
    static constexpr int kLds = ST * kStage;
    // How the sums are rounded.  Every MFMA of a chain rounds its accumulator once, and a chain that takes the lo products
    // along (2^-9 of the hi ones) loses their low bits in the large sum: one chain over a whole reduction is less exact than
    // the batched core, whose waves and parts add up short ones (1 to 2 % of a draft step's error, most of which is the 16
    // bits of the activations).  So where the registers allow, the lo halves have accumulators of their own; the smallest tiles
    // also have one set per half step; and the sums move to another set every CHAIN steps - in the smallest tiles and, for
    // tiles of up to 24 accumulators, in the output head, whose sums are outputs (elsewhere the error is the batched core's
    // without that).  Costs 0.5 % of a step of a 1024-wide head, nothing measurable at 4096.
    static constexpr bool kApart = TI * TJ <= 8;
    static constexpr int SETS = TI * TJ <= 2 ? 2 : 1, CHAIN = TI * TJ <= 24 ? 16 : 0;
    static_assert(SETS == 1 || BK == 64, "half steps");
    static constexpr bool HALF = HALF_;
    static_assert(BK == 32 || BK == 64, "the chunk order below");
    static_assert(!HALF || BK == 64, "half a step");
    static_assert(BN % (kPieceRows * kWaves) == 0 && (AP % kWaves == 0 || kWaves % AP == 0), "whole pieces per wave");
    static_assert((ST - 2) * NL < 64, "the wait counts the requests of the later stages");
};

// The output head over many rows: BgHead's operands; CAND: also the best (logit, position) of every row among the
// workgroup's weight rows (callers that want drafts), else logits only.
template <bool CAND>
struct BgHeadRows : BgBase {
    static constexpr int WHICH = BG_LMHEAD;
    static constexpr bool STREAM = false, GATHER = true, CANDS = CAND;
    static constexpr int SCALE = SSQ_X2;
    int step;
    __device__ BgHeadRows(const DraftParams &p_, int step_) : BgBase(p_, p_.d, p_.n, p_.act[1]), step(step_) {
        ids = p_.ids;
    }
    __device__ __forceinline__ void tile(int vt, const uint16_t *&base, int &mat_rows, int &row0, int &row_end) const {
        base = p.lm_head;
        mat_rows = p.V;
        row_end = p.n;
        row0 = vt * 16;
    }
    __device__ __forceinline__ void epi_best(int bf, int vt, int j, const f32x4 &s, const float *scale,
                                             unsigned long long (&best)[4]) const {
        const int pos = vt * 16 + j;
        const float v[4] = {s.x, s.y, s.z, s.w};
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            const int bl = bf + c;
            if (bl < p.nb && pos < p.n) {
                const float logit = v[c] * scale[bl];
                if (p.logits_out) p.logits_out[((size_t)(p.b0 + bl) * p.K + step) * p.logit_stride + pos] = logit;
                if (CAND) {
                    const unsigned long long key = argmax_key(logit, (uint32_t)pos);
                    best[c] = key > best[c] ? key : best[c];
                }
            }
        }
    }
    __device__ __forceinline__ void epi(int, int, int, const f32x4 (&)[1], const float *) const {}
};
template <class Ph>
struct IsHeadRows {
    static constexpr bool value = false, cands = false;
};
template <bool CAND>
struct IsHeadRows<BgHeadRows<CAND>> {
    static constexpr bool value = true, cands = CAND;
};

// One 1 KB piece from memory into LDS: lane l fetches 16 bytes at voff[l] + soff of the buffer, they land at lds + 16 l.
// In assembler because the compiler, which cannot tell the stages of the ring apart, would wait for ALL such loads in
// flight before the next LDS read; there are no output registers, and the counted waits of the main loop are the only
// ones these loads need.  (One wait state between the write of m0 and its use; m0 is reserved, the compiler writes it itself
// wherever it needs it.)
__device__ __forceinline__ void rg_load_lds(const u32x4 &rs, uint32_t lds, int voff, int soff) {
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, %3 offen lds"
                 :
                 : "s"(lds), "v"(voff), "s"(rs), "s"(soff)
                 : "memory");
}
// buffer descriptor of `bytes` bytes at a wave-uniform address: out-of-range reads return zeros
__device__ __forceinline__ u32x4 rg_rsrc(const uint16_t *base, uint32_t bytes) {
    const unsigned long long a = (unsigned long long)(uintptr_t)base;
    return u32x4{(uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)a),
                 (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(a >> 32)) & 0xffffu,
                 (uint32_t)__builtin_amdgcn_readfirstlane((int)bytes), 0x00020000u};
}

// pin: the DraftParams of the launch (all rows); the phase object is built on a copy whose (b0, nb) name the
// workgroup's rows, which is what the epilogues index with.  KP > 1: the workgroup's sums go to the partial buffer
// ([part][virtual tile][row tile], k_rows_epilogue adds them up).
template <class T, class Ph, class Make>
__device__ __forceinline__ void rows_gemm(const DraftParams &pin, Make make_phase, int KP, char *smem) {
    constexpr int NMAT = Ph::NMAT, BM = T::BM, BN = T::BN, NA = T::NA, NW = T::NW, NL = T::NL, ST = T::ST;
    constexpr int TI = T::TI, TJ = T::TJ, WN = T::WN;
    constexpr bool kApart = T::kApart;
    constexpr int SETS = T::SETS;
    constexpr int kChain = SETS > 1 || IsHeadRows<Ph>::value ? T::CHAIN : 0; // (see RowsTile)
    constexpr bool kPairApart = TJ % NMAT != 0; // the tiles of a pair sit in neighbouring waves
    static_assert(!kPairApart || (TJ == 1 && NMAT == 2 && T::WM == 1), "pairs of tiles: inside a wave's piece, or one each");
    const int tid = threadIdx.x, lane = tid & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
    const int i16 = lane & 15, g = lane >> 4;

    DraftParams p = pin;
    Ph ph = make_phase(p);
    constexpr int kRow = T::kRow, PR = T::kPieceRows;
    const int K = ph.K, nk = (K + (T::HALF ? 32 : 0)) / T::BK;
    const int ntv = ((ph.rows + 15) / 16) * NMAT; // virtual 16-row tiles
    const int R = pin.seq_hi - pin.seq_lo; // rows of the launch: all of the call's, or those that share an id list
    const int MB = (R + BM - 1) / BM, NB = (ntv * 16 + BN - 1) / BN;
    // Workgroups are dealt to the XCDs round robin.  The M blocks of one (N block, part) read the same weights: numbered
    // eight apart they run on the same XCD at about the same time, and its L2 serves all but the first.
    const int x = blockIdx.x, grp = x / (8 * MB), r = x % (8 * MB);
    const int mblk = r / 8, unit = grp * 8 + (r & 7);
    if (unit >= NB * KP) return; // uniform
    // (said to be wave-uniform: a division runs on the vector unit, and the requests want scalar offsets)
    const int nblk = __builtin_amdgcn_readfirstlane(unit / KP), kp = unit - nblk * KP;
    const int k0 = __builtin_amdgcn_readfirstlane(kp * nk / KP);
    const int k1 = __builtin_amdgcn_readfirstlane((kp + 1) * nk / KP); // k1 > k0: KP <= nk
    // Workgroups of a call with one block of rows start at different places of their rows (and come back to the beginning):
    // rows lie a power of two apart, and while all of them read the same 128 bytes of their rows only some of the memory
    // channels have work (64 rows, 32768 weight rows of 8 KB: 71 us without, 63 with).  The workgroups of a die are spread evenly
    // over the reduction (five steps on from one to the next left some of 32 close together; three id lists at 24 sequences, whole call:
    // within what runs differ by).  With several blocks of rows the
    // workgroups of a die stay together instead, so that the activations they read come from their L2.
    // (HALF: a reduction of an odd number of 32s in steps of 64.  The half step keeps its place at the end, kw ends the whole
    // ones; what its second half brings lies behind the rows' ends and is not multiplied.  Kernels of its own, because the
    // few instructions cost every other width 1 to 2 % of a short step.)
    const int kw = T::HALF && k1 == nk ? k1 - 1 : k1;
    const int rot = MB == 1 ? ((unit >> 3) & 31) * (kw - k0) >> 5 : 0;
    p.b0 = pin.seq_lo + mblk * BM;
    p.nb = min(BM, pin.seq_hi - p.b0);

    // memory -> LDS: a lane fills one 16-byte position of one row of the piece, with the chunk that belongs there
    auto chunk_order = [](int row) { return T::BK == 64 ? row & 7 : (row >> 1) & 3; };
    const int prow = lane / T::kChunks, pchunk = (lane % T::kChunks) ^ chunk_order(prow);
    const size_t lo_bytes = p.a_lo * 2;
    u32x4 ar = rg_rsrc(ph.in, (uint32_t)(2 * lo_bytes));
    int voff_a[NA], dst_a[NA];
#pragma unroll
    for (int i = 0; i < NA; ++i) {
        const int q = (wave + kWaves * i) % T::AP, lo = q >= BM / PR ? 1 : 0, row = (q - lo * (BM / PR)) * PR + prow;
        voff_a[i] = (int)((size_t)min(p.b0 + row, pin.seq_hi - 1) * p.a_stride * 2 + (lo ? lo_bytes : 0) + pchunk * 16);
        dst_a[i] = q * 1024; // the lo rows lie behind the hi rows
    }
    u32x4 wr[NW];
    int voff_w[NW];
#pragma unroll
    for (int i = 0; i < NW; ++i) {
        const int q0 = (wave + kWaves * i) * PR; // first row of the piece in the block
        const int vt = min(nblk * (BN / 16) + q0 / 16, ntv - 1);
        const uint16_t *base;
        int mat_rows, row0, row_end;
        ph.tile(vt, base, mat_rows, row0, row_end);
        wr[i] = rg_rsrc(base, (uint32_t)((size_t)mat_rows * K * 2));
        int wrow = min(row0 + q0 % 16 + prow, row_end - 1);
        if (Ph::GATHER && ph.ids) wrow = ph.ids[wrow];
        voff_w[i] = (int)((size_t)wrow * K * 2 + pchunk * 16);
    }
    // an LDS address is the low half of the generic one
    const uint32_t lds0 = __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)(__attribute__((address_space(3))) char *)smem);
    // Steps past the range are requested beyond the buffers' ends (zeros, no traffic): the count of requests in flight does
    // not depend on the step.
    auto request = [&](int ks, int stage) {
        const bool live = ks < k1;
        const int kr = T::HALF && ks >= kw ? ks : ks + rot >= kw ? ks + rot - (kw - k0) : ks + rot;
        const int soff = live ? kr * kRow : 0;
        const uint32_t at = lds0 + stage * T::kStage;
#pragma unroll
        for (int i = 0; i < NA; ++i) rg_load_lds(ar, at + dst_a[i], live ? voff_a[i] : (int)kOobOffset, soff);
#pragma unroll
        for (int i = 0; i < NW; ++i)
            rg_load_lds(wr[i], at + 2 * (BM * kRow) + (wave + i * kWaves) * 1024, live ? voff_w[i] : (int)kOobOffset, soff);
    };

    // s_b = 1/sqrt(mean(u_b^2) + eps) of the workgroup's rows from the producer's per-tile sums of squares: kBlock / BM
    // threads per row, asked for here (eight loads at a time) so that the epilogue finds it in a register
    constexpr int TPR = kBlock / BM;
    float my_scale = 0.f;
    if (Ph::SCALE >= 0 && KP == 1) {
        const int npart = p.d / 16, sub = tid & (TPR - 1);
        const float *part = p.ssq + ((size_t)Ph::SCALE * p.max_batch + min(p.b0 + tid / TPR, pin.seq_hi - 1)) * npart;
        float sum = 0.f;
        for (int i0 = sub; i0 < npart; i0 += TPR * 8) {
            float v[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) v[u] = i0 + u * TPR < npart ? part[i0 + u * TPR] : 0.f;
#pragma unroll
            for (int u = 0; u < 8; ++u) sum += v[u];
        }
#pragma unroll
        for (int off = 1; off < TPR; off <<= 1) sum += __shfl_xor(sum, off, kWave);
        my_scale = 1.0f / sqrtf(sum / (float)p.d + p.eps);
    }

    const int wm = wave / WN, wn = wave % WN; // the wave's piece: rows 16 TI wm .., weight rows 16 TJ wn ..
    int frag[T::BK / 32]; // 16-byte chunk g of half h of a row, where the order of the chunks puts it
#pragma unroll
    for (int h = 0; h < T::BK / 32; ++h) frag[h] = i16 * kRow + (((4 * h + g) ^ chunk_order(i16)) * 16);
    const char *abase = smem + wm * (16 * TI) * kRow, *wbase = smem + 2 * (BM * kRow) + wn * (16 * TJ) * kRow;
    // acc: the sums of the present chains; lo: of the lo halves, where they are apart; tot: of the chains before
    f32x4 acc[SETS][TI][TJ], lo[kApart ? TI : 1][kApart ? TJ : 1], tot[kChain ? TI : 1][kChain ? TJ : 1];
#pragma unroll
    for (int ti = 0; ti < TI; ++ti)
#pragma unroll
        for (int tj = 0; tj < TJ; ++tj) {
#pragma unroll
            for (int u = 0; u < SETS; ++u) acc[u][ti][tj] = f32x4{0.f, 0.f, 0.f, 0.f};
            if constexpr (kApart) lo[ti][tj] = acc[0][ti][tj];
            if constexpr (kChain > 0) tot[ti][tj] = acc[0][ti][tj];
        }
    auto end_chains = [&]() {
#pragma unroll
        for (int ti = 0; ti < TI; ++ti)
#pragma unroll
            for (int tj = 0; tj < TJ; ++tj) {
                f32x4 a = acc[0][ti][tj];
                if constexpr (SETS == 2) a += acc[SETS - 1][ti][tj];
                tot[kChain ? ti : 0][kChain ? tj : 0] += a;
#pragma unroll
                for (int u = 0; u < SETS; ++u) acc[u][ti][tj] = f32x4{0.f, 0.f, 0.f, 0.f};
            }
    };

    // (a scalar register written by the vector unit needs five wait states before a load reads it; the compiler does not
    // look into the assembler of the requests)
    asm volatile("s_nop 7" : "+s"(ar));
#pragma unroll
    for (int i = 0; i < NW; ++i) asm volatile("s_nop 7" : "+s"(wr[i]));
#pragma unroll
    for (int u = 0; u < ST - 1; ++u) request(k0 + u, u);
    int stage = 0;
    // This wave's pieces of step ks have landed (those of the later steps may still be on their way) and its LDS reads of
    // step ks - 1 are back; after the barrier that holds for all waves: step ks can be read, and the stage of step
    // ks - 1 takes step ks + ST - 1.
    auto await_step = [&]() { asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" : : "n"((ST - 2) * NL) : "memory"); };
    auto multiply = [&](int stage, int h) {
        const char *as = abase + stage * T::kStage, *ws = wbase + stage * T::kStage;
        u32x4 wf[TJ];
#pragma unroll
        for (int tj = 0; tj < TJ; ++tj) wf[tj] = *reinterpret_cast<const u32x4 *>(ws + frag[h] + tj * 16 * kRow);
#pragma unroll
        for (int ti = 0; ti < TI; ++ti) {
            const u32x4 ah = *reinterpret_cast<const u32x4 *>(as + frag[h] + ti * 16 * kRow);
            const u32x4 al = *reinterpret_cast<const u32x4 *>(as + frag[h] + (BM * kRow) + ti * 16 * kRow);
#pragma unroll
            for (int tj = 0; tj < TJ; ++tj) acc[h % SETS][ti][tj] = mfma16(ah, wf[tj], acc[h % SETS][ti][tj]);
#pragma unroll
            for (int tj = 0; tj < TJ; ++tj) {
                f32x4 &l = kApart ? lo[kApart ? ti : 0][kApart ? tj : 0] : acc[h % SETS][ti][tj];
                l = mfma16(al, wf[tj], l);
            }
        }
    };
    // (chains in an outer loop, so that the inner one stays short: with the moves behind a branch of the inner loop a draft
    // step of a 1024-wide head took 2.5 % longer, most launches of which are 8 to 16 steps)
    int ks = k0;
    // Large pieces in turns: the four waves of one half of the workgroup (one per SIMD) read their operands of a step while the
    // other four multiply, then the halves change places.  In step with one another all eight read first (128 KB a step, 1000
    // cycles of the LDS) and the matrix cores waited for most of it.  The second half runs one barrier behind.  A step is
    // read by the first half in interval 2 ks and by the second in 2 ks + 1; its stage is requested again from interval
    // 2 ks + 2 on, and a wave has waited for its own pieces of a step before the barrier that opens the step's first interval.
    constexpr bool kTurns = T::BK == 32 && TI * TJ >= 24 && kChain == 0 && ST == 3;
    if constexpr (kTurns) {
        const bool second = wave >= kWaves / 2; // uniform
        auto landed = [&]() { asm volatile("s_waitcnt vmcnt(%0)" : : "n"(NL) : "memory"); }; // all but the newest step
        auto turn = [&]() {
            asm volatile("s_barrier" : : : "memory");
            __builtin_amdgcn_sched_barrier(0);
        };
        landed();
        turn();
        if (second) turn();
        for (; ks < kw; ++ks) {
            const char *as = abase + stage * T::kStage + frag[0], *ws = wbase + stage * T::kStage + frag[0];
            request(ks + ST - 1, stage == 0 ? ST - 1 : stage - 1);
            u32x4 wf[TJ], ah[TI], al[TI];
#pragma unroll
            for (int tj = 0; tj < TJ; ++tj) wf[tj] = *reinterpret_cast<const u32x4 *>(ws + tj * 16 * kRow);
#pragma unroll
            for (int ti = 0; ti < TI; ++ti) {
                ah[ti] = *reinterpret_cast<const u32x4 *>(as + ti * 16 * kRow);
                al[ti] = *reinterpret_cast<const u32x4 *>(as + (BM * kRow) + ti * 16 * kRow);
            }
            asm volatile("s_waitcnt lgkmcnt(0)" : : : "memory");
            if (second) landed();
            __builtin_amdgcn_sched_barrier(0);
            turn();
#pragma unroll
            for (int ti = 0; ti < TI; ++ti) {
#pragma unroll
                for (int tj = 0; tj < TJ; ++tj) acc[0][ti][tj] = mfma16(ah[ti], wf[tj], acc[0][ti][tj]);
#pragma unroll
                for (int tj = 0; tj < TJ; ++tj) acc[0][ti][tj] = mfma16(al[ti], wf[tj], acc[0][ti][tj]);
            }
            __builtin_amdgcn_sched_barrier(0);
            if (!second) landed();
            turn();
            stage = stage == ST - 1 ? 0 : stage + 1;
        }
        if (!second) turn();
    } else
    do {
        const int end = kChain > 0 ? min(ks + kChain, kw) : kw;
        for (; ks < end; ++ks) {
            await_step();
            request(ks + ST - 1, stage == 0 ? ST - 1 : stage - 1);
#pragma unroll
            for (int h = 0; h < T::BK / 32; ++h) multiply(stage, h);
            stage = stage == ST - 1 ? 0 : stage + 1;
        }
        if (T::HALF && ks == kw && kw < k1) { // the half step (requested with the others)
            await_step();
            multiply(stage, 0);
        }
        if constexpr (kChain > 0) end_chains();
    } while (kChain > 0 && ks < kw);
    f32x4(&sum)[TI][TJ] = kChain > 0 ? reinterpret_cast<f32x4(&)[TI][TJ]>(tot) : acc[0];
    if constexpr (kApart)
#pragma unroll
        for (int ti = 0; ti < TI; ++ti)
#pragma unroll
            for (int tj = 0; tj < TJ; ++tj) sum[ti][tj] += lo[ti][tj];
    // the trailing requests have landed and every wave is done reading: the LDS is free
    asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" : : : "memory");

    // D[i][j] of a 16 x 16 tile: lane (i16, g) holds rows 4 g + v (v = 0..3), weight row i16 - the batched core's layout
    if (KP > 1) {
        const int RT = MB * (BM / 16);
#pragma unroll
        for (int ti = 0; ti < TI; ++ti)
#pragma unroll
            for (int tj = 0; tj < TJ; ++tj) {
                const int vt = nblk * (BN / 16) + wn * TJ + tj, rt = mblk * (BM / 16) + wm * TI + ti;
                if (vt < ntv && rt * 16 < R)
                    *reinterpret_cast<f32x4 *>(p.part + ((((size_t)kp * ntv + vt) * RT + rt) * kWave + lane) * 4) = sum[ti][tj];
            }
        return;
    }
    float *scale = reinterpret_cast<float *>(smem);
    if (Ph::SCALE >= 0) {
        if ((tid & (TPR - 1)) == 0) scale[tid / TPR] = my_scale;
        __syncthreads();
    }
    if constexpr (IsHeadRows<Ph>::value) {
        unsigned long long *red = reinterpret_cast<unsigned long long *>(smem + BM * 4); // [WN][BM]
#pragma unroll
        for (int ti = 0; ti < TI; ++ti) {
            unsigned long long best[4] = {0ull, 0ull, 0ull, 0ull};
#pragma unroll
            for (int tj = 0; tj < TJ; ++tj)
                ph.epi_best(16 * (TI * wm + ti) + 4 * g, nblk * (BN / 16) + wn * TJ + tj, i16, sum[ti][tj], scale, best);
            if (Ph::CANDS) {
#pragma unroll
                for (int c = 0; c < 4; ++c) {
                    const unsigned long long m = row16_max_u64(best[c]);
                    if (i16 == 0) red[wn * BM + 16 * (TI * wm + ti) + 4 * g + c] = m;
                }
            }
        }
        if (Ph::CANDS) {
            __syncthreads();
            if (tid < p.nb) { // BM <= 256 < kBlock; one candidate per (row, N block)
                unsigned long long m = 0ull;
#pragma unroll
                for (int w = 0; w < WN; ++w) m = red[w * BM + tid] > m ? red[w * BM + tid] : m;
                p.cand[((size_t)ph.step * p.max_batch + p.b0 + tid) * p.head_grid + nblk] = m;
            }
        }
    } else if constexpr (kPairApart) {
        f32x4 *half = reinterpret_cast<f32x4 *>(smem + 16 * BM); // [kWaves][TI][kWave], behind the scales
        if (wn & 1)
#pragma unroll
            for (int ti = 0; ti < TI; ++ti) half[(wn * TI + ti) * kWave + lane] = sum[ti][0];
        __syncthreads();
        const int vt = nblk * (BN / 16) + wn;
        if (!(wn & 1) && vt < ntv)
#pragma unroll
            for (int ti = 0; ti < TI; ++ti) {
                const f32x4 sums[NMAT] = {sum[ti][0], half[((wn + 1) * TI + ti) * kWave + lane]};
                ph.epi(16 * ti + 4 * g, vt, i16, sums, scale);
            }
    } else {
#pragma unroll
        for (int ti = 0; ti < TI; ++ti)
#pragma unroll
            for (int tj = 0; tj < TJ; tj += NMAT) {
                const int vt = nblk * (BN / 16) + wn * TJ + tj;
                if (vt >= ntv) continue; // uniform per wave
                f32x4 sums[NMAT];
#pragma unroll
                for (int m = 0; m < NMAT; ++m) sums[m] = sum[ti][tj + m];
                ph.epi(16 * (TI * wm + ti) + 4 * g, vt, i16, sums, scale);
            }
    }
}

// The epilogue of a phase whose reduction was split: workgroup (rt, y) adds the KP parts of sixteen rows, in the order of
// the parts, for every gridDim.y-th group of eight virtual tiles (or pairs), one wave per tile.
template <class Ph, class Make>
__device__ __forceinline__ void rows_epilogue(const DraftParams &pin, Make make_phase, int KP, int RT, float *scale) {
    constexpr int NMAT = Ph::NMAT;
    DraftParams p = pin;
    const int rt = blockIdx.x, tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid / kWave;
    p.b0 = pin.seq_lo + rt * 16;
    p.nb = min(16, pin.seq_hi - p.b0);
    Ph ph = make_phase(p);
    if (Ph::SCALE >= 0) { // thirty-two threads per row
        const int npart = p.d / 16, sub = tid & 31;
        const float *part = p.ssq + ((size_t)Ph::SCALE * p.max_batch + min(p.b0 + tid / 32, pin.seq_hi - 1)) * npart;
        float sum = 0.f;
        for (int i0 = sub; i0 < npart; i0 += 32 * 8) {
            float v[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) v[u] = i0 + u * 32 < npart ? part[i0 + u * 32] : 0.f;
#pragma unroll
            for (int u = 0; u < 8; ++u) sum += v[u];
        }
        sum = sum16(row16_sum(sum));
        if (sub == 0) scale[tid / 32] = 1.0f / sqrtf(sum / (float)p.d + p.eps);
    }
    __syncthreads();
    const int ntv = ((ph.rows + 15) / 16) * NMAT;
    const size_t kstride = (size_t)ntv * RT * kWave * 4;
    unsigned long long best[4] = {0ull, 0ull, 0ull, 0ull};
    for (int vt = (blockIdx.y * kWaves + wave) * NMAT; vt < ntv; vt += gridDim.y * kWaves * NMAT) {
        f32x4 sums[NMAT];
#pragma unroll
        for (int m = 0; m < NMAT; ++m) {
            const float *src = p.part + (((size_t)(vt + m) * RT + rt) * kWave + lane) * 4;
            f32x4 s = {0.f, 0.f, 0.f, 0.f};
            for (int k2 = 0; k2 < KP; k2 += 8) { // eight loads in flight
                f32x4 v[8];
#pragma unroll
                for (int u = 0; u < 8; ++u) v[u] = *reinterpret_cast<const f32x4 *>(src + (size_t)min(k2 + u, KP - 1) * kstride);
#pragma unroll
                for (int u = 0; u < 8; ++u)
                    if (k2 + u < KP) s += v[u];
            }
            sums[m] = s;
        }
        if constexpr (IsHeadRows<Ph>::value)
            ph.epi_best((lane >> 4) * 4, vt, lane & 15, sums[0], scale, best);
        else
            ph.epi((lane >> 4) * 4, vt, lane & 15, sums, scale);
    }
    if constexpr (IsHeadRows<Ph>::cands) { // one candidate per (row, blockIdx.y)
        unsigned long long *red = reinterpret_cast<unsigned long long *>(scale + 16); // [kWaves][16]
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            const unsigned long long m = row16_max_u64(best[c]);
            if ((lane & 15) == 0) red[wave * 16 + (lane >> 4) * 4 + c] = m;
        }
        __syncthreads();
        if (tid < p.nb) {
            unsigned long long m = 0ull;
#pragma unroll
            for (int w = 0; w < kWaves; ++w) m = red[w * 16 + tid] > m ? red[w * 16 + tid] : m;
            p.cand[((size_t)ph.step * p.max_batch + p.b0 + tid) * p.head_grid + blockIdx.y] = m;
        }
    }
}

} // namespace mtp
