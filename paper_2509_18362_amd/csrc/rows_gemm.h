// The matrix phases over many rows at once (gfx950): one LDS-tiled matrix product on the matrix cores per phase, for
// calls with more rows than one pass of the batched core (batch.h) serves: a prompt-sized block of positions, a large
// batch, the teacher-forced forward of Sec. 2.1, Eq. (1).  The batched core streams every weight once per 64 rows; here
// a weight tile is read once per block of BM rows and the blocks of one weight tile share an L2.
//
// A workgroup owns BM rows x BN weight rows of the result and walks the reduction in steps of 32 elements.  Activations
// are the bf16 hi + lo halves the producing phase left (the float value to 16 bits of mantissa): two MFMAs per weight
// fragment.  Eight waves, each with a 64 x (16 TJ) piece in accumulators.
// What bounds it: LDS reads.  A step of a wave's piece reads 2 x 64 rows of activations (both halves) and 16 TJ weight
// rows of 64 bytes for 8 TJ MFMAs, so a CU needs 2048 (2 x 64 + 16 TJ) / (64 x 16 TJ) bytes per clock at the matrix
// cores' full rate: 64 with TJ = 8, 160 with the 64 x 32 pieces this kernel had before, of the 128 the LDS delivers; and
// from L2 (2 BM + BN) x 64 bytes per step, 24 bytes per clock and CU with 256 x 256 against 48 with 128 x 128.  Hence
// the largest pieces the registers hold (128 accumulator registers), and where a phase has too few such tiles to fill
// the chip the reduction is split over KP workgroups instead of making the tiles smaller.
// Both operands go from memory straight into LDS (no registers, no store instructions): three stages, a stage requested
// two steps before it is multiplied.  Such a load fills 1 KB of LDS in lane order, so rows cannot be padded; the 16-byte
// chunks of a 64-byte row are stored at position chunk ^ ((row >> 1) & 3) instead (the lane that fills a position
// fetches the chunk that belongs there), which puts the eight rows a quarter of a read covers on different banks.
// Measured at 512 rows of the 7B-shaped head (us; the kernel before, with 64 x 128 to 128 x 256 tiles, operands through
// registers and no split, in brackets): 2d -> d 68 + 16 for the sum of eight parts [111], q/k/v 55 + 14 [139], output
// projection 45 + 16 [68], gate/up 183 [264], down 87 + 22 [154], head of 151680 rows 1210 [1221], of 32768 rows 263 with
// candidates [670: eight passes of the batched core].  The large ones run at 1.05 PFLOP/s of MFMAs, where a plain library
// product of the same size reaches 1.1 (the chip holds about 2 GHz then); reading the next step's fragments ahead of the
// barrier, in two orders, changed nothing.
// The phases and their epilogues are the batched core's (the Bg* structs: same operands, same result layout of a
// 16 x 16 tile).
#pragma once
#include "batch.h"

namespace mtp {

constexpr int kRgBK = 32;            // elements per reduction step
constexpr int kRgRow = kRgBK * 2;    // bytes per LDS row
constexpr int kRgStages = 3;

// WM x WN waves (8 in all), TJ tiles of 16 weight rows per wave
template <int WM, int WN, int TJ>
struct RowsTile {
    static_assert(WM * WN == kWaves, "eight waves");
    static constexpr int WAVES_N = WN, BM = 64 * WM, BN = 16 * TJ * WN;
    static constexpr int NA = BM / 16 / kWaves, NW = BN / 16 / kWaves; // 1 KB pieces per wave and stage: hi (as many lo), weights
    static constexpr int NL = 2 * NA + NW;
    static constexpr int kStage = (2 * BM + BN) * kRgRow;
    static constexpr int kLds = kRgStages * kStage;
    static_assert(BM % (16 * kWaves) == 0 && BN % (16 * kWaves) == 0, "whole pieces per wave");
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
// ones these loads need.  (One wait state between the write of m0 and its use.)
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
template <int WM, int WN, int TJ, class Ph, class Make>
__device__ __forceinline__ void rows_gemm(const DraftParams &pin, Make make_phase, int KP, char *smem) {
    using T = RowsTile<WM, WN, TJ>;
    constexpr int NMAT = Ph::NMAT, BM = T::BM, BN = T::BN, NA = T::NA, NW = T::NW, NL = T::NL;
    constexpr int TI = 4;
    static_assert(TJ % NMAT == 0, "pairs of tiles stay inside a wave's piece");
    const int tid = threadIdx.x, lane = tid & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
    const int i16 = lane & 15, g = lane >> 4;

    DraftParams p = pin;
    Ph ph = make_phase(p);
    const int K = ph.K, nk = K / kRgBK;
    const int ntv = ((ph.rows + 15) / 16) * NMAT; // virtual 16-row tiles
    const int MB = (pin.B + BM - 1) / BM, NB = (ntv * 16 + BN - 1) / BN;
    // Workgroups are dealt to the XCDs round robin.  The M blocks of one (N block, part) read the same weights: numbered
    // eight apart they run on the same XCD at about the same time, and its L2 serves all but the first.
    const int x = blockIdx.x, grp = x / (8 * MB), r = x % (8 * MB);
    const int mblk = r / 8, unit = grp * 8 + (r & 7);
    if (unit >= NB * KP) return; // uniform
    const int nblk = unit / KP, kp = unit % KP;
    const int k0 = (int)((long long)kp * nk / KP), k1 = (int)((long long)(kp + 1) * nk / KP); // k1 > k0: KP <= nk
    p.b0 = mblk * BM;
    p.nb = min(BM, pin.B - p.b0);

    // memory -> LDS: piece = sixteen rows x 64 bytes; lane l fills row l / 4, position l % 4
    const int prow = lane >> 2, pchunk = (lane & 3) ^ ((prow >> 1) & 3);
    const size_t lo_bytes = p.a_lo * 2;
    u32x4 ar = rg_rsrc(ph.in, (uint32_t)(2 * lo_bytes));
    int voff_a[NA];
#pragma unroll
    for (int i = 0; i < NA; ++i)
        voff_a[i] = (int)((size_t)min(p.b0 + 16 * (wave + kWaves * i) + prow, pin.B - 1) * p.a_stride * 2 + pchunk * 16);
    u32x4 wr[NW];
    int voff_w[NW];
#pragma unroll
    for (int i = 0; i < NW; ++i) {
        const int vt = min(nblk * (BN / 16) + wave + kWaves * i, ntv - 1);
        const uint16_t *base;
        int mat_rows, row0, row_end;
        ph.tile(vt, base, mat_rows, row0, row_end);
        wr[i] = rg_rsrc(base, (uint32_t)((size_t)mat_rows * K * 2));
        int wrow = min(row0 + prow, row_end - 1);
        if (Ph::GATHER && ph.ids) wrow = ph.ids[wrow];
        voff_w[i] = (int)((size_t)wrow * K * 2 + pchunk * 16);
    }
    // an LDS address is the low half of the generic one
    const uint32_t lds0 = __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)(__attribute__((address_space(3))) char *)smem);
    auto request = [&](int ks, int stage) { // steps past the range repeat its last one (in bounds, nobody reads them)
        const int soff = min(ks, k1 - 1) * kRgRow;
        const uint32_t at = lds0 + stage * T::kStage + wave * 1024;
#pragma unroll
        for (int i = 0; i < NA; ++i) {
            rg_load_lds(ar, at + i * kWaves * 1024, voff_a[i], soff);
            rg_load_lds(ar, at + (BM * kRgRow) + i * kWaves * 1024, voff_a[i], soff + (int)lo_bytes);
        }
#pragma unroll
        for (int i = 0; i < NW; ++i) rg_load_lds(wr[i], at + 2 * (BM * kRgRow) + i * kWaves * 1024, voff_w[i], soff);
    };

    // s_b = 1/sqrt(mean(u_b^2) + eps) of the workgroup's rows from the producer's per-tile sums of squares: kBlock / BM
    // threads per row, asked for here (eight loads at a time) so that the epilogue finds it in a register
    constexpr int TPR = kBlock / BM;
    float my_scale = 0.f;
    if (Ph::SCALE >= 0 && KP == 1) {
        const int npart = p.d / 16, sub = tid & (TPR - 1);
        const float *part = p.ssq + ((size_t)Ph::SCALE * p.max_batch + min(p.b0 + tid / TPR, pin.B - 1)) * npart;
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

    const int wm = wave / WN, wn = wave % WN; // the wave's piece: rows 64 wm .., weight rows 16 TJ wn ..
    const int frag = i16 * kRgRow + ((g ^ ((i16 >> 1) & 3)) * 16);
    const char *abase = smem + wm * 64 * kRgRow + frag, *wbase = smem + 2 * (BM * kRgRow) + wn * (16 * TJ) * kRgRow + frag;
    f32x4 acc[TI][TJ];
#pragma unroll
    for (int ti = 0; ti < TI; ++ti)
#pragma unroll
        for (int tj = 0; tj < TJ; ++tj) acc[ti][tj] = f32x4{0.f, 0.f, 0.f, 0.f};

    // (a scalar register written by the vector unit needs five wait states before a load reads it; the compiler does not
    // look into the assembler of the requests)
    asm volatile("s_nop 7" : "+s"(ar));
#pragma unroll
    for (int i = 0; i < NW; ++i) asm volatile("s_nop 7" : "+s"(wr[i]));
    request(k0, 0);
    request(k0 + 1, 1);
    int stage = 0;
    for (int ks = k0; ks < k1; ++ks) {
        // This wave's pieces of step ks have landed (those of ks + 1 may still be on their way) and its LDS reads of step
        // ks - 1 are back; after the barrier that holds for all waves: step ks can be read, and the stage of step
        // ks - 1 takes step ks + 2.
        asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" : : "n"(NL) : "memory");
        request(ks + 2, stage == 0 ? kRgStages - 1 : stage - 1);
        const char *as = abase + stage * T::kStage, *ws = wbase + stage * T::kStage;
        u32x4 wf[TJ];
#pragma unroll
        for (int tj = 0; tj < TJ; ++tj) wf[tj] = *reinterpret_cast<const u32x4 *>(ws + tj * 16 * kRgRow);
#pragma unroll
        for (int ti = 0; ti < TI; ++ti) {
            const u32x4 ah = *reinterpret_cast<const u32x4 *>(as + ti * 16 * kRgRow);
            const u32x4 al = *reinterpret_cast<const u32x4 *>(as + (BM * kRgRow) + ti * 16 * kRgRow);
#pragma unroll
            for (int tj = 0; tj < TJ; ++tj) acc[ti][tj] = mfma16(ah, wf[tj], acc[ti][tj]);
#pragma unroll
            for (int tj = 0; tj < TJ; ++tj) acc[ti][tj] = mfma16(al, wf[tj], acc[ti][tj]);
        }
        stage = stage == kRgStages - 1 ? 0 : stage + 1;
    }
    // the trailing requests have landed and every wave is done reading: the LDS is free
    asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" : : : "memory");

    // D[i][j] of a 16 x 16 tile: lane (i16, g) holds rows 4 g + v (v = 0..3), weight row i16 - the batched core's layout
    if (KP > 1) {
        const int RT = MB * (BM / 16);
#pragma unroll
        for (int ti = 0; ti < TI; ++ti)
#pragma unroll
            for (int tj = 0; tj < TJ; ++tj) {
                const int vt = nblk * (BN / 16) + wn * TJ + tj, rt = mblk * (BM / 16) + wm * 4 + ti;
                if (vt < ntv && rt * 16 < pin.B)
                    *reinterpret_cast<f32x4 *>(p.part + ((((size_t)kp * ntv + vt) * RT + rt) * kWave + lane) * 4) = acc[ti][tj];
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
                ph.epi_best(64 * wm + 16 * ti + 4 * g, nblk * (BN / 16) + wn * TJ + tj, i16, acc[ti][tj], scale, best);
            if (Ph::CANDS) {
#pragma unroll
                for (int c = 0; c < 4; ++c) {
                    unsigned long long m = best[c];
#pragma unroll
                    for (int off = 1; off < 16; off <<= 1) {
                        const unsigned long long o = __shfl_xor(m, off, kWave);
                        m = o > m ? o : m;
                    }
                    if (i16 == 0) red[wn * BM + 64 * wm + 16 * ti + 4 * g + c] = m;
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
    } else {
#pragma unroll
        for (int ti = 0; ti < TI; ++ti)
#pragma unroll
            for (int tj = 0; tj < TJ; tj += NMAT) {
                const int vt = nblk * (BN / 16) + wn * TJ + tj;
                if (vt >= ntv) continue; // uniform per wave
                f32x4 sums[NMAT];
#pragma unroll
                for (int m = 0; m < NMAT; ++m) sums[m] = acc[ti][tj + m];
                ph.epi(64 * wm + 16 * ti + 4 * g, vt, i16, sums, scale);
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
    p.b0 = rt * 16;
    p.nb = min(16, pin.B - p.b0);
    Ph ph = make_phase(p);
    if (Ph::SCALE >= 0) { // thirty-two threads per row
        const int npart = p.d / 16, sub = tid & 31;
        const float *part = p.ssq + ((size_t)Ph::SCALE * p.max_batch + min(p.b0 + tid / 32, pin.B - 1)) * npart;
        float sum = 0.f;
        for (int i0 = sub; i0 < npart; i0 += 32 * 8) {
            float v[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) v[u] = i0 + u * 32 < npart ? part[i0 + u * 32] : 0.f;
#pragma unroll
            for (int u = 0; u < 8; ++u) sum += v[u];
        }
#pragma unroll
        for (int off = 1; off < 32; off <<= 1) sum += __shfl_xor(sum, off, kWave);
        if (sub == 0) scale[tid / 32] = 1.0f / sqrtf(sum / (float)p.d + p.eps);
    }
    __syncthreads();
    const int ntv = ((ph.rows + 15) / 16) * NMAT;
    const size_t kstride = (size_t)ntv * RT * kWave * 4;
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
        ph.epi((lane >> 4) * 4, vt, lane & 15, sums, scale);
    }
}

} // namespace mtp
