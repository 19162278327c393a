// Attention of a long block of new positions (a prompt or a piece of one, the teacher-forced forward) on the matrix cores
// (gfx950): a workgroup of four or eight waves per (sequence, KV head, 16 / G neighbouring positions).
//
// The block's keys and values are in the cache; the sixteen MFMA columns are G query heads of 16 / G positions, which read every
// key and value together, as in phase_attn_mfma (layouts and arithmetic are that kernel's; there the reasons).  There such an
// item has a compute unit to itself (eight waves, 127 KB of LDS) and its splits meet in memory: right for few items of
// thousands of tokens.  With hundreds of positions there are several items for every unit, each of them two rounds of tokens
// between 5 us of set-up and 5 us until the waves' results have met.  Here an item is small - 33 KB of LDS, the merge in the
// place of the tiles, results written whole - so that several of them share a unit and one's set-up and merge pass while others
// multiply.  What bounds it is the chain of a wave's rounds of 32 tokens, 1.2 us each.  509 positions of an
// empty cache, 32 query and 8 KV heads of 128: 75 us there, 30 here with four waves, 34 with eight.  (24 with four sums of a column's
// tokens instead of eight, see below; of those: 26 and 40 with the registers cut for three or four waves per SIMD, 43 with a wave per
// item and no merge.)  Where there are fewer items than units, eight waves.
#pragma once
#include "attn_mfma.h"

namespace mtp {

template <int G, int HD, int W>
struct AttnRowsLds {
    static constexpr int NC = 16, VS = HD * 2 + 16;
    static constexpr bool VREG = HD == 128;
    struct Tiles {
        alignas(16) uint16_t qs[2][NC][HD + 8];
        alignas(16) unsigned char k[W][16][VS];
        alignas(16) unsigned char v[VREG ? 1 : W][VREG ? 1 : 32][VS];
    };
    struct Merge { // (columns four banks apart)
        alignas(16) float acc[W][NC][HD + 4];
        float ml[kWaves][NC][2];
    };
    union {
        Tiles t;
        Merge m;
    };
};

// W: waves of the workgroup.  Round r of 32 tokens belongs to stream r % 8, as in phase_attn_mfma, whose wave r % 8 has it: with four waves
// each has two streams, in turn.  A context that is one split there gives the same bits here, with four waves as with eight (four
// streams of twice the rounds are another order of the sums: 8e-5 of a prompt's logits, 3e-4 of a training forward's, through
// cache entries that round to the neighbouring bf16 value).
template <int G, int HD, int W>
__device__ __forceinline__ void attn_rows(const DraftParams &p, char *smem) {
    using L = AttnRowsLds<G, HD, W>;
    constexpr int kThreads = W * kWave;
    constexpr int JP = 16 / G, NC = 16, NS = HD / 32, NDB = HD / 16, LPT = HD / 8, TPI = kWave / LPT, NV = 32 / TPI;
    constexpr int PER = kWaves / W; // streams of a wave
    constexpr float kLog2e = 1.4426950408889634f, kLn2 = 0.6931471805599453f;
    const int lane = threadIdx.x & (kWave - 1), i16 = lane & 15, g4 = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x / kWave));
    L &lds = *reinterpret_cast<L *>(smem);
    auto &s = lds.t;
    const int nseq = p.ext_B, mpos = p.B / nseq, JG = (mpos + JP - 1) / JP;
    const int kvh = blockIdx.x % p.Hkv, unit = blockIdx.x / p.Hkv;
    const int b = unit % nseq, jg = JG - 1 - unit / nseq; // the longest first
    int len = 0, lenj[JP]; // tokens the longest position sees, and each (0: not part of the block)
#pragma unroll
    for (int jp = 0; jp < JP; ++jp) lenj[jp] = p.kv_len[min(jg * JP + jp, mpos - 1) * nseq + b];
#pragma unroll
    for (int jp = 0; jp < JP; ++jp) {
        const int L = __builtin_amdgcn_readfirstlane(lenj[jp]);
        lenj[jp] = jg * JP + jp < mpos && L >= 0 && L + p.K <= p.cap ? L + 1 : 0; // (seq_dead)
        len = max(len, lenj[jp]);
    }
    if (len == 0) return;
    const uint16_t *kc = p.k_cache + ((size_t)b * p.Hkv + kvh) * p.cap * HD;
    const uint16_t *vc = p.v_cache + ((size_t)b * p.Hkv + kvh) * p.cap * HD;
    u32x4 kn[2][NS], vr[NV];
    auto load_k = [&](int it) { // past the end: the last row again
#pragma unroll
        for (int tl = 0; tl < 2; ++tl)
#pragma unroll
            for (int u = 0; u < NS; ++u) {
                const int tok = min(it * 32 + tl * 16 + u * TPI + lane / LPT, len - 1);
                kn[tl][u] = ldg16(kc + (size_t)tok * HD + (lane % LPT) * 8);
            }
    };
    auto load_v = [&](int it) {
#pragma unroll
        for (int u = 0; u < NV; ++u) {
            const int tok = min(it * 32 + u * TPI + lane / LPT, len - 1);
            vr[u] = ldg16(vc + (size_t)tok * HD + (lane % LPT) * 8);
        }
    };
    // the query: thread -> elements jj and jj + HD/2 of columns c0 .. c0 + NQ - 1, neighbours so that few positions are turned
    constexpr int CL = kThreads / (HD / 2), NQ = NC / CL;
    const int jj = threadIdx.x % (HD / 2), c0 = threadIdx.x / (HD / 2) * NQ;
    const double inv_freq = p.rope_inv[jj];
    float qa[NQ], qb[NQ];
    uint16_t ba[NQ], bb[NQ];
#pragma unroll
    for (int k = 0; k < NQ; ++k) {
        const int c = c0 + k, hq = kvh * G + c % G;
        const float *src = p.qkv + (size_t)(min(jg * JP + c / G, mpos - 1) * nseq + b) * p.qkv_dim + (size_t)hq * HD;
        qa[k] = src[jj];
        qb[k] = src[jj + HD / 2];
        ba[k] = p.b_q ? p.b_q[hq * HD + jj] : (uint16_t)0;
        bb[k] = p.b_q ? p.b_q[hq * HD + jj + HD / 2] : (uint16_t)0;
    }
    load_k(wave);
    load_v(wave);
    const float scale = 1.0f / sqrtf((float)HD);
    float cs = 1.f, sn = 0.f;
#pragma unroll
    for (int k = 0; k < NQ; ++k) {
        const int c = c0 + k;
        if (k % (G < NQ ? G : NQ) == 0) {
            int pos = 0;
#pragma unroll
            for (int u = 0; u < JP; ++u) pos = u == c / G ? max(lenj[u] - 1, 0) : pos;
            rope_cos_sin(pos, inv_freq, cs, sn);
        }
        const float a = qa[k] + bf16_to_f32(ba[k]), e = qb[k] + bf16_to_f32(bb[k]);
        split_bf16(rope_lower(a, e, cs, sn) * scale * kLog2e, s.qs[0][c][jj], s.qs[1][c][jj]);
        split_bf16(rope_upper(a, e, cs, sn) * scale * kLog2e, s.qs[0][c][jj + HD / 2], s.qs[1][c][jj + HD / 2]);
    }
    lds_barrier();
    u32x4 qh[NS], ql[NS];
#pragma unroll
    for (int u = 0; u < NS; ++u) {
        const int at = g4 * (HD / 4) + u * 8;
        qh[u] = *reinterpret_cast<const u32x4 *>(&s.qs[0][i16][at]);
        ql[u] = *reinterpret_cast<const u32x4 *>(&s.qs[1][i16][at]);
    }
    int lim = 0; // tokens this lane's column sees
#pragma unroll
    for (int u = 0; u < JP; ++u) lim = u == i16 / G ? lenj[u] : lim;
    float mx[PER], lsum[PER];
    f32x4 oacc[PER][NDB];
#pragma unroll
    for (int v = 0; v < PER; ++v) {
        mx[v] = -INFINITY;
        lsum[v] = 0.f;
#pragma unroll
        for (int db = 0; db < NDB; ++db) oacc[v][db] = f32x4{0.f, 0.f, 0.f, 0.f};
    }
    unsigned char *vrow = &s.v[L::VREG ? 0 : wave][0][0], *krow = &s.k[wave][0][0];
    const int niter = (len + 31) / 32;
    for (int it = wave; it < niter;) {
#pragma unroll
        for (int v = 0; v < PER; ++v) {
            attn_round<HD>(it * 32, lim, krow, vrow, kn, vr, qh, ql, [&] { load_k(it + W); }, [&] { load_v(it + W); }, mx[v], lsum[v],
                           oacc[v]);
            it += W;
            if (it >= niter) break;
        }
    }
    // The streams' results meet in the place of the tiles, one of every wave at a time, in order.  Thread -> E neighbouring
    // dimensions of column c
    constexpr int E = NC * HD / kThreads;
    static_assert(E == 8 || E == 4 || E == 2, "pieces of a column");
    const int c = threadIdx.x / (HD / E), e0 = threadIdx.x % (HD / E) * E;
    int mine = 0;
#pragma unroll
    for (int u = 0; u < JP; ++u) mine = u == c / G ? lenj[u] : mine;
    float M = -INFINITY, ls = 0.f, r[E];
#pragma unroll
    for (int i = 0; i < E; ++i) r[i] = 0.f;
#pragma unroll
    for (int v = 0; v < PER; ++v) {
        lds_barrier();
#pragma unroll
        for (int db = 0; db < NDB; db += L::VREG ? 4 : 1) // four neighbouring dimensions at a time
#pragma unroll
            for (int e = 0; e < (L::VREG ? 4 : 1); ++e) {
                const f32x4 o = L::VREG ? f32x4{oacc[v][db][e], oacc[v][L::VREG ? db + 1 : 0][e], oacc[v][L::VREG ? db + 2 : 0][e],
                                                oacc[v][L::VREG ? db + 3 : 0][e]}
                                        : oacc[v][db];
                *reinterpret_cast<f32x4 *>(&lds.m.acc[wave][i16][L::VREG ? 8 * (4 * g4 + e) + db : db * 16 + g4 * 4]) = o;
            }
        if (v == 0)
#pragma unroll
            for (int u = 0; u < PER; ++u) {
                const float l = rows_sum(lsum[u]);
                if (g4 == 0) {
                    lds.m.ml[u * W + wave][i16][0] = mx[u] * kLn2;
                    lds.m.ml[u * W + wave][i16][1] = l;
                }
            }
        lds_barrier();
        if (v == 0)
#pragma unroll
            for (int w = 0; w < kWaves; ++w) M = fmaxf(M, lds.m.ml[w][c][0]);
#pragma unroll
        for (int w = 0; w < W; ++w) {
            const float mm = lds.m.ml[v * W + w][c][0];
            const bool seen = mm != -INFINITY; // (a stream without a token of the column adds nothing, whatever it holds)
            const float f = seen ? exp_weight(mm - M) : 0.f;
            ls += lds.m.ml[v * W + w][c][1] * f;
#pragma unroll
            for (int i = 0; i < E; ++i) r[i] += (seen ? lds.m.acc[w][c][e0 + i] : 0.f) * f;
        }
    }
    if (mine == 0) return; // not part of the block
    uint32_t h[E / 2], l[E / 2];
#pragma unroll
    for (int i = 0; i < E / 2; ++i) split_bf16x2(r[2 * i] / ls, r[2 * i + 1] / ls, h[i], l[i]);
    uint16_t *dst = p.attn_split + act_index(p, (jg * JP + c / G) * nseq + b, (kvh * G + c % G) * HD + e0);
    if constexpr (E == 8) {
        *reinterpret_cast<u32x4 *>(dst) = u32x4{h[0], h[1], h[2], h[3]};
        *reinterpret_cast<u32x4 *>(dst + p.a_lo) = u32x4{l[0], l[1], l[2], l[3]};
    } else if constexpr (E == 4) {
        *reinterpret_cast<u32x2 *>(dst) = u32x2{h[0], h[1]};
        *reinterpret_cast<u32x2 *>(dst + p.a_lo) = u32x2{l[0], l[1]};
    } else {
        *reinterpret_cast<uint32_t *>(dst) = h[0];
        *reinterpret_cast<uint32_t *>(dst + p.a_lo) = l[0];
    }
}

} // namespace mtp
