// Single-launch path for ONE sequence without grid barriers (gfx950): all phases of all K draft steps in one
// kernel (one workgroup per compute unit, all resident; narrow heads: a quarter of them, see flow_admit) whose workgroups hand their results over element by element.
//
// A draft step at batch 1 is a chain of dependent matrix-vector products (Sec. 2.1) of 30-270 MB each; between two of
// them every workgroup needs the whole result vector of the phase before.  With a grid barrier that hand-over is a
// chain of its own (acknowledge the stores, arrive, count, release, poll, then load the vector: six to nine
// microseconds at 1-2 us per trip while HBM is busy) during which the weight stream runs dry.  Here
//  * every element of a vector that crosses between phases is a 64-bit word holding the float and a tag that names the
//    (call, step, phase) that produced it (device-coherent 8-byte accesses are single-copy atomic).  The consumer
//    polls the elements it needs until they carry the tag it expects: one store and one load separate the last
//    producer from the first consumer, and nobody counts arrivals;
//  * a wave's register ring of weight chunks is not drained at the end of a phase: the slots freed by the last chunks
//    of a phase are refilled with the first chunks of the NEXT phase (weights do not depend on activations), so the
//    memory system keeps streaming while results are handed over and staged;
//  * the projection is split into its hidden-state half and its embedding half (W_p c = W_p[:, :d] c_h + W_p[:, d:] c_e):
//    the hidden-state half needs no result of another workgroup (every workgroup normalises the step's output hidden
//    state itself), so it runs while the output head's argmax candidates travel;
//  * SiLU(gate) * up is formed by the wave that computed both rows, which halves what the down projection polls.
// Why a consumer can never see a tag NEWER than the one it waits for: a workgroup stores results of phase P+1 only
// after it has seen every result of phase P, i.e. after every workgroup has finished computing P and therefore
// finished reading the results of P-1; a vector is rewritten one whole step after it was read.
#pragma once
#include "phases.h"

namespace mtp {

// parts the query heads of a KV head are dealt to in the attention of the single-launch kernel (phase_attn, GS)
template <int G>
constexpr int kFlowAttnParts = G >= 2 ? 2 : 1;

// time stamps of every workgroup (mtp_set_phase_trace): [step][section][point][workgroup]
constexpr int kTraceSections = 8; // projection (embedding half), q/k/v, attention, output projection, gate/up, down,
                                  // output head, projection (hidden-state half)
constexpr int kTracePoints = 4;
enum : int { kTraceRequested = 0, kTraceReleased, kTraceStaged, kTraceDone };

// LDS region shared by the staged activations of every matrix phase (one sequence): bf16 hi then lo halves, each padded
// with zeros to whole 512-element blocks (a row's last block is multiplied in full: the weights beyond the row read as
// zeros, so what stands beside them only has to be finite)
__host__ __device__ inline int flow_kpad(int K) { return (K + 511) / 512 * 512; }
__host__ __device__ inline size_t flow_gemv_region(int d, int qd, int F) {
    int m = flow_kpad(d);
    m = flow_kpad(qd) > m ? flow_kpad(qd) : m;
    m = flow_kpad(F) > m ? flow_kpad(F) : m;
    return ((size_t)m * 4 + 255) / 256 * 256;
}

enum FlowPhase : int { FL_PROJH = 0, FL_PROJE, FL_QKV, FL_O, FL_GATEUP, FL_DOWN, FL_HEAD, FL_NONE };

// One matrix phase as a list of rows: up to three matrices stacked row-wise, wave w takes the virtual rows w, w + nw, ...
// Gate and up: the rows of [w_gate; w_up] dealt so that a wave gets row q of both, one after the other (its j-th row is gate or
// up row (j / 2) * nw + w for j < 2 * pair_rounds; the rem = F % nw rows of each matrix that are left over are dealt singly:
// rem gate rows, then rem up rows, numbered on from the pairs - 2 rem may exceed nw, the waves then get a second
// round of them).  Virtual row v = w + j * nw, as in every other phase.
// A wave's share comes in chunks of CL 1 KiB loads (eight, or four or two where rows are shorter: a half-empty chunk requests,
// reads and multiplies zeros); a chunk never straddles rows; the chunk count is padded to an odd number of at least three (a
// phase's first three chunks sit in register slot 0, register slot 1 and the LDS slot, the rest alternate between the register
// slots).
//
// All of it stands in three registers for the whole call: lane 8 * phase + field.  A field is one instruction away, where
// forming it anew (a division, a choice between the phases and loads of the arguments, twice per phase) stood in every phase's
// chain, and keeping it in scalar registers pushed others out into vector lanes.  K = 3, one sequence, d = 256: 121 -> 108 us, d = 4096:
// 386 -> 384 (its chains hide behind the weights on their way).
struct FlowTab {
    int num, ptr, io;
};
enum FlowNum : int { FN_K = 0, FN_PITCH, FN_ROWS, FN_NREAL, FN_CPR, FN_LAST, FN_A, FN_B }; // LAST: the wave's last row;
                                                         // A, B: first rows of w_k, w_v; pair_rounds, rem of gate and up
enum FlowPtr : int { FP_MAT = 0, FP_IDS = 6 };           // up to three matrices; the row list of the output head
enum FlowIo : int { FI_GAIN = 0, FI_OUT = 2, FI_IN = 4 }; // gains of the phase's norm, vector it writes, vector it polls
__device__ __forceinline__ int flow_num(const FlowTab &t, int ph, int f) { return __builtin_amdgcn_readlane(t.num, ph * 8 + f); }
__device__ __forceinline__ unsigned long long flow_word2(int v, int ph, int f) {
    return ((unsigned long long)(unsigned)__builtin_amdgcn_readlane(v, ph * 8 + f + 1) << 32) |
           (unsigned)__builtin_amdgcn_readlane(v, ph * 8 + f);
}
template <class T>
__device__ __forceinline__ T *flow_ptr(int v, int ph, int f) { return reinterpret_cast<T *>(flow_word2(v, ph, f)); }

template <int CL>
__device__ __forceinline__ int flow_chunks(int K) { return ((K + 511) / 512 + CL - 1) / CL; } // of a row
__device__ __forceinline__ int flow_rows(int rows, int wr0, int nw) { return wr0 < rows ? (rows - wr0 + nw - 1) / nw : 0; }
template <int CL>
__device__ __forceinline__ FlowTab flow_tab(const DraftParams &p, int wr0, int nw) {
    const int lane = threadIdx.x & (kWave - 1), ph = lane >> 3, f = lane & 7; // (FL_NONE: no rows)
    const int K = ph == FL_O ? p.qd : ph == FL_DOWN ? p.F : p.d;
    const int rows = ph == FL_QKV ? p.qkv_dim : ph == FL_GATEUP ? 2 * p.F : ph == FL_HEAD ? p.n : ph == FL_NONE ? 0 : p.d;
    const int pitch = ph <= FL_PROJE ? 2 * p.d : K;
    const int cpr = flow_chunks<CL>(K), nrows = flow_rows(rows, wr0, nw);
    const int rounds = p.F / nw;
    FlowTab t;
    t.num = f == FN_K ? K : f == FN_PITCH ? pitch : f == FN_ROWS ? rows : f == FN_NREAL ? nrows * cpr : f == FN_CPR ? cpr
            : f == FN_LAST ? wr0 + max(nrows - 1, 0) * nw
            : f == FN_A ? (ph == FL_QKV ? p.qd : rounds) : (ph == FL_QKV ? p.qd + p.kvd : p.F - rounds * nw);
    const void *m = nullptr, *v = nullptr;
    const int mat = f >> 1;
    if (mat == 0)
        m = ph == FL_PROJH ? p.w_proj : ph == FL_PROJE ? p.w_proj + p.d : ph == FL_QKV ? p.w_q : ph == FL_O ? p.w_o
            : ph == FL_GATEUP ? p.w_gate : ph == FL_DOWN ? p.w_down : p.lm_head;
    if (mat == 1) m = ph == FL_QKV ? p.w_k : p.w_up;
    if (mat == 2) m = p.w_v;
    if (mat == 3 && ph == FL_HEAD) m = p.ids;
    if (mat == 0)
        v = ph == FL_PROJH ? p.g_h : ph == FL_PROJE ? p.g_e : ph == FL_QKV ? p.g_attn : ph == FL_GATEUP ? p.g_mlp : p.g_final;
    if (mat == 1)
        v = ph == FL_PROJE ? p.xt : ph == FL_QKV ? p.qkvt : ph == FL_O ? p.ot : ph == FL_GATEUP ? p.gut : p.dnt;
    if (mat == 2)
        v = ph == FL_QKV ? p.xt : ph == FL_O ? p.attnt : ph == FL_GATEUP ? p.ot : ph == FL_DOWN ? p.gut : p.dnt;
    const unsigned long long mw = reinterpret_cast<unsigned long long>(m), vw = reinterpret_cast<unsigned long long>(v);
    t.ptr = (int)(f & 1 ? mw >> 32 : mw);
    t.io = (int)(f & 1 ? vw >> 32 : vw);
    return t;
}

// load cursor of a wave: which phase it is requesting chunks of, and where in the wave's share it stands
struct FlowLoad {
    int id;            // FlowPhase the cursor is in
    const uint16_t *base;           // its first matrix
    int K, pitch, nreal, cpr, last;
    int row, jr, c, n; // next chunk: virtual row, its round, chunk within the row, chunks requested so far
    int rid;           // id-list entry of `row` (requested when the cursor moved there, used at the next request)
};
// The id list is read-only during the call and row indices are wave-uniform: a scalar load (a vector load would make
// the wave wait for every weight chunk in flight before it can form the row's address).
__device__ __forceinline__ int flow_row_id(const FlowTab &t, int id, int v) {
    typedef const int __attribute__((address_space(4))) *const_int_ptr;
    if (id != FL_HEAD) return 0;
    const int *ids = flow_ptr<const int>(t.ptr, FL_HEAD, FP_IDS);
    return ids ? *((const_int_ptr)(ids + min(v, flow_num(t, FL_HEAD, FN_ROWS) - 1))) : v;
}
__device__ __forceinline__ void flow_load_begin(FlowLoad &L, const FlowTab &t, int id, int wr0) {
    L.id = id;
    L.base = flow_ptr<const uint16_t>(t.ptr, id, FP_MAT);
    L.K = flow_num(t, id, FN_K);
    L.pitch = flow_num(t, id, FN_PITCH);
    L.nreal = flow_num(t, id, FN_NREAL);
    L.cpr = flow_num(t, id, FN_CPR);
    L.last = flow_num(t, id, FN_LAST);
    L.row = wr0;
    L.jr = 0;
    L.c = 0;
    L.n = 0;
    L.rid = flow_row_id(t, id, wr0);
}
// the row the cursor stands in (past the wave's last chunk a zero-length buffer), then the cursor moves on by a chunk; voff: the
// lane's offset of the chunk in the row
template <int CL>
__device__ __forceinline__ row_rsrc flow_next(FlowLoad &L, const FlowTab &t, int nw, int lane, int &voff) {
    const bool live = L.n < L.nreal;
    int v = min(L.row, L.last), mat = 0;
    if (L.id == FL_GATEUP) {
        const int pairs = flow_num(t, FL_GATEUP, FN_A), rem = flow_num(t, FL_GATEUP, FN_B);
        if (L.jr < 2 * pairs) {
            mat = L.jr & 1;
            v = (L.jr >> 1) * nw + v - L.jr * nw;
        } else {
            const int i = v - 2 * pairs * nw; // 0 .. 2 rem - 1
            mat = i < rem ? 0 : 1;
            v = pairs * nw + (i < rem ? i : i - rem);
        }
    } else if (L.id == FL_QKV) {
        const int k0 = flow_num(t, FL_QKV, FN_A), v0 = flow_num(t, FL_QKV, FN_B);
        mat = v < k0 ? 0 : v < v0 ? 1 : 2;
        v -= v < k0 ? 0 : v < v0 ? k0 : v0;
    } else if (L.id == FL_HEAD) {
        v = L.rid;
    }
    const uint16_t *base = L.base;
    if (mat != 0) base = flow_ptr<const uint16_t>(t.ptr, L.id, FP_MAT + 2 * mat);
    const uint16_t *row = base + (size_t)(live ? v : 0) * L.pitch;
    const row_rsrc rs = make_row_rsrc(row, live ? L.K * 2 : 0); // wave-uniform
    // The block's offset travels in the per-lane offset, which the buffer's range check covers: whatever lies beyond the
    // row (the tail of its last block, the empty slots of its last chunk) reads as zeros and moves no data.
    voff = lane * 16 + L.c * (CL * 1024);
    ++L.n;
    if (++L.c == L.cpr) {
        L.c = 0;
        L.row += nw;
        ++L.jr;
        L.rid = flow_row_id(t, L.id, L.row);
    }
    return rs;
}
// Request the cursor's next chunk into a ring slot.  Past the wave's last chunk (padding, or no next phase) the
// request goes to a zero-length buffer: it returns zeros and moves no data, so the ring is refilled without a branch
// around any load and the compiler can count the loads in flight.
template <int CL>
__device__ __forceinline__ void flow_issue(FlowLoad &L, const FlowTab &t, int nw, u32x4 (&buf)[CL], int lane) {
    int voff;
    const row_rsrc rs = flow_next<CL>(L, t, nw, lane, voff);
#pragma unroll
    for (int u = 0; u < CL; ++u) buf[u] = row_load16<true>(rs, voff + u * 1024, 0);
}

// The same request into the wave's LDS slot (8 KiB: up to eight loads of 1 KiB, each lane's 16 bytes where a register load
// would have put them).  The compiler counts these loads like the others but does not wait for them before LDS reads:
// the reader does (flow_wait_lds_slot).
constexpr int kLdsSlotBytes = kChunkLoads * 1024;
template <int CL>
__device__ __forceinline__ void flow_issue_lds(FlowLoad &L, const FlowTab &t, int nw, char *slot, int lane) {
    int voff;
    const row_rsrc rs = flow_next<CL>(L, t, nw, lane, voff);
#pragma unroll
    for (int u = 0; u < CL; ++u)
        __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, (__attribute__((address_space(3))) void *)(slot + u * 1024), 16,
                                                 voff + u * 1024, 0, 0, 2);
}
// Every load that the wave has asked for has landed, the LDS slot's chunk among them.  (Not just all but the two register chunks that are
// requested behind it: a phase of three chunks puts those off until its end, and the slot's is the last there is.  The compiler waits
// like this before every pass of the loop over the chunks as it is, but for the registers' sake: it does not know of the slot.)
__device__ __forceinline__ void flow_wait_loads() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }

// ---- polling -----------------------------------------------------------------------------------------------
// This thread's elements e = (it * kBlock + tid) * 4 .. + 3 < n of a tagged vector (n a multiple of 4), polled until
// all of them carry `tag`.  NIT * kBlock * 4 >= n.
// A phase is a chain of instructions and round trips, and this is a link of every one.  The wave looks, and leaves, as one:
// a loop that lanes leave one by one, with a branch for each condition, keeps a lane mask for each and took about 100 scalar
// instructions a look (and, where the compiler no longer knew the address to be the wave's, a loop around every load).  Reading
// less again of what had arrived, and pausing between looks, change nothing.  K = 3 at d = 4096, one sequence: 401 -> 393 us,
// d = 256: 129 -> 124 us.
template <int NIT>
__device__ __forceinline__ void poll_vec(const DraftParams &p, const unsigned long long *src, int n, unsigned tag,
                                         float (&v)[NIT][4]) {
    const row_rsrc rs = make_vec_rsrc(src, (size_t)n * 8);
    u32x4 w[NIT][2];
    PollClock clk;
    bool late;
    do {
        unsigned off = 0u; // bits by which a tag differs from the wanted one
#pragma unroll
        for (int it = 0; it < NIT; ++it) {
            const int e = (it * kBlock + (int)threadIdx.x) * 4;
            w[it][0] = ld_coherent16(rs, e * 8); // beyond n: zeros, not checked
            w[it][1] = ld_coherent16(rs, e * 8 + 16);
        }
#pragma unroll
        for (int it = 0; it < NIT; ++it) {
            const int e = (it * kBlock + (int)threadIdx.x) * 4;
            const unsigned o = (w[it][0].y ^ tag) | (w[it][0].w ^ tag) | (w[it][1].y ^ tag) | (w[it][1].w ^ tag);
            off |= e < n ? o : 0u;
        }
        late = __any((int)off) != 0;
    } while (late && !clk.expired(p));
#pragma unroll
    for (int it = 0; it < NIT; ++it) {
        v[it][0] = __uint_as_float(w[it][0].x);
        v[it][1] = __uint_as_float(w[it][0].z);
        v[it][2] = __uint_as_float(w[it][1].x);
        v[it][3] = __uint_as_float(w[it][1].z);
    }
}

// four consecutive tagged elements at each of two places, polled together
__device__ __forceinline__ void poll4x2(const DraftParams &p, row_rsrc rs, int a_byte, int b_byte, unsigned tag,
                                        float (&va)[4], float (&vb)[4]) {
    PollClock clk;
    for (;;) {
        const u32x4 a0 = ld_coherent16(rs, a_byte), a1 = ld_coherent16(rs, a_byte + 16), b0 = ld_coherent16(rs, b_byte),
                    b1 = ld_coherent16(rs, b_byte + 16);
        va[0] = __uint_as_float(a0.x);
        va[1] = __uint_as_float(a0.z);
        va[2] = __uint_as_float(a1.x);
        va[3] = __uint_as_float(a1.z);
        vb[0] = __uint_as_float(b0.x);
        vb[1] = __uint_as_float(b0.z);
        vb[2] = __uint_as_float(b1.x);
        vb[3] = __uint_as_float(b1.z);
        const unsigned off = (a0.y ^ tag) | (a0.w ^ tag) | (a1.y ^ tag) | (a1.w ^ tag) | (b0.y ^ tag) | (b0.w ^ tag) |
                             (b1.y ^ tag) | (b1.w ^ tag);
        if (__any((int)off) == 0 || clk.expired(p)) break;
    }
}

// Workgroup barrier of this kernel: the wave's own LDS reads and writes have completed, nothing else is waited for.
// (A fence on LDS would also wait for the chunk that is on its way INTO the LDS slot, i.e. for every load in flight.)
__device__ __forceinline__ void flow_barrier() {
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
}

// workgroup sum whose barriers order LDS traffic only (weight chunks stay in flight); red holds kWaves floats
__device__ __forceinline__ float block_sum_lds(float x, float *red) {
    x = wave_sum(x);
    flow_barrier();
    if ((threadIdx.x & (kWave - 1)) == 0) red[threadIdx.x / kWave] = x;
    flow_barrier();
    float t = 0.f;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) t += red[w];
    return t;
}
__device__ __forceinline__ unsigned long long block_max_u64_lds(unsigned long long v, unsigned long long *red64) {
    v = wave_max_u64(v);
    flow_barrier();
    if ((threadIdx.x & (kWave - 1)) == 0) red64[threadIdx.x / kWave] = v;
    flow_barrier();
    unsigned long long r = 0ull;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) r = red64[w] > r ? red64[w] : r;
    return r;
}

// RMSNorm(u; gain) of the values this thread holds (v[it][q] = element (it * kBlock + tid) * 4 + q of a d-vector, gq[it]
// the four bf16 gains of the same elements) into hi/lo.  keep_raw (LDS, optional) receives u itself, keep_norm (LDS, optional) and out_global (optional) the result.
__device__ __forceinline__ void flow_norm(float (&v)[kMaxNormIter][4], const u32x2 (&gq)[kMaxNormIter], int d, int kpad, float eps,
                                          uint16_t *hi, uint16_t *lo, float *red, float *keep_raw, float *keep_norm,
                                          float *out_global) {
    float ss = 0.f;
#pragma unroll
    for (int it = 0; it < kMaxNormIter; ++it) {
        const int e = (it * kBlock + (int)threadIdx.x) * 4;
        if (e < d) {
#pragma unroll
            for (int q = 0; q < 4; ++q) ss += v[it][q] * v[it][q];
            if (keep_raw) *reinterpret_cast<f32x4 *>(keep_raw + e) = f32x4{v[it][0], v[it][1], v[it][2], v[it][3]};
        }
    }
    const float tot = block_sum_lds(ss, red);
    const float inv = 1.0f / sqrtf(tot / (float)d + eps);
#pragma unroll
    for (int it = 0; it < kMaxNormIter; ++it) {
        const int e = (it * kBlock + (int)threadIdx.x) * 4;
        if (e < d) {
            const u32x2 g = gq[it];
            float o[4];
            o[0] = lo_half(g.x) * (v[it][0] * inv);
            o[1] = hi_half(g.x) * (v[it][1] * inv);
            o[2] = lo_half(g.y) * (v[it][2] * inv);
            o[3] = hi_half(g.y) * (v[it][3] * inv);
            u32x2 h, l;
            split_bf16x4(o, h, l);
            *reinterpret_cast<u32x2 *>(hi + e) = h;
            *reinterpret_cast<u32x2 *>(lo + e) = l;
            const f32x4 w = {o[0], o[1], o[2], o[3]};
            if (keep_norm) *reinterpret_cast<f32x4 *>(keep_norm + e) = w;
            if (out_global) *reinterpret_cast<f32x4 *>(out_global + e) = w;
        } else if (e < kpad) { // the tail of the last 512-element block
            *reinterpret_cast<u32x2 *>(hi + e) = u32x2{0u, 0u};
            *reinterpret_cast<u32x2 *>(lo + e) = u32x2{0u, 0u};
        }
    }
}

// four floats of this thread -> hi/lo at element e
__device__ __forceinline__ void flow_split4(const float (&m)[4], uint16_t *hi, uint16_t *lo, int e) {
    u32x2 h, l;
    split_bf16x4(m, h, l);
    *reinterpret_cast<u32x2 *>(hi + e) = h;
    *reinterpret_cast<u32x2 *>(lo + e) = l;
}

__device__ __forceinline__ float silu_mul(float g, float u) { return (g / (1.0f + expf(-g))) * u; }

// LDS of the kernel: [activations hi/lo of the widest phase | attention scratch] then the residual stream (d floats),
// the wave-private strips of the projection's first half, and reduction scratch
__host__ __device__ inline size_t flow_part_floats(int d, int nvb) { return (size_t)kWaves * ((d + nvb * kWaves - 1) / (nvb * kWaves)) + 8; }
// bytes behind the shared region: the waves' LDS chunk slots, the residual stream, the projection's strips, scratch
__host__ __device__ inline size_t flow_tail_bytes(int d, int nvb) {
    return (size_t)kWaves * kLdsSlotBytes + ((size_t)d + flow_part_floats(d, nvb)) * 4 + 256;
}

// ---------------------------------------------------------------------------------------------------
// Whether the launch's workgroups may wait for one another (p.admit set: heads that do not take every compute unit, whose calls
// may overlap other kernels).  Workgroups that wait hold their compute units; two launches that each have part of the units
// would wait for good.  So every workgroup first counts itself in and waits until all are there: from then on nothing that they
// wait for depends on another launch.  If that takes too long, ONE workgroup (the one whose flag gets in) does the whole call
// by itself, as a launch of one workgroup would, and the others leave: no wait depends on more than one resident workgroup.
// One 64-bit word decides, so that all of them decide alike: arrivals in its upper half, which only grow - every workgroup of
// every call arrives exactly once, and a call's place in them follows from what an arrival finds, whoever has called before -
// and below the mark of the call that one workgroup does alone.  (Nothing has to be cleared or counted on the host.)
// admit_ticks: the longest wait (100 MHz), 0: never all of them (the first to arrive does the call).
// ---------------------------------------------------------------------------------------------------
enum : int { kAdmitLeave = 0, kAdmitAll = 1, kAdmitOne = 2 };
__device__ __forceinline__ int flow_admit(const DraftParams &p, int *flag) {
    if (threadIdx.x == 0) {
        const long long t0 = wall_clock64(), limit = p.admit_ticks != 0 ? p.admit_ticks : p.bar_timeout;
        const unsigned all = gridDim.x;
        unsigned long long w = __hip_atomic_fetch_add(p.admit, 1ull << 32, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        const unsigned before = (unsigned)(w >> 32), place = before % all, first = before - place, mark = first + 1u;
        w += 1ull << 32; // (as it was right after this arrival)
        auto put_mark = [&](unsigned m) { // false: w is now what others have made of the word
            return __hip_atomic_compare_exchange_strong(p.admit, &w, (w & 0xffffffff00000000ull) | m, __ATOMIC_RELAXED,
                                                        __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        };
        int state = -1;
        while (state < 0) {
            const bool late = (p.admit_ticks == 0 && place == 0u) || wall_clock64() - t0 > limit;
            if ((unsigned)w == mark) {
                state = kAdmitLeave;
            } else if (p.admit_ticks != 0 && (unsigned)(w >> 32) - first == all) {
                // (a mark of an earlier call is taken away, long before its number could come round again)
                if ((unsigned)w == 0u || place != all - 1u || put_mark(0u)) state = kAdmitAll;
            } else if (late) {
                if (put_mark(mark)) state = kAdmitOne;
            } else {
                w = __hip_atomic_load(p.admit, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
        }
        *flag = state;
    }
    __syncthreads();
    const int state = __builtin_amdgcn_readfirstlane(*flag);
    __syncthreads(); // the flag's place is used for other things from here on
    return state;
}

// ---------------------------------------------------------------------------------------------------
// the kernel body, workgroup vb of nvb
// ---------------------------------------------------------------------------------------------------
template <int G, int HD, int CL>
__device__ __forceinline__ void flow_steps(const DraftParams &p, char *smem, int vb, int nvb) {
    const int d = p.d, F = p.F;
    const int lane = threadIdx.x & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x / kWave));
    const int nw = nvb * kWaves, wr0 = vb * kWaves + wave;
    char *slot = smem + p.fused_gemv_bytes + (size_t)wave * kLdsSlotBytes; // this wave's third chunk slot
    float *resid = reinterpret_cast<float *>(smem + p.fused_gemv_bytes + (size_t)kWaves * kLdsSlotBytes); // x, x1 = x + o,
                                                                           // then the step's output state
    const int part_rows = (d + nw - 1) / nw;                             // rows of the projection per wave
    float *ppart = resid + d + (size_t)wave * part_rows;                 // this wave's first-half sums
    unsigned long long *red64 = reinterpret_cast<unsigned long long *>(resid + d + flow_part_floats(d, nvb));
    float *red = reinterpret_cast<float *>(red64 + kWaves);

    auto stamp = [&](int step, int sec, int pt) {
        if (p.trace && threadIdx.x == 0)
            p.trace[(((size_t)step * kTraceSections + sec) * kTracePoints + pt) * p.trace_wgs + vb] = wall_clock64();
    };
    if (vb == 0 && threadIdx.x == 0 && seq_dead(p, 0)) atomicOr(p.err, kErrKvOverflow);

    // winner of the output head of `step`: maximum over the workgroups' candidates, as a token id (all threads; barriers)
    auto winner = [&](int step) {
        const unsigned tag = step_tag(p, step, TS_CAND);
        const row_rsrc rs = make_vec_rsrc(p.candt + (size_t)step * p.head_grid * 2, (size_t)nvb * 16);
        unsigned long long best = 0ull;
        for (int w = threadIdx.x; w < nvb; w += kBlock) {
            u32x4 c;
            PollClock clk;
            bool late;
            do {
                c = ld_coherent16(rs, w * 16);
                late = __any((int)((c.y ^ tag) | (c.w ^ tag))) != 0;
            } while (late && !clk.expired(p));
            const unsigned long long key = ((unsigned long long)c.x << 32) | (unsigned long long)(0xffffffffu - c.z);
            best = key > best ? key : best;
        }
        best = block_max_u64_lds(best, red64);
        unsigned id = 0xffffffffu - (unsigned)best;
        if (id >= (unsigned)p.V) id = 0; // no workgroup had a candidate (cannot happen with n >= 1), or the wait gave up
        return (int)id;
    };

    u32x4 ring[2][CL];
    // The call's first requests go out before the table is formed, which waits for all of the arguments.
    FlowTab tab = {0, 0, 0};
    FlowLoad L;
    L.id = FL_PROJH;
    L.base = p.w_proj;
    L.K = d;
    L.pitch = 2 * d;
    L.cpr = flow_chunks<CL>(d);
    L.nreal = flow_rows(d, wr0, nw) * L.cpr;
    L.last = wr0 + max(flow_rows(d, wr0, nw) - 1, 0) * nw;
    L.row = wr0;
    L.jr = L.c = L.n = L.rid = 0;
    flow_issue(L, tab, nw, ring[0], lane);
    flow_issue(L, tab, nw, ring[1], lane);
    flow_issue_lds<CL>(L, tab, nw, slot, lane);
    tab = flow_tab<CL>(p, wr0, nw);
    bool slot_late = false; // the LDS slot's chunk of the phase that begins has not been requested yet

    for (int step = 0; step < p.K; ++step) {
#pragma unroll 1
        for (int ph = FL_PROJH; ph <= FL_HEAD; ++ph) {
            const int K = flow_num(tab, ph, FN_K), nblk = (K + 511) / 512, kpad = nblk * 512;
            const int nreal = flow_num(tab, ph, FN_NREAL), cpr = flow_num(tab, ph, FN_CPR), nchunks = max(3, nreal | 1);
            uint16_t *act_hi = reinterpret_cast<uint16_t *>(smem), *act_lo = act_hi + kpad;
            const int sec = ph == FL_PROJH ? 7 : ph == FL_PROJE ? 0 : ph == FL_QKV ? 1 : ph + 0; // O..HEAD are 3..6
            stamp(step, sec, kTraceRequested);
            flow_barrier(); // every wave has finished with the activations of the phase before

            // ---- stage this phase's input vector into LDS as bf16 hi + lo ------------------------------------------
            {
                float v[kMaxNormIter][4];
                // The gains of this phase's norm are requested before anything is polled: they do not depend on it, and a
                // load issued after the poll would add its own trip through the (busy) memory system to the hand-over.
                const uint16_t *gain = flow_ptr<const uint16_t>(tab.io, ph, FI_GAIN);
                u32x2 gq[kMaxNormIter];
#pragma unroll
                for (int it = 0; it < kMaxNormIter; ++it) {
                    const int e = (it * kBlock + (int)threadIdx.x) * 4;
                    gq[it] = (e < d && ph != FL_O && ph != FL_DOWN) ? *reinterpret_cast<const u32x2 *>(gain + e) : u32x2{0u, 0u};
                }
                switch (ph) {
                case FL_PROJH: {
                    if (step == 0) {
#pragma unroll
                        for (int it = 0; it < kMaxNormIter; ++it) {
                            const int e = (it * kBlock + (int)threadIdx.x) * 4;
                            if (e < d) {
                                if (!p.own_hidden) {
                                    const u32x2 raw = *reinterpret_cast<const u32x2 *>(p.hidden_in + e);
                                    v[it][0] = lo_half(raw.x);
                                    v[it][1] = hi_half(raw.x);
                                    v[it][2] = lo_half(raw.y);
                                    v[it][3] = hi_half(raw.y);
                                } else {
                                    const f32x4 raw = *reinterpret_cast<const f32x4 *>(p.hhat + e);
                                    v[it][0] = raw.x;
                                    v[it][1] = raw.y;
                                    v[it][2] = raw.z;
                                    v[it][3] = raw.w;
                                }
                            }
                        }
                    } else { // the head's own output of the step before: every workgroup kept it
#pragma unroll
                        for (int it = 0; it < kMaxNormIter; ++it) {
                            const int e = (it * kBlock + (int)threadIdx.x) * 4;
                            if (e < d) {
                                const f32x4 raw = *reinterpret_cast<const f32x4 *>(resid + e);
                                v[it][0] = raw.x;
                                v[it][1] = raw.y;
                                v[it][2] = raw.z;
                                v[it][3] = raw.w;
                            }
                        }
                    }
                    stamp(step, sec, kTraceReleased);
                    flow_norm(v, gq, d, kpad, p.eps, act_hi, act_lo, red, nullptr, nullptr, nullptr);
                    break;
                }
                case FL_PROJE: {
                    int tok;
                    if (step == 0) {
                        tok = p.token_in[0];
                    } else {
                        const int did = winner(step - 1);
                        tok = p.forced ? p.forced[step - 1] : did;
                        if (vb == 0 && threadIdx.x == 0) p.draft_out[step - 1] = seq_dead(p, 0) ? -1 : did;
                    }
                    if (tok < 0 || tok >= p.V) { // reported, and replaced by id 0 so that every access stays in bounds
                        if (threadIdx.x == 0) atomicOr(p.err, kErrTokenRange);
                        tok = 0;
                    }
                    stamp(step, sec, kTraceReleased);
                    const uint16_t *src = p.embed + (size_t)tok * d;
#pragma unroll
                    for (int it = 0; it < kMaxNormIter; ++it) {
                        const int e = (it * kBlock + (int)threadIdx.x) * 4;
                        if (e < d) {
                            const u32x2 raw = *reinterpret_cast<const u32x2 *>(src + e);
                            v[it][0] = lo_half(raw.x);
                            v[it][1] = hi_half(raw.x);
                            v[it][2] = lo_half(raw.y);
                            v[it][3] = hi_half(raw.y);
                        }
                    }
                    flow_norm(v, gq, d, kpad, p.eps, act_hi, act_lo, red, nullptr, nullptr, nullptr);
                    break;
                }
                case FL_QKV:
                    poll_vec<kMaxNormIter>(p, flow_ptr<const unsigned long long>(tab.io, FL_QKV, FI_IN), d, step_tag(p, step, TS_X), v);
                    stamp(step, sec, kTraceReleased);
                    flow_norm(v, gq, d, kpad, p.eps, act_hi, act_lo, red, resid, nullptr, nullptr);
                    break;
                case FL_GATEUP: { // x1 = x + w_o a
                    poll_vec<kMaxNormIter>(p, flow_ptr<const unsigned long long>(tab.io, FL_GATEUP, FI_IN), d, step_tag(p, step, TS_O), v);
                    stamp(step, sec, kTraceReleased);
#pragma unroll
                    for (int it = 0; it < kMaxNormIter; ++it) {
                        const int e = (it * kBlock + (int)threadIdx.x) * 4;
                        if (e < d) {
                            const f32x4 r = *reinterpret_cast<const f32x4 *>(resid + e);
                            v[it][0] = r.x + v[it][0];
                            v[it][1] = r.y + v[it][1];
                            v[it][2] = r.z + v[it][2];
                            v[it][3] = r.w + v[it][3];
                        }
                    }
                    flow_norm(v, gq, d, kpad, p.eps, act_hi, act_lo, red, resid, nullptr, nullptr);
                    break;
                }
                case FL_HEAD: { // x2 = x1 + w_down m; the step's output hidden state
                    poll_vec<kMaxNormIter>(p, flow_ptr<const unsigned long long>(tab.io, FL_HEAD, FI_IN), d, step_tag(p, step, TS_DN), v);
                    stamp(step, sec, kTraceReleased);
#pragma unroll
                    for (int it = 0; it < kMaxNormIter; ++it) {
                        const int e = (it * kBlock + (int)threadIdx.x) * 4;
                        if (e < d) {
                            const f32x4 r = *reinterpret_cast<const f32x4 *>(resid + e);
                            v[it][0] = r.x + v[it][0];
                            v[it][1] = r.y + v[it][1];
                            v[it][2] = r.z + v[it][2];
                            v[it][3] = r.w + v[it][3];
                        }
                    }
                    float *ho = (vb == 0 && p.hidden_out) ? p.hidden_out + (size_t)step * d : nullptr;
                    flow_norm(v, gq, d, kpad, p.eps, act_hi, act_lo, red, nullptr, resid, ho);
                    break;
                }
                case FL_O: { // the attention's result, as it is
                    const int n = p.qd;
                    const unsigned tag = step_tag(p, step, TS_ATTN);
                    for (int e0 = 0; e0 < kpad; e0 += kMaxNormIter * kBlock * 4) {
                        poll_vec<kMaxNormIter>(p, p.attnt + e0, max(min(n - e0, kMaxNormIter * kBlock * 4), 0), tag, v);
#pragma unroll
                        for (int it = 0; it < kMaxNormIter; ++it) {
                            const int e = e0 + (it * kBlock + (int)threadIdx.x) * 4;
                            if (e < kpad) {
                                const float z[4] = {0.f, 0.f, 0.f, 0.f};
                                flow_split4(e < n ? v[it] : z, act_hi, act_lo, e);
                            }
                        }
                    }
                    stamp(step, sec, kTraceReleased);
                    break;
                }
                default: { // FL_DOWN: m = silu(gate) * up: formed by the producers except for the rows dealt singly
                    const int pn = (F / nw) * nw, rem = F - pn; // pairs, then rem gate values, then rem up values
                    const unsigned tag = step_tag(p, step, TS_GU);
                    const row_rsrc gu_rs = make_vec_rsrc(p.gut, (size_t)(F + rem) * 8);
                    for (int e0 = 0; e0 < kpad; e0 += kMaxNormIter * kBlock * 4) {
                        poll_vec<kMaxNormIter>(p, p.gut + e0, max(min(pn - e0, kMaxNormIter * kBlock * 4), 0), tag, v);
#pragma unroll
                        for (int it = 0; it < kMaxNormIter; ++it) {
                            const int e = e0 + (it * kBlock + (int)threadIdx.x) * 4;
                            if (e < kpad) {
                                float m[4] = {0.f, 0.f, 0.f, 0.f};
                                if (e < pn) {
#pragma unroll
                                    for (int q = 0; q < 4; ++q) m[q] = v[it][q];
                                } else if (e < F) { // a group of four never straddles: pn, rem and F are multiples of 8
                                    float gt[4], up[4];
                                    poll4x2(p, gu_rs, e * 8, (e + rem) * 8, tag, gt, up);
#pragma unroll
                                    for (int q = 0; q < 4; ++q) m[q] = silu_mul(gt[q], up[q]);
                                }
                                flow_split4(m, act_hi, act_lo, e);
                            }
                        }
                    }
                    stamp(step, sec, kTraceReleased);
                    break;
                }
                }
            }
            if (slot_late) { // the third chunk requested ahead for this phase (see the end of a phase)
                flow_issue_lds<CL>(L, tab, nw, slot, lane);
                slot_late = false;
            }
            flow_barrier();
            stamp(step, sec, kTraceStaged);

            // ---- stream this wave's rows --------------------------------------------------------------------------
            const int next = ph == FL_QKV ? FL_NONE : ph == FL_HEAD ? (step + 1 < p.K ? FL_PROJH : FL_NONE) : ph + 1;
            const unsigned out_tag = step_tag(p, step, ph == FL_PROJE ? TS_X : ph == FL_QKV ? TS_QKV : ph == FL_O ? TS_O
                                                       : ph == FL_GATEUP ? TS_GU : TS_DN);
            unsigned long long *out_t = flow_ptr<unsigned long long>(tab.io, ph, FI_OUT); // (of the phases that have one)
            float *logits = (ph == FL_HEAD && p.logits_out) ? p.logits_out + (size_t)step * p.n : nullptr;
            unsigned long long best = 0ull; // output head: best (logit, row) this wave has seen (lane 0)
            float gate_saved = 0.f;
            const int pair_rounds = flow_num(tab, FL_GATEUP, FN_A), pair_rows = 2 * pair_rounds;
            const bool throttle = nchunks >= 8;

            f32x4 acc_h = {0.f, 0.f, 0.f, 0.f}, acc_l = {0.f, 0.f, 0.f, 0.f};
            const int dv = (lane & 15) - 4 * (lane >> 4); // which of this lane's four results lies on the diagonal
            int c_row = wr0, c_j = 0, c_c = 0;
            // one chunk: eight blocks of the row against the staged activations; w(u) = the chunk's u-th 1 KiB
            auto consume = [&](auto w) {
#pragma unroll
                for (int u = 0; u < CL; ++u) {
                    // slots past the row's last block hold zero weights: they re-read the last block's activations
                    const int e0 = min(c_c * CL + u, nblk - 1) * 512 + lane * 8;
                    const u32x4 ah = *reinterpret_cast<const u32x4 *>(act_hi + e0);
                    const u32x4 al = *reinterpret_cast<const u32x4 *>(act_lo + e0);
                    const u32x4 wv = w(u);
                    acc_h = mfma16(ah, wv, acc_h);
                    acc_l = mfma16(al, wv, acc_l);
                }
            };
            // the cursor moves on to the phase that follows once this phase's share is exhausted
            auto advance_cursor = [&]() {
                if (L.n >= nchunks && L.id == ph && next != FL_NONE) flow_load_begin(L, tab, next, wr0);
            };
            auto row_end = [&](int n) {
                if (n < nreal && ++c_c == cpr) { // end of a row: sum the diagonal
                    c_c = 0;
                    const f32x4 t = acc_h + acc_l;
                    float val = dv == 0 ? t.x : dv == 1 ? t.y : dv == 2 ? t.z : dv == 3 ? t.w : 0.f;
                    val = wave_sum(val);
                    acc_h = f32x4{0.f, 0.f, 0.f, 0.f};
                    acc_l = f32x4{0.f, 0.f, 0.f, 0.f};
                    if (lane == 0) {
                        const int li = c_j; // this wave's c_j-th row
                        switch (ph) {
                        case FL_PROJH: ppart[li] = val; break;
                        case FL_PROJE: st_tagged(out_t + c_row, ppart[li] + val, out_tag); break;
                        case FL_GATEUP: {
                            const int w = c_row - c_j * nw;
                            if (c_j < pair_rows) {
                                if ((c_j & 1) == 0)
                                    gate_saved = val;
                                else
                                    st_tagged(out_t + (c_j >> 1) * nw + w, silu_mul(gate_saved, val), out_tag);
                            } else { // dealt singly: gate values, then up values, behind the pairs
                                st_tagged(out_t + c_row - pair_rounds * nw, val, out_tag);
                            }
                            break;
                        }
                        case FL_HEAD: {
                            if (logits) logits[c_row] = val;
                            const unsigned long long key = argmax_key(val, (uint32_t)c_row);
                            best = key > best ? key : best;
                            break;
                        }
                        default: st_tagged(out_t + c_row, val, out_tag); break;
                        }
                    }
                    c_row += nw;
                    ++c_j;
                }
            };
            // Chunks n0 and n0 + 1 sit in the register slots; the phase's third chunk sits in the LDS slot and is taken
            // after the first two.  Every register slot is refilled as soon as it is free; the LDS slot is refilled once,
            // at the end of the phase, with the third chunk of the phase that follows.
            int pend = 0; // register slots whose refill waits for the end of the phase
            flow_wait_loads();
            for (int n0 = 0; n0 < nchunks; n0 += (n0 == 0 ? 3 : 2)) {
#pragma unroll
                for (int s = 0; s < 2; ++s) {
                    consume([&](int u) { return ring[s][u]; });
                    advance_cursor();
                    // Long phases keep ONE chunk in flight per wave while they stream (the other slot's loads are waited
                    // for before the next request goes out): 16 MiB over the chip already covers the memory latency, more
                    // only deepens the queues, and the compute dies then share the bandwidth unevenly (output head: the
                    // odd-numbered dies finished 6 us after the even ones with two chunks in flight).  The other slots
                    // earn their keep at the ends of a phase, where the requests run ahead into the next one.
                    // The phase's last chunks (the cursor has moved on to the phase that follows): the row's result goes
                    // out first, and the slot's next request waits until the wave has published all its results.  A
                    // request can wait a microsecond for room in the memory queues, and other workgroups poll for
                    // these results.
                    if (L.id != ph) {
                        row_end(n0 + s);
                        pend |= 1 << s;
                    } else {
                        if (throttle) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
                        flow_issue(L, tab, nw, ring[s], lane);
                        row_end(n0 + s);
                    }
                }
                if (n0 == 0) {
                    consume([&](int u) { return *reinterpret_cast<const u32x4 *>(slot + u * 1024 + lane * 16); });
                    row_end(2);
                }
            }
            if (pend & 1) flow_issue(L, tab, nw, ring[0], lane);
            if (pend & 2) flow_issue(L, tab, nw, ring[1], lane);
            // The LDS slot's chunk of the next phase is requested by that phase, behind its polls (a wave's loads
            // complete in order, and a poll behind three chunks per wave returns 2 us later than behind two; with one
            // chunk or none in front of them the polls gain less than the memory system loses: 141.7 and 149.5 us per
            // step against 137.4).
            if (next != FL_NONE) { // (no next phase: nothing is written into LDS that the attention may be using)
                advance_cursor();
                slot_late = true;
            }
            if (ph == FL_HEAD) {
                // the workgroup's candidate: (logit, token id), each with the tag in its upper half
                const unsigned long long m = block_max_u64_lds(best, red64);
                if (threadIdx.x == 0) {
                    unsigned lg = 0u, id = 0xffffffffu; // no row in this workgroup: loses against every candidate
                    if (m != 0ull) {
                        const uint32_t row = key_index(m);
                        lg = (unsigned)(m >> 32);
                        id = p.ids ? (unsigned)p.ids[row] : row;
                    }
                    const unsigned tag = step_tag(p, step, TS_CAND);
                    unsigned long long *c = p.candt + ((size_t)step * p.head_grid + vb) * 2;
                    __hip_atomic_store(c, ((unsigned long long)tag << 32) | lg, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    __hip_atomic_store(c + 1, ((unsigned long long)tag << 32) | id, __ATOMIC_RELAXED,
                                       __HIP_MEMORY_SCOPE_AGENT);
                }
            }
            stamp(step, sec, kTraceDone);
            if (ph == FL_QKV) { // attention: polls q, k, v itself and publishes its result as tagged elements
                stamp(step, 2, kTraceRequested);
                flow_barrier(); // the activations' LDS becomes the attention's
                stamp(step, 2, kTraceReleased);
                stamp(step, 2, kTraceStaged);
                call_attn<G, HD, true, true, true, kFlowAttnParts<G>>(p, step, vb, nvb, smem);
                stamp(step, 2, kTraceDone);
                // Nothing was requested ahead: the attention has the registers.  (Requested here, not where the phase begins:
                // there the ring would count as in use all through the attention.)
                flow_load_begin(L, tab, FL_O, wr0);
                flow_issue(L, tab, nw, ring[0], lane);
                flow_issue(L, tab, nw, ring[1], lane);
                flow_issue_lds<CL>(L, tab, nw, slot, lane);
            }
        }
    }
    // publish the last draft id
    if (vb == 0) {
        flow_barrier();
        const int did = winner(p.K - 1);
        if (threadIdx.x == 0) p.draft_out[p.K - 1] = seq_dead(p, 0) ? -1 : did;
    }
}

} // namespace mtp
