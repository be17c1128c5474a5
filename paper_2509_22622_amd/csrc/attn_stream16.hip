// The software-pipelined sink+window attention kernel of attn_stream.hip with both products on the 16x16x32 bf16
// MFMA instead of the 32x32x16 one (same mathematics, same cache layout in HBM, same LDS ring, same step plan).
//
// Why a second shape: under a full matrix load with real operand bits the chip is power-limited, and the 16x16x32
// instruction moves half as many accumulator bits per flop (a pure stream of them sustains about 13 % more than a
// stream of 32x32x16 MFMAs on the same chip).  A wave still owns 32 queries, now as two column blocks of 16, so every
// K or V^T fragment read from LDS feeds two MFMAs and the LDS traffic per flop is unchanged.
//
// Operand geometry (lane = 16 * g + n, g = 0..3, n = 0..15):
//   S^T block (m, qb) = K rows of key group m  x  queries 16 qb + n, contraction over 32 features per MFMA:
//       A: lane (g, n) holds A-row n, features 32 s + 8 g + 0..7;  B: query 16 qb + n, the same features;
//       C: lane (g, n) register j = A-row 4 g + j.
//     A-row r of key group m is taken from stored row (r & 7) + 8 m + 16 (r >> 3) of the K kblock (which holds key
//     swap23(row), see kernels.h), so that register j of lane (g, n) is key 8 g + 4 m + j: the eight scores a lane
//     holds for one query block are keys 8 g .. 8 g + 7 in the order (m, j).
//   O^T block (dq, qb) = V^T rows 16 dq + n  x  queries 16 qb + n, contraction over the kblock's 32 keys in ONE MFMA:
//       A: lane (g, n) holds feature 16 dq + n, keys 8 g + 0..7: one 16-byte piece of the V kblock as stored;
//       B: lane (g, n) holds keys 8 g + 0..7 of query 16 qb + n: exactly its own eight softmax weights.
//     So the weights never leave the lane here either.
// The K fragments are permuted on their way into LDS (direct-to-LDS loads take any 16 bytes of memory per lane but
// write lane l at offset 16 l): lane (c, m, r) of a load fetches stored row (r & 7) + 8 m + 16 (r >> 3) of 16-byte
// chunk c, which puts the 16 rows an MFMA's lane group reads side by side (no bank conflicts).
//
// A step (one kblock) keeps the 16 (D = 128) slots of attn_stream.hip, each now opened by the TWO MFMAs that share a
// fragment: K fragment k = (s = k / 2, m = k % 2) feeds S^T blocks (m, 0) and (m, 1); the O^T slots take the query
// block qb = 0 first (V^T fragments 2 j, 2 j + 1 in slot j), then qb = 1 with the same fragments again, so the
// weights of query block 0 are needed when the O^T slots begin and those of block 1 half way through them, as the
// two key halves were in the 32x32x16 form.  Exponentials, packing, row sums, the running maximum, fragment reads,
// direct-to-LDS loads, waits and barriers sit in the same slots (lds_plan.h: LdsPlan16, RingPlan).
//
// A launch of few rows and heads has fewer 256-row tiles than the chip has CUs, and every workgroup of it walks all
// keys.  Such a launch deals a tile's keys to G = 2, 4 or 8 groups of the workgroup's waves (template parameter G; the rule is
// key_groups_log2 in attn_kernel.hip): a tile is 256 / G rows, a group of 8 / G waves walks its share through a ring
// of its own (lds_plan.h: GroupRing), and the groups' results meet in LDS, so no memory outside the workgroup is
// needed.  What bounds it: with 256 / G rows per kblock the LDS (fragment reads and ring writes, 144, 160 and 192 KB
// per step at G = 1, 2, 4 and head_dim 128) and, with all CUs at work, L2 (12.5 TB/s at G = 4).  Measured, us: 270 rows x 43 kblocks x
// 6 heads x 64: 25 -> 10 (G = 8); 1170 x 183 x 12 x 128: 121 -> 57 (G = 4; 52 with keys from memory, brought into L2 ahead: S16Touch); 1560 x 634 x 12 x 128: 361 -> 231 (G = 2).  One barrier per step with
// loads three steps ahead instead of one per two steps and one period ahead was slower (head_dim 64, G = 2: 55 against 48).
// A streamed chunk may also have its tiles' keys dealt to several workgroups (rule: attn_split in attn_kernel.hip), which need
// not share one CU's LDS and its 64 bytes a clock from L2 and whose rings can be long again: G * splits shares of a tile's
// keys, partial results through the slots of split.h, and a second kernel that adds them up.  What bounds
// it then: some 7 us of a workgroup around its steps, the merge's launch, and the partial results' way (0.25 us per MB there
// and back).  us without and with: 190 rows x 143 kblocks x 4 heads x 128 34 -> 19, 1560 x 634 x 12 x 128 206 -> 165.
#include "kernels.h"
#include "lds_plan.h"
#include "split.h"

namespace ll {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
typedef unsigned u32x2 __attribute__((ext_vector_type(2)));

constexpr float S16_RESCALE_SLACK = 6.0f;        // log2 units: p stays below 2^6 between rescales
constexpr int S16_THREADS = 512;
// Fixed-reference pass: a row sum above this (weights of 2^(score - reference), reference = largest score of the first
// kblock) sends the tile to the pass that follows the maximum.  Far below what fp32 sums and bf16 weights can hold.
constexpr float S16_FIXED_REF_LIMIT = 0x1p48f;

__device__ __forceinline__ unsigned s16_pack_bf16(float a, float b) {
    f32x2 v = {a, b};
    return __builtin_bit_cast(unsigned, __builtin_convertvector(v, bf16x2));
}
template <int N>
__device__ __forceinline__ void s16_wait_vmcnt() {
    __builtin_amdgcn_s_waitcnt((N & 0xF) | ((N >> 4) << 14) | (0x7 << 4) | (0xF << 8));
}
// LDS reads the compiler does not see; see attn_stream.hip.  The read leaves `dst` pending until s16_lds_wait<N>(dst)
// has run with N = reads issued after it by then.
__device__ __forceinline__ void s16_lds_read(u32x4& dst, unsigned addr, int offset) {
    asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(dst) : "v"(addr), "n"(offset));
}
template <int N>
__device__ __forceinline__ void s16_lds_wait(u32x4& x) {
    asm volatile("s_waitcnt lgkmcnt(%1)" : "+v"(x) : "n"(N));
}
__device__ __forceinline__ void s16_lds_wait_n(u32x4& x, int n) {
    switch (n < 15 ? n : 15) {
        case 0: s16_lds_wait<0>(x); break;
        case 1: s16_lds_wait<1>(x); break;
        case 2: s16_lds_wait<2>(x); break;
        case 3: s16_lds_wait<3>(x); break;
        case 4: s16_lds_wait<4>(x); break;
        case 5: s16_lds_wait<5>(x); break;
        case 6: s16_lds_wait<6>(x); break;
        case 7: s16_lds_wait<7>(x); break;
        case 8: s16_lds_wait<8>(x); break;
        case 9: s16_lds_wait<9>(x); break;
        case 10: s16_lds_wait<10>(x); break;
        case 11: s16_lds_wait<11>(x); break;
        case 12: s16_lds_wait<12>(x); break;
        case 13: s16_lds_wait<13>(x); break;
        case 14: s16_lds_wait<14>(x); break;
        default: s16_lds_wait<15>(x); break;
    }
}
// a register that arrived together with (or before) one just waited for: only ties it to this point of the program
__device__ __forceinline__ void s16_lds_arrived(u32x4& x) { asm volatile("" : "+v"(x)); }

__device__ __forceinline__ int s16_pick(int v, int n0, int n01, int a0, int a1, int a2) {
    return v < n0 ? a0 : (v < n01 ? a1 : a2);
}
// (`dead`: first step of a share past its last kblock, 0x7FFFFFFF where there is none)
__device__ __forceinline__ int s16_next_edge(int v, int n0, int n01, int T, int dead) {
    const int cand[6] = {0, n0 - 1, n0, n01 - 1, n01, T - 1};
    int best = dead > v ? dead : 0x7FFFFFFF;
#pragma unroll
    for (int c = 0; c < 6; ++c)
        if (cand[c] > v && cand[c] < best) best = cand[c];
    return best;
}
// bit e set: key key0 + 8 g + e (the e-th of the eight keys lane group g holds of a kblock) is inside [rs, re)
__device__ __forceinline__ unsigned s16_live_mask(int key0, int rs, int re, int g) {
    unsigned live = 0;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        const int key = key0 + 8 * g + e;
        if (key >= rs && key < re) live |= 1u << e;
    }
    return live;
}

// Softmax state of the 32 queries of a wave: lane (g, n) holds, for query 16 qb + n, O^T rows 16 dq + 4 g + j
// (unnormalised), the row sum over the keys this lane saw (the four lane groups of a column add up to the query's
// sum) and the reference all four share.
template <int D>
struct S16State {
    f32x4 o[D / 16][2];
    float l[2], m[2];
};

// byte offset, inside a 1 KB K fragment as stored, of the 16 bytes that load lane `lane` fetches (see the file header)
__device__ __forceinline__ unsigned s16_k_load_offset(int lane) {
    const int c = lane >> 5, m = (lane >> 4) & 1, r = lane & 15;
    return unsigned(c * 32 + (r & 7) + 8 * m + 16 * (r >> 3)) * 16u;
}

// Virtual kblocks [vb, ve) of chunk `ch` for the 32 queries starting at row q0 of head `head`.
// SCHED selects where a step's vector and LDS work sits (bit 0: exponentials of the second query block moved behind
// the S^T slots; bit 1: one LDS fragment read per slot instead of two in half of the slots; bit 2: no issue priority)
// and, bit 3, whether the reference is fixed: the scores' running maximum is then not followed at all (no max3, no
// vote, no rescaling), the reference stays at the first kblock's maximum, and the caller must look at the row sums
// afterwards: a sum beyond S16_FIXED_REF_LIMIT (or not a number) means some score rose far above the reference, and
// the tile has to be computed again with the reference followed.
// G: key groups of the workgroup (lds_plan.h: GroupRing).  G == 1: all eight waves walk the chunk's kblocks [vb, ve)
// through one ring.  G > 1: this wave's group of 8 / G waves walks its own share [vb, ve) through its own ring and runs
// n_steps >= ve - vb steps, as many as the longest share has (a step past ve has no live key).
// `gate` is the barrier behind the first loads; where it says no (to the whole workgroup) nothing is computed: false.
// (Kernel: keeps what the kernels of this file share apart, which otherwise changes with every user of it: 5 registers more and 1.5 %
// of the time of the unsplit kernels)
template <int Kernel>
struct S16Barrier {
    static constexpr bool STOPS = false;
    using Again = S16Barrier;
    __device__ __forceinline__ bool operator()() const { __builtin_amdgcn_s_barrier(); return true; }
};
using S16Unsplit = S16Barrier<0>;
using S16NextShare = S16Barrier<1>;
// `touch` (GroupRing::TOUCHES in lds_plan.h): the periods whose kblocks this tile brings into L2.
// Where the key set has S16_TOUCH_BYTES and more: a few layers of it do not fit the 256 MB of the last-level cache, so it comes from
// memory.  us a call with the keys of many layers in turn, without and with: 1170 rows x 183 kblocks x 12 heads x 128 (36 MB)
// 70 -> 52, x 293 107 -> 78, 800 x 125 x 16 51 -> 39; a key set that is in that cache (four layers' just written) 50.8 and 49.8.
constexpr int S16_TOUCH_BYTES = 16 << 20;
struct S16Touch { int every = 0, first = 0; };                   // (0: none)
// The tiles of a head walk the same keys, more or less in step; those on one XCD take turns.  total: workgroups of a
// launch that deals them out evenly, this one the idx-th of its XCD; 0 where whole (head, chunk) groups lie on an XCD.
template <int D, int G>
__device__ __forceinline__ S16Touch s16_take_turns(const AttnChunk& ch, int heads, int row0, int tile, int idx, int total) {
    S16Touch t;
    if (!GroupRing<D, G>::TOUCHES || ch.n_kblocks * heads < S16_TOUCH_BYTES / (4 * KBLOCK * D)) return t;
    int before = tile - ch.tile_begin, after = (ch.q_end - 1 - row0) / (256 / G);
    if (total > 0) {
        const int xcd = blockIdx.x & 7, here = (((xcd + 1) * total + 7) >> 3) - ((xcd * total + 7) >> 3);
        before = min(before, idx);
        after = min(after, here - 1 - idx);
    }
    const int n = before + 1 + after;
    t.every = n >= 8 ? 8 : n >= 4 ? 4 : n >= 2 ? 2 : 1;
    t.first = before & (t.every - 1);
    return t;
}
// (TOUCH: a form of its own, since the code for it costs a call that does not touch 0.4 us of 25)
template <int D, bool QSCALE, int SCHED, int G, bool TOUCH, typename Gate>
__device__ __forceinline__ bool s16_segment(const AttnParams& p, const AttnChunk& ch, int tid, int head, int q0, int vb, int ve,
                                            int n_steps, char* lds, S16State<D>& st, const float2* shift_cs, Gate gate, S16Touch touch = {}) {
    using Plan = LdsPlan16<D, (SCHED & 2) != 0>;
    constexpr bool TRACK = !(SCHED & 8);
    constexpr int KS = Plan::KS;                // K fragments per kblock = S^T slots (two MFMAs each)
    constexpr int NV = Plan::NV;                // V^T fragments per kblock = O^T slots (two MFMAs each)
    constexpr int NQ = D / 32;                  // contraction steps of S^T
    constexpr int HV = NV / 2;                  // O^T slots per query block
    constexpr int KB_BYTES = KBLOCK * D * 2;
    constexpr int STAGE_BYTES = 2 * KB_BYTES;   // [K kblock | V kblock]
    constexpr int NS = RingPlan::STAGES;
    constexpr int NF = KS + NV;                 // 1 KB fragments per stage
    using GR = GroupRing<D, G>;
    constexpr int NW = 8 / G;                   // waves that share a ring
    constexpr int PERIOD = G == 1 ? 2 : GR::PERIOD;             // steps per barrier
    constexpr int LPW = G == 1 ? NF / NW : PERIOD * NF / NW;    // direct-to-LDS loads per wave, per kblock (per period)
    constexpr int PF = RingPlan::AHEAD;
    constexpr int LAND = RingPlan::LANDED;
    // A share of the keys may begin with a kblock that scores -inf throughout for some query, although the key set does not:
    // the pass that follows the maximum then has no reference (mref -inf, scores relative to 0) until a live score comes.
    // (The fixed-reference pass makes NaN of it, which sends the tile there.)
    constexpr bool NO_REF = TRACK;
    static_assert(NF % NW == 0 && (G == 1 || KS % NW == 0), "fragments must split over the waves");
    static_assert(PF >= LAND && PF + 2 <= NS, "ring too short for the prefetch distance");

    const int lane = tid & 63;
    const int wave_wg = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wave = wave_wg % NW;              // among the waves that share this ring
    const int n = lane & 15, g = lane >> 4;
    char* const lds_touch = lds + G * GR::BYTES + wave_wg * GR::LDS_TOUCH;
    if (G > 1) lds += (wave_wg / NW) * GR::BYTES;

    const int n_ranges = ch.n_ranges;
    const int rs0 = ch.rs[0], re0 = ch.re[0];
    int rs1 = ch.rs[1], re1 = ch.re[1], rs2 = ch.rs[2], re2 = ch.re[2];
    if (n_ranges < 2) rs1 = re1 = 0;
    if (n_ranges < 3) rs2 = re2 = 0;
    const int kb0 = rs0 / KBLOCK, ke0 = (re0 + KBLOCK - 1) / KBLOCK;
    const int kb1 = rs1 / KBLOCK, ke1 = (re1 + KBLOCK - 1) / KBLOCK;
    const int kb2 = rs2 / KBLOCK, ke2 = (re2 + KBLOCK - 1) / KBLOCK;
    const int q_end = ch.q_end;
    const int T = (ke0 - kb0) + (ke1 - kb1) + (ke2 - kb2);
    const int n0 = ke0 - kb0, n01 = n0 + (ke1 - kb1);
#define S16_PHYS_KB(v) ((v) + s16_pick((v), n0, n01, kb0, kb1 - n0, kb2 - n01))
#define S16_LIVE(v) (G > 1 && (v) >= ve ? 0u : \
    s16_live_mask(S16_PHYS_KB(v) * KBLOCK, s16_pick((v), n0, n01, rs0, rs1, rs2), s16_pick((v), n0, n01, re0, re1, re2), g))
    const int v_end = G == 1 ? ve : vb + n_steps;
    const int dead = G > 1 && v_end > ve ? ve : 0x7FFFFFFF;

    const char* kbase = reinterpret_cast<const char*>(p.k_cache + head * p.head_stride);
    const char* vbase = reinterpret_cast<const char*>(p.v_cache + head * p.head_stride);

    const unsigned lane_off = lane * 16;
    const unsigned k_load_off = s16_k_load_offset(lane);
    // LDS byte address of this lane's 16 bytes in fragment 0 of stage 0; fragment f of a kind adds s16_frag(f)
    const unsigned lds_a = (unsigned)(size_t)(__attribute__((address_space(3))) char*)lds + g * 512 + n * 16;
#define S16_FRAG(f) (((f) >> 1) * 2048 + ((f) & 1) * 256)
    auto issue_load = [&](int kb, int stage, int l) {
        const int64_t kb_off = int64_t(kb) * KB_BYTES;
        const int f = wave + NW * l;            // fragment of the stage this wave fetches (wave-uniform)
        const char* src = (f < KS ? kbase + f * 1024 + k_load_off : vbase + (f - KS) * 1024 + lane_off) + kb_off;
        char* dst = lds + stage * STAGE_BYTES + f * 1024;
        __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)(src),
                                         (__attribute__((address_space(3))) void*)(dst), 16, 0, 0);
    };

    // G > 1: load l of the period that begins with step `first` (relative to vb): V of its kblocks, K two kblocks on
    auto issue_group = [&](int first, int l) {
        constexpr int DEPTH = GR::DEPTH;
        const int j = (NW * l) / NF, part = (NW * l) % NF;          // compile-time where l is
        const bool is_k = part < KS;
        const int rel = first + j + (is_k ? 2 : 0);
        const int v = min(vb + rel, ve - 1);
        const int fr = (is_k ? part : part - KS) + wave;
        const char* src = (is_k ? kbase + k_load_off : vbase + lane_off) + int64_t(S16_PHYS_KB(v)) * KB_BYTES + fr * 1024;
        char* dst = lds + ((is_k ? 0 : DEPTH) + (rel & (DEPTH - 1))) * KB_BYTES + fr * 1024;
        __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)(src),
                                         (__attribute__((address_space(3))) void*)(dst), 16, 0, 0);
    };
    // the kblock of the period that begins with step `first` (a period is one step where anything is touched), 128 bytes a lane (past
    // the share's end the last one again)
    auto touch_period = [&](int first) {
        const int in = wave * 64 + lane;         // of a kblock's K and V
        const char* src = (in < D / 2 ? kbase : vbase) + in % (D / 2) * 128 + int64_t(S16_PHYS_KB(min(vb + first, ve - 1))) * KB_BYTES;
        __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)(src),
                                         (__attribute__((address_space(3))) void*)(lds_touch), 4, 0, 0);
    };
    int touch_in = touch.first, touch_at = (touch.first + 1 + GR::TOUCH_AHEAD) * PERIOD;        // periods to the next touch; its step
    // end of a period of a group's ring: what this wave loaded for the next one has landed (but not what it touches now), and
    // its K fragment reads, whose stages the loads issued next overwrite, have returned; then every wave's have
    auto group_handover = [&](u32x4 (&kf)[KS]) {
#pragma unroll
        for (int k = 0; k < KS; ++k) s16_lds_wait<0>(kf[k]);
        if (TOUCH && --touch_in < 0) {
            asm volatile("" ::: "memory");       // the touch is the last load in front of the wait that leaves one out: not even
            touch_period(touch_at);              // the compiler may move another between them
            touch_in += touch.every;
            touch_at += touch.every * PERIOD;
            asm volatile("s_waitcnt vmcnt(%0)" ::"n"(GR::TOUCH_LOADS) : "memory");
        } else {
            s16_wait_vmcnt<0>();
        }
        if constexpr (NW > 1) __builtin_amdgcn_s_barrier();
    };

    // the ring's first loads go out before the queries are fetched: one memory latency for both
    u32x4 kfr[KS];                               // K fragments of kblock i + 1
    u32x4 kfirst[G == 1 ? 1 : KS];               // G > 1: those of kblock vb; the ring begins with kblock vb + 2
    if constexpr (G == 1) {
#pragma unroll
        for (int j = 0; j < PF; ++j) {
            const int v = min(vb + j, ve - 1);
#pragma unroll
            for (int l = 0; l < LPW; ++l) issue_load(S16_PHYS_KB(v), (vb + j) & (NS - 1), l);
        }
    } else {
#pragma unroll
        for (int l = 0; l < LPW; ++l) issue_group(0, l);
        if constexpr (TOUCH)
            for (int t = touch.first; t < GR::TOUCH_AHEAD; t += touch.every) touch_period((t + 1) * PERIOD);
        // the same 16 bytes per lane as the reads of the permuted fragments below, straight from memory
        const unsigned k_lane = (g >> 1) * 1024 + ((g & 1) * 32 + (n & 7) + 16 * (n >> 3)) * 16;
        const char* k0 = kbase + int64_t(S16_PHYS_KB(vb)) * KB_BYTES + k_lane;
        const char* k1 = kbase + int64_t(S16_PHYS_KB(min(vb + 1, ve - 1))) * KB_BYTES + k_lane;
#pragma unroll
        for (int k = 0; k < KS; ++k) {
            kfirst[k] = *reinterpret_cast<const u32x4*>(k0 + (k >> 1) * 2048 + (k & 1) * 128);
            kfr[k] = *reinterpret_cast<const u32x4*>(k1 + (k >> 1) * 2048 + (k & 1) * 128);
        }
    }

    // Q^T fragments (pre-scaled by log2(e)/sqrt(D)): fragment (qb, s) holds features 32 s + 8 g + 0..7 of query q0 + 16 qb + n
    bf16x8 qf[2][NQ];
    const uint16_t* q_src[2];
#pragma unroll
    for (int qb = 0; qb < 2; ++qb) {
        q_src[qb] = p.q + (int64_t(min(q0 + 16 * qb + n, q_end - 1)) * p.H + head) * D + g * 8;
#pragma unroll
        for (int s = 0; s < NQ; ++s) qf[qb][s] = *reinterpret_cast<const bf16x8*>(q_src[qb] + s * 32);
    }
    if constexpr ((SCHED & 16) != 0) {
        // the queries come as the model's projection made them: turn this lane's pairs (3D rotary embedding, the
        // frame axis from the table the cache write left, rows and columns from the cache's tables) and fold in the
        // softmax scale, with the arithmetic of the cache-write kernel (kernels.h: rope_turn_scaled).  The tables are read two
        // pairs at a time: the lanes' addresses scatter, and one pair each (32 loads a lane at head_dim 128) kept the
        // address units busy for 2.6 us in front of a workgroup's first step, two 1.3.
        constexpr int NH = D / 6, NT = D / 2 - 2 * NH;              // rotary pairs of the row (and column) axis, of the frame axis
        static_assert(NT % 2 == 0, "two neighbouring pairs lie on one axis, but for the last of an odd row axis");
        typedef float f32x4_8 __attribute__((ext_vector_type(4), aligned(8)));
#pragma unroll
        for (int qb = 0; qb < 2; ++qb) {
            const int rel = min(q0 + 16 * qb + n, q_end - 1) - ch.q_begin;
            const int fi = rel / p.P, tok = rel - fi * p.P;
            const int y = tok / p.grid_w, x = tok - y * p.grid_w;
            const float2* t_cs = p.t_table + (ch.t_row + fi) * MAX_T_PAIRS;
            const float2* r_cs = p.row_cs + y * NH - NT;
            const float2* c_cs = p.col_cs + x * NH - NT - NH;
#pragma unroll
            for (int s = 0; s < NQ; ++s)
#pragma unroll
                for (int j = 0; j < 4; j += 2) {
                    const int pi = 16 * s + 4 * g + j;      // rotary pairs of features 32 s + 8 g + 2 j .. + 3
                    f32x4 w = *reinterpret_cast<const f32x4_8*>((pi < NT ? t_cs : pi < NT + NH ? r_cs : c_cs) + pi);
                    constexpr int LAST = NT + NH - 1;       // the row axis's last pair (its row's end is not the table's)
                    if (LAST % 2 == 0 && LAST / 16 == s && LAST % 4 == j) {
                        const float2 first = c_cs[LAST + 1];
                        if (pi == LAST) {
                            w[2] = first.x;
                            w[3] = first.y;
                        }
                    }
#pragma unroll
                    for (int k = 0; k < 2; ++k) {
                        float re, im;
                        rope_turn_scaled(float(qf[qb][s][2 * (j + k)]), float(qf[qb][s][2 * (j + k) + 1]), make_float2(w[2 * k], w[2 * k + 1]), p.q_scale, re, im);
                        qf[qb][s][2 * (j + k)] = __bf16(re);
                        qf[qb][s][2 * (j + k) + 1] = __bf16(im);
                    }
                }
        }
    }
    if constexpr (QSCALE) {
        const float c = p.scale_log2e;
#pragma unroll
        for (int qb = 0; qb < 2; ++qb)
#pragma unroll
            for (int s = 0; s < NQ; ++s)
#pragma unroll
                for (int j = 0; j < 8; ++j) qf[qb][s][j] = __bf16(float(qf[qb][s][j]) * c);
    }
    // Sink at a fixed rotary distance (see attn_stream.hip): range 0 is the sink, scored with the queries turned back
    // by sink_shift frames on the frame axis; the unturned queries are loaded again in step n0 - 1.
    // (a share that begins behind the sink has nothing to turn)
    const int sink_shift = vb >= n0 ? 0 : ch.sink_shift;
    if (sink_shift != 0) {
#pragma unroll
        for (int qb = 0; qb < 2; ++qb)
#pragma unroll
            for (int s = 0; s < NQ; ++s)
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const int pi = 16 * s + 4 * g + j;      // rotary pair of features 32 s + 8 g + 2 j, + 1
                    if (pi < p.n_t) {
                        const float2 cs = shift_cs[pi];
                        const float re = float(qf[qb][s][2 * j]), im = float(qf[qb][s][2 * j + 1]);
                        qf[qb][s][2 * j] = __bf16(re * cs.x + im * cs.y);
                        qf[qb][s][2 * j + 1] = __bf16(im * cs.x - re * cs.y);
                    }
                }
    }

    s16_wait_vmcnt<G == 1 ? (PF - LAND) * LPW : 0>();
    if constexpr (NW > 1 || Gate::STOPS) {
        if (!gate()) {
            __builtin_amdgcn_s_waitcnt(0);
            return false;
        }
    }

    // dead slots may hold anything, even NaN: zero the V elements of keys outside the range
    auto mask_v = [&](u32x4 (&av)[NV], unsigned live) {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const unsigned b0 = (live >> (2 * e)) & 1, b1 = (live >> (2 * e + 1)) & 1;
            const unsigned msk = (b0 ? 0x0000FFFFu : 0u) | (b1 ? 0xFFFF0000u : 0u);
#pragma unroll
            for (int f = 0; f < NV; ++f) av[f][e] &= msk;
        }
    };
    auto mask_s = [&](f32x4 (&s)[2][2], unsigned live) {
#pragma unroll
        for (int m = 0; m < 2; ++m)
#pragma unroll
            for (int j = 0; j < 4; ++j)
                if (!((live >> (4 * m + j)) & 1)) {
                    s[m][0][j] = -INFINITY;
                    s[m][1][j] = -INFINITY;
                }
    };
    auto max_s = [&](const f32x4 (&s)[2][2], int qb) {
        float m = fmaxf(fmaxf(s[0][qb][0], s[0][qb][1]), s[0][qb][2]);
        m = fmaxf(fmaxf(m, s[0][qb][3]), s[1][qb][0]);
        m = fmaxf(fmaxf(m, s[1][qb][1]), s[1][qb][2]);
        return fmaxf(m, s[1][qb][3]);
    };
    // largest of the four lane groups that hold one query column
    auto col_max = [&](float x) {
        x = fmaxf(x, __shfl_xor(x, 16));
        return fmaxf(x, __shfl_xor(x, 32));
    };

    float lsum[2][2];                            // row sums of this lane's keys per query block (two chains each)
    float mref[2];                               // reference maximum per query block (log2 domain)
    f32x4 negm[2];                               // every element = -mref[qb]: the score accumulators start from it
    float mx[2];                                 // largest score of kblock i among this lane's keys, per query block
    f32x4 sA[2][2], sB[2][2];                    // scores [m][qb] (log2 domain) of kblocks i and i + 1
    u32x4 vfr[NV];                               // V^T fragments of kblock i

    // ---- prologue: scores of kblock vb, the first reference, K fragments of kblock vb + 1
    if constexpr (G == 1) {
        const char* kt = lds + (vb & (NS - 1)) * STAGE_BYTES + g * 512 + n * 16;
#pragma unroll
        for (int k = 0; k < KS; ++k) kfr[k] = *reinterpret_cast<const u32x4*>(kt + S16_FRAG(k));
    }
#pragma unroll
    for (int f = 0; f < NV; ++f)
#pragma unroll
        for (int qb = 0; qb < 2; ++qb) st.o[f][qb] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int m = 0; m < 2; ++m)
#pragma unroll
        for (int qb = 0; qb < 2; ++qb) sA[m][qb] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int k = 0; k < KS; ++k)
#pragma unroll
        for (int qb = 0; qb < 2; ++qb)
            sA[k & 1][qb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, G == 1 ? kfr[k] : kfirst[G == 1 ? 0 : k]),
                                                                    qf[qb][k >> 1], sA[k & 1][qb], 0, 0, 0);
    mask_s(sA, S16_LIVE(vb));
#pragma unroll
    for (int qb = 0; qb < 2; ++qb) {
        mref[qb] = col_max(max_s(sA, qb));       // a kblock of a range holds a live key: finite, unless that key scores -inf
        const float base = NO_REF && mref[qb] == -INFINITY ? 0.f : mref[qb];
        negm[qb] = f32x4{-base, -base, -base, -base};
#pragma unroll
        for (int m = 0; m < 2; ++m) sA[m][qb] -= base;
        mx[qb] = -INFINITY;
        lsum[qb][0] = lsum[qb][1] = 0.f;
    }
    if constexpr (G == 1) {
#pragma unroll
        for (int k = 0; k < KS; ++k) s16_lds_read(kfr[k], lds_a + ((vb + 1) & (NS - 1)) * STAGE_BYTES, S16_FRAG(k));
    }

    // ---- main loop: see attn_stream.hip for the plan; every slot here opens with two MFMAs
    constexpr int NSLOT = KS + NV;
    constexpr int NPAIR = 8;                     // score pairs per lane: pair j is word j % 4 of the P^T fragment of query block j / 4
    constexpr int MAX_FIRST = NSLOT - 4;
    constexpr int SPAN = KS + HV - 2;
    static_assert((3 * SPAN) / NPAIR + 1 <= KS - 1, "a packed pair would be late for its MFMA");
    static_assert(MAX_FIRST >= KS, "the running maximum would read scores still being accumulated");
    constexpr int DMA_STEP = G == 1 ? NSLOT / LPW : 1, DMA_FIRST = DMA_STEP - 1;
#define S16_PIN(x) asm volatile("" ::"v"(x))
#define S16_STEP(I, S_CUR, S_NEXT, EDGE, BAR)                                                                       \
    {                                                                                                               \
        const bool edge = EDGE && (I) == next_edge;                                                                 \
        if (__builtin_expect(edge || vote, 0)) {                                                                    \
            if (edge) {                                                                                             \
                next_edge = s16_next_edge((I), n0, n01, T, dead);                                                   \
                mask_s(S_CUR, S16_LIVE(I));                                                                         \
                if (TRACK) {                                                                                        \
                    mx[0] = max_s(S_CUR, 0);                                                                        \
                    mx[1] = max_s(S_CUR, 1);                                                                        \
                }                                                                                                   \
                if (sink_shift != 0 && (I) == n0 - 1) {     /* the sink ends here: back to the unturned queries */  \
                    _Pragma("unroll") for (int qb = 0; qb < 2; ++qb)                                                \
                        _Pragma("unroll") for (int s = 0; s < NQ; ++s)                                              \
                            qf[qb][s] = *reinterpret_cast<const bf16x8*>(q_src[qb] + s * 32);                       \
                }                                                                                                   \
            }                                                                                                       \
            if (TRACK) _Pragma("unroll") for (int qb = 0; qb < 2; ++qb) {                                           \
                const float top = col_max(mx[qb]);                                                                  \
                const bool first = NO_REF && mref[qb] == -INFINITY;      /* no reference yet: nothing to rescale */ \
                const float delta = first ? (top == -INFINITY ? 0.f : top) : fmaxf(top, 0.f);                       \
                const float alpha = first ? 1.f : __builtin_amdgcn_exp2f(-delta);                                   \
                mref[qb] = first ? top : mref[qb] + delta;                                                          \
                lsum[qb][0] *= alpha;                                                                               \
                lsum[qb][1] *= alpha;                                                                               \
                _Pragma("unroll") for (int f = 0; f < NV; ++f) st.o[f][qb] *= alpha;                                \
                negm[qb] -= delta;                                                                                  \
                S_CUR[0][qb] -= delta;                                                                              \
                S_CUR[1][qb] -= delta;                                                                              \
            }                                                                                                       \
        }                                                                                                           \
        const unsigned vt_a = lds_a + (G == 1 ? ((I) & (NS - 1)) * STAGE_BYTES + KB_BYTES                           \
                                              : (GR::DEPTH + (((I) - vb) & (GR::DEPTH - 1))) * KB_BYTES);           \
        const unsigned kt_a = lds_a + (G == 1 ? (((I) + 2) & (NS - 1)) * STAGE_BYTES                                \
                                              : (((I) + 2 - vb) & (GR::DEPTH - 1)) * KB_BYTES);                     \
        float d0[NPAIR], d1[NPAIR];                                                                                 \
        unsigned pb[2][4];                                                                                          \
        float m_run[2] = {-INFINITY, -INFINITY};                                                                    \
        _Pragma("unroll") for (int k = 0; k < NSLOT; ++k) {                                                         \
            if (k == 0 && !(SCHED & 4)) __builtin_amdgcn_s_setprio(1);                                              \
            if (k == KS && !(SCHED & 4)) __builtin_amdgcn_s_setprio(0);                                             \
            if (k < KS) {                                                                                           \
                const int m = k & 1, s = k >> 1;                                                                    \
                s16_lds_wait_n(kfr[k], Plan::wait_k(k));                                                            \
                S_NEXT[m][0] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, kfr[k]), qf[0][s], \
                                                                        s == 0 ? negm[0] : S_NEXT[m][0], 0, 0, 0);  \
                S_NEXT[m][1] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, kfr[k]), qf[1][s], \
                                                                        s == 0 ? negm[1] : S_NEXT[m][1], 0, 0, 0);  \
            } else {                                                                                                \
                const int qb = (k - KS) / HV, j = (k - KS) % HV;                                                    \
                const u32x4 bv = {pb[qb][0], pb[qb][1], pb[qb][2], pb[qb][3]};                                      \
                if (qb == 0) {                                                                                      \
                    s16_lds_wait_n(vfr[2 * j + 1], Plan::wait_v(j));                                                \
                    s16_lds_arrived(vfr[2 * j]);                                                                    \
                }                                                                                                   \
                st.o[2 * j][qb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, vfr[2 * j]),   \
                                      __builtin_bit_cast(bf16x8, bv), st.o[2 * j][qb], 0, 0, 0);                    \
                st.o[2 * j + 1][qb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, vfr[2 * j + 1]), \
                                          __builtin_bit_cast(bf16x8, bv), st.o[2 * j + 1][qb], 0, 0, 0);            \
            }                                                                                                       \
            if (G > 1) {                                                                                            \
                /* the next period's loads, in the period's first step */                                           \
                if (PERIOD == 1 || (BAR) == 0 || ((BAR) == 2 && !(((I) - vb) & 1)))                                 \
                    _Pragma("unroll") for (int l = 0; l < LPW; ++l)                                                 \
                        if (GR::dma_slot(l, LPW, NSLOT) == k) issue_group((I) - vb + PERIOD, l);                    \
            } else if (k >= DMA_FIRST && (k - DMA_FIRST) % DMA_STEP == 0 && (k - DMA_FIRST) / DMA_STEP < LPW) {     \
                const int v = min((I) + PF, ve - 1);                                                                \
                issue_load(S16_PHYS_KB(v), ((I) + PF) & (NS - 1), (k - DMA_FIRST) / DMA_STEP);                      \
            }                                                                                                       \
            _Pragma("unroll") for (int j = 0; j < NPAIR; ++j) {                                                     \
                const int qb = j / 4, w = j % 4;                                                                    \
                const int e = !(SCHED & 1) ? (j * SPAN) / NPAIR                                                     \
                              : (qb == 0 ? (w * (KS - 1)) / 4 : KS - 1 + (w * (HV - 1)) / 3);                       \
                if (k == e) {                                                                                       \
                    d0[j] = __builtin_amdgcn_exp2f(S_CUR[w >> 1][qb][2 * (w & 1)]);                                 \
                    d1[j] = __builtin_amdgcn_exp2f(S_CUR[w >> 1][qb][2 * (w & 1) + 1]);                             \
                    S16_PIN(d0[j]);                                                                                 \
                    S16_PIN(d1[j]);                                                                                 \
                }                                                                                                   \
                if (k == e + 1) {                                                                                   \
                    pb[qb][w] = s16_pack_bf16(d0[j], d1[j]);                                                        \
                    S16_PIN(pb[qb][w]);                                                                             \
                    lsum[qb][0] += d0[j];                                                                           \
                    lsum[qb][1] += d1[j];                                                                           \
                    S16_PIN(lsum[qb][0]);                                                                           \
                    S16_PIN(lsum[qb][1]);                                                                           \
                }                                                                                                   \
            }                                                                                                       \
            if (TRACK && k >= MAX_FIRST) {                                                                          \
                const int qb = (k - MAX_FIRST) >> 1, m = (k - MAX_FIRST) & 1;                                       \
                m_run[qb] = fmaxf(fmaxf(m_run[qb], S_NEXT[m][qb][0]), S_NEXT[m][qb][1]);                            \
                m_run[qb] = fmaxf(fmaxf(m_run[qb], S_NEXT[m][qb][2]), S_NEXT[m][qb][3]);                            \
            }                                                                                                       \
            _Pragma("unroll") for (int f = 0; f < NV; ++f)                                                          \
                if (Plan::vslot(f) == k) s16_lds_read(vfr[f], vt_a, S16_FRAG(f));                                   \
            _Pragma("unroll") for (int f = 0; f < KS; ++f)                                                          \
                if (Plan::kslot(f) == k) s16_lds_read(kfr[f], kt_a, S16_FRAG(f));                                   \
            __builtin_amdgcn_sched_barrier(0);                                                                      \
            if (EDGE && k == KS - 1 && edge) {                                                                      \
                _Pragma("unroll") for (int f = 0; f < NV; ++f) s16_lds_wait<0>(vfr[f]);                             \
                mask_v(vfr, S16_LIVE(I));                                                                           \
            }                                                                                                       \
        }                                                                                                           \
        if (TRACK) {                                                                                                \
            mx[0] = m_run[0];                                                                                       \
            mx[1] = m_run[1];                                                                                       \
            vote = __any(fmaxf(mx[0], mx[1]) > S16_RESCALE_SLACK                                                    \
                         || (NO_REF && ((mref[0] == -INFINITY && mx[0] != -INFINITY) || (mref[1] == -INFINITY && mx[1] != -INFINITY)))); \
        }                                                                                                           \
        if (PERIOD == 1 || BAR == 1 || (BAR == 2 && RingPlan::barrier_after((I) - vb))) {                           \
            if constexpr (G == 1) {                                                                                 \
                s16_wait_vmcnt<(PF - LAND) * LPW>();                                                                \
                __builtin_amdgcn_s_barrier();                                                                       \
            } else {                                                                                                \
                group_handover(kfr);                                                                                \
            }                                                                                                       \
        }                                                                                                           \
    }

    int next_edge = s16_next_edge(vb - 1, n0, n01, T, dead);
    bool vote = false;
    int i = vb;
    while (i < v_end) {
        while (i < v_end && (((i - vb) & 1) || i + 1 >= v_end || i == next_edge || i + 1 == next_edge)) {
            S16_STEP(i, sA, sB, 1, 2)
#pragma unroll
            for (int m = 0; m < 2; ++m)
#pragma unroll
                for (int qb = 0; qb < 2; ++qb) sA[m][qb] = sB[m][qb];
            ++i;
        }
        for (int cnt = (min(v_end, next_edge) - i) >> 1; cnt > 0; --cnt) {
            S16_STEP(i, sA, sB, 0, 0)
            S16_STEP(i + 1, sB, sA, 0, 1)
            i += 2;
        }
    }
#undef S16_STEP
#undef S16_PIN
#undef S16_PHYS_KB
#undef S16_LIVE
    __builtin_amdgcn_s_waitcnt(0);               // no load may still be writing LDS or registers past this point
#pragma unroll
    for (int qb = 0; qb < 2; ++qb) {
        st.l[qb] = lsum[qb][0] + lsum[qb][1];
        st.m[qb] = mref[qb];
    }
    return true;
}

// A wave without queries (a chunk's short last tile) still owes its workgroup its share of the direct-to-LDS loads,
// with the same waits and the same number of barriers.
template <int D, typename Gate>
__device__ __forceinline__ bool s16_segment_loads_only(const AttnParams& p, const AttnChunk& ch, int tid, int head, int vb, int ve, char* lds, Gate gate) {
    constexpr int KS = D / 16, NV = D / 16;
    constexpr int KB_BYTES = KBLOCK * D * 2, STAGE_BYTES = 2 * KB_BYTES;
    constexpr int NS = RingPlan::STAGES, NW = 8, LPW = (KS + NV) / NW, PF = RingPlan::AHEAD, LAND = RingPlan::LANDED;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int n_ranges = ch.n_ranges;
    const int rs0 = ch.rs[0], re0 = ch.re[0];
    int rs1 = ch.rs[1], re1 = ch.re[1], rs2 = ch.rs[2];
    if (n_ranges < 2) rs1 = re1 = 0;
    if (n_ranges < 3) rs2 = 0;
    const int kb0 = rs0 / KBLOCK, ke0 = (re0 + KBLOCK - 1) / KBLOCK;
    const int kb1 = rs1 / KBLOCK, ke1 = (re1 + KBLOCK - 1) / KBLOCK;
    const int kb2 = rs2 / KBLOCK;
    const int n0 = ke0 - kb0, n01 = n0 + (ke1 - kb1);
    const char* kbase = reinterpret_cast<const char*>(p.k_cache + head * p.head_stride);
    const char* vbase = reinterpret_cast<const char*>(p.v_cache + head * p.head_stride);
    const unsigned lane_off = lane * 16, k_load_off = s16_k_load_offset(lane);
    auto issue_loads = [&](int v, int stage) {
        const int kb = v + s16_pick(v, n0, n01, kb0, kb1 - n0, kb2 - n01);
        const int64_t kb_off = int64_t(kb) * KB_BYTES;
#pragma unroll
        for (int l = 0; l < LPW; ++l) {
            const int f = wave + NW * l;
            const char* src = (f < KS ? kbase + f * 1024 + k_load_off : vbase + (f - KS) * 1024 + lane_off) + kb_off;
            char* dst = lds + stage * STAGE_BYTES + f * 1024;
            __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)(src),
                                             (__attribute__((address_space(3))) void*)(dst), 16, 0, 0);
        }
    };
#pragma unroll
    for (int j = 0; j < PF; ++j) issue_loads(min(vb + j, ve - 1), (vb + j) & (NS - 1));
    s16_wait_vmcnt<(PF - LAND) * LPW>();
    if (!gate()) {
        __builtin_amdgcn_s_waitcnt(0);
        return false;
    }
    for (int i = vb; i < ve; ++i) {
        issue_loads(min(i + PF, ve - 1), (i + PF) & (NS - 1));
        if (RingPlan::barrier_after(i - vb)) {
            s16_wait_vmcnt<(PF - LAND) * LPW>();
            __builtin_amdgcn_s_barrier();
        }
    }
    __builtin_amdgcn_s_waitcnt(0);
    return true;
}

// The same for a wave of a key group (G > 1) that has no queries, or whose group has no kblocks (loads nothing then).
template <int D, int G, typename Gate>
__device__ __forceinline__ bool s16_group_idle(const AttnParams& p, const AttnChunk& ch, int tid, int head, int vb, int ve, int n_steps, char* lds, Gate gate) {
    using GR = GroupRing<D, G>;
    constexpr int KS = D / 16, NF = 2 * KS, NW = 8 / G, PERIOD = GR::PERIOD, DEPTH = GR::DEPTH, LPW = PERIOD * NF / NW;
    constexpr int KB_BYTES = KBLOCK * D * 2;
    if constexpr (NW == 1) {                     // a ring of its own: nobody waits for this wave
        if constexpr (Gate::STOPS) return gate();
        return true;
    }
    const int lane = tid & 63;
    const int wave_wg = __builtin_amdgcn_readfirstlane(tid >> 6), wave = wave_wg % NW;
    lds += (wave_wg / NW) * GR::BYTES;
    const int n_ranges = ch.n_ranges;
    const int rs0 = ch.rs[0], re0 = ch.re[0];
    int rs1 = ch.rs[1], re1 = ch.re[1], rs2 = ch.rs[2];
    if (n_ranges < 2) rs1 = re1 = 0;
    if (n_ranges < 3) rs2 = 0;
    const int kb0 = rs0 / KBLOCK, ke0 = (re0 + KBLOCK - 1) / KBLOCK;
    const int kb1 = rs1 / KBLOCK, ke1 = (re1 + KBLOCK - 1) / KBLOCK;
    const int kb2 = rs2 / KBLOCK;
    const int n0 = ke0 - kb0, n01 = n0 + (ke1 - kb1);
    const char* kbase = reinterpret_cast<const char*>(p.k_cache + head * p.head_stride);
    const char* vbase = reinterpret_cast<const char*>(p.v_cache + head * p.head_stride);
    const unsigned lane_off = lane * 16, k_load_off = s16_k_load_offset(lane);
    auto issue_period = [&](int first) {
        if (ve <= vb) return;
#pragma unroll
        for (int l = 0; l < LPW; ++l) {
            const int j = (NW * l) / NF, part = (NW * l) % NF;
            const bool is_k = part < KS;
            const int rel = first + j + (is_k ? 2 : 0);
            const int v = min(vb + rel, ve - 1), kb = v + s16_pick(v, n0, n01, kb0, kb1 - n0, kb2 - n01);
            const int fr = (is_k ? part : part - KS) + wave;
            const char* src = (is_k ? kbase + k_load_off : vbase + lane_off) + int64_t(kb) * KB_BYTES + fr * 1024;
            char* dst = lds + ((is_k ? 0 : DEPTH) + (rel & (DEPTH - 1))) * KB_BYTES + fr * 1024;
            __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)(src),
                                             (__attribute__((address_space(3))) void*)(dst), 16, 0, 0);
        }
    };
    issue_period(0);
    s16_wait_vmcnt<0>();
    if (!gate()) return false;
    for (int r = 0; r + PERIOD <= n_steps; r += PERIOD) {
        issue_period(r + PERIOD);
        s16_wait_vmcnt<0>();
        __builtin_amdgcn_s_barrier();
    }
    if (n_steps % PERIOD != 0) issue_period(n_steps / PERIOD * PERIOD + PERIOD);
    __builtin_amdgcn_s_waitcnt(0);
    return true;
}

// 16 dq + 4 g + j, j = 0..3, of a row's unnormalised output (with reference m and row sum l) to where the call wants it
template <int D, bool LSE>
__device__ __forceinline__ void s16_store_unit(const AttnParams& p, int head, int row, int dq, int g, const f32x4& o, float m, float l) {
    const float inv = 1.0f / l;
    const u32x2 w = {s16_pack_bf16(o[0] * inv, o[1] * inv), s16_pack_bf16(o[2] * inv, o[3] * inv)};
    uint16_t* dst = p.out_frag != nullptr        // uniform
        ? p.out_frag + op_frag_offset(row, head * (D / 32) + (dq >> 1), g, p.H * (D / 32)) + (dq & 1) * 4
        : p.out + (int64_t(row) * p.H + head) * D + dq * 16 + g * 4;
    *reinterpret_cast<u32x2*>(dst) = w;
    if constexpr (LSE) {
        if (p.lse != nullptr && dq == 0 && g == 0) p.lse[int64_t(head) * p.lse_stride + row] = m + __builtin_amdgcn_logf(l);
        if (p.out32 != nullptr) *reinterpret_cast<f32x4*>(p.out32 + (int64_t(row) * p.H + head) * D + dq * 16 + g * 4) = o * inv;
    }
}

// Share `split` of `splits` of a tile's keys, or (one split) all of them, dealt to G groups of 8 / G waves: kblocks
// [T j / G, T (j + 1) / G) to group j (with splits: the split's G of the G * splits shares).  Each group's result is relative to
// its own reference; they meet in LDS (the rings' memory), where s16_add_groups adds up what a wave asks for.  This wave's rows
// begin at q0.
template <int D, bool QSCALE, int SCHED, int G, typename Gate>
__device__ __forceinline__ bool s16_groups(const AttnParams& p, const AttnChunk& ch, int tid, int head, int q0, int split, int splits, char* lds,
                                           const float2* shift_cs, float2 (*ml)[2][16], Gate gate, S16Touch touch) {
    constexpr int NW = 8 / G, UNITS = D / 16 * 2;                // (dq, qb) blocks of a wave's O^T
    static_assert(UNITS % G == 0, "the O^T blocks must split over the groups");
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int group = wave / NW;
    const int lane = tid & 63, n = lane & 15, g = lane >> 4;
    const int T = ch.n_kblocks;
    int vb = T * group / G, ve = T * (group + 1) / G, n_steps = (T + G - 1) / G;
    if (splits > 1) {                            // uniform (and three divisions, in front of everything else)
        const int shares = G * splits, share = G * split + group;
        vb = T * share / shares;
        ve = T * (share + 1) / shares;
        n_steps = (T + shares - 1) / shares;
    }
    const bool works = q0 < ch.q_end && ve > vb;
    S16State<D> st;
    constexpr bool TOUCH = GroupRing<D, G>::TOUCHES && !QSCALE;  // (a prompt's keys are few)
    if (!(works ? (TOUCH && touch.every > 0
                       ? s16_segment<D, QSCALE, SCHED, G, TOUCH>(p, ch, tid, head, q0, vb, ve, n_steps, lds, st, shift_cs, gate, touch)
                       : s16_segment<D, QSCALE, SCHED, G, false>(p, ch, tid, head, q0, vb, ve, n_steps, lds, st, shift_cs, gate))
                : s16_group_idle<D, G>(p, ch, tid, head, vb, ve, n_steps, lds, gate)))
        return false;
    if constexpr ((SCHED & 8) != 0) {
        const bool ran_away = works && !(st.l[0] < S16_FIXED_REF_LIMIT && st.l[1] < S16_FIXED_REF_LIMIT);
        if (__syncthreads_or(ran_away)) {
            if (works) s16_segment<D, QSCALE, SCHED & ~8, G, false>(p, ch, tid, head, q0, vb, ve, n_steps, lds, st, shift_cs, typename Gate::Again{});
            else s16_group_idle<D, G>(p, ch, tid, head, vb, ve, n_steps, lds, typename Gate::Again{});
        }
    }
    if (!works) {
#pragma unroll
        for (int qb = 0; qb < 2; ++qb) {
            st.l[qb] = 0.f;
            st.m[qb] = -INFINITY;
#pragma unroll
            for (int dq = 0; dq < D / 16; ++dq) st.o[dq][qb] = f32x4{0.f, 0.f, 0.f, 0.f};
        }
    }
    __syncthreads();                             // every group has left its ring
    f32x4* part = reinterpret_cast<f32x4*>(lds);                 // [wave][unit][lane]
#pragma unroll
    for (int qb = 0; qb < 2; ++qb) {
        float l = st.l[qb];
        l += __shfl_xor(l, 16);
        l += __shfl_xor(l, 32);
        if (g == 0) ml[wave][qb][n] = make_float2(st.m[qb], l);
#pragma unroll
        for (int dq = 0; dq < D / 16; ++dq) part[(wave * UNITS + dq * 2 + qb) * 64 + lane] = st.o[dq][qb];
    }
    __syncthreads();
    return true;
}

// Unit u = (dq, qb) of the tile's O^T blocks over all groups, relative to reference m: weights 2^(m_j - max m)
template <int D, int G>
__device__ __forceinline__ void s16_add_groups(int tid, const char* lds, const float2 (*ml)[2][16], int u, bool may_be_weightless, float& m, float& l, f32x4& o) {
    constexpr int NW = 8 / G, UNITS = D / 16 * 2;
    const int rb = __builtin_amdgcn_readfirstlane(tid >> 6) % NW;
    const int lane = tid & 63, n = lane & 15, qb = u & 1;
    const f32x4* part = reinterpret_cast<const f32x4*>(lds);
    m = -INFINITY;
    l = 0.f;
    o = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int j = 0; j < G; ++j) m = fmaxf(m, ml[j * NW + rb][qb][n].x);
    const float base = may_be_weightless && m == -INFINITY ? 0.f : m;
#pragma unroll
    for (int j = 0; j < G; ++j) {
        const float2 s = ml[j * NW + rb][qb][n];
        const float a = __builtin_amdgcn_exp2f(s.x - base);
        l = __builtin_fmaf(s.y, a, l);
        const f32x4 x = part[((j * NW + rb) * UNITS + u) * 64 + lane];
#pragma unroll
        for (int e = 0; e < 4; ++e) o[e] = __builtin_fmaf(x[e], a, o[e]);
    }
}

// Kblocks [vb, ve) for the wave's rows from q0 on, all eight waves walking through one ring.
template <int D, bool QSCALE, int SCHED, typename Gate>
__device__ __forceinline__ bool s16_whole(const AttnParams& p, const AttnChunk& ch, int tid, int head, int q0, int vb, int ve, char* lds, S16State<D>& st,
                                          const float2* shift_cs, Gate gate) {
    // wave-uniform: a wave without rows in the chunk's last tile only takes its share of the loads and barriers
    const bool has_rows = q0 < ch.q_end;
    if (!(has_rows ? s16_segment<D, QSCALE, SCHED, 1, false>(p, ch, tid, head, q0, vb, ve, ve - vb, lds, st, shift_cs, gate)
                   : s16_segment_loads_only<D>(p, ch, tid, head, vb, ve, lds, gate)))
        return false;
    if constexpr ((SCHED & 8) != 0) {
        // the pass above kept its first reference: fine unless some row's sum ran away (a score far above the first
        // kblock's maximum); then the whole workgroup (the waves share the ring and its barriers) takes the tile again
        // with the reference followed.  The barrier inside the vote also ends every wave's reads of the first pass.
        const bool ran_away = has_rows && !(st.l[0] < S16_FIXED_REF_LIMIT && st.l[1] < S16_FIXED_REF_LIMIT);
        if (__syncthreads_or(ran_away)) {
            if (has_rows) s16_segment<D, QSCALE, SCHED & ~8, 1, false>(p, ch, tid, head, q0, vb, ve, ve - vb, lds, st, shift_cs, typename Gate::Again{});
            else s16_segment_loads_only<D>(p, ch, tid, head, vb, ve, lds, typename Gate::Again{});
        }
    }
    return true;
}

__device__ __forceinline__ void s16_shift_table(const AttnParams& p, const AttnChunk& ch, float2* shift_cs) {
    if (ch.sink_shift == 0) return;              // uniform over the workgroup
    if ((int)threadIdx.x < p.n_t) {
        double sn, cs;
        sincos(double(ch.sink_shift) * p.inv_freq_t[threadIdx.x], &sn, &cs);
        shift_cs[threadIdx.x] = make_float2(float(cs), float(sn));
    }
    __syncthreads();
}

// The partial results of a tile's splits, for the 16-row blocks [first, first + n_blocks) of the tile, added up in order.
// Bounded by latency and by the partials' way through the last-level cache.  False (for the whole workgroup, and for all of
// the tile's) if some split found no room for its partial result: nothing is written then.
template <int D, bool LSE>
__device__ __forceinline__ bool s16_merge(const AttnParams& p, const AttnChunk& ch, int tid, int head, int tile, int splits, int row0, int first,
                                          int n_blocks, int* slots) {
    constexpr int DQ = D / 16;
    const int lane = tid & 63, n = lane & 15, g = lane >> 4;
    if (tid < splits) slots[tid] = split_find(p.pool, (head * p.splits + tid) * p.n_tiles + tile, p.token);
    __syncthreads();
    bool all = true;
    for (int s = 0; s < splits; ++s) all = all && slots[s] >= 0;
    all = __builtin_amdgcn_readfirstlane(all);
    if (all) {
        for (int u = tid >> 6; u < n_blocks * DQ; u += S16_THREADS / 64) {
            const int blk = first + u / DQ, dq = u % DQ, row = row0 + (blk - first) * 16 + n;
            float m = -INFINITY, l = 0.f;
            f32x4 o = {0.f, 0.f, 0.f, 0.f};
            for (int s0 = 0; s0 < splits; s0 += 4) {
                float2 w[4];
                f32x4 x[4];
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const int slot = slots[min(s0 + e, splits - 1)];
                    w[e] = p.pool->ml[slot][blk * 16 + n];
                    x[e] = reinterpret_cast<const f32x4*>(p.pool->o[slot])[(blk * DQ + dq) * 64 + lane];
                }
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    if (s0 + e < splits) {
                        float a, b;
                        split_weights(m, l, w[e].x, w[e].y, a, b);
                        o = split_add(o, a, x[e], b);
                    }
            }
            if (row < ch.q_end) s16_store_unit<D, LSE>(p, head, row, dq, g, o, m, l);
        }
    }
    __syncthreads();                             // every read of the partial results has returned
    if (tid < splits && slots[tid] >= 0) split_release(p.pool, slots[tid]);
    return all;
}

// ---- one workgroup per (head, query tile): placement on the XCDs as in attn_stream.hip.  G: key groups
template <int D, bool QSCALE, bool LSE, int SCHED, int G>
__global__ __launch_bounds__(S16_THREADS) __attribute__((amdgpu_waves_per_eu(2, 2))) void ll_attn_stream16_kernel(const AttnParams p) {
    extern __shared__ __attribute__((aligned(16))) char lds[];
    __shared__ float2 shift_cs[64];
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int lane = tid & 63, n = lane & 15, g = lane >> 4;
    // The arguments lie in several cache lines; where a launch has one chunk, all that a workgroup needs of them is
    // fetched here in one go instead of one cold scalar load after another.
    AttnChunk ch = p.chunk[0];
    asm volatile("" ::"s"(ch.q_begin), "s"(ch.q_end), "s"(ch.tile_begin), "s"(ch.n_ranges), "s"(ch.rs[0]), "s"(ch.rs[1]), "s"(ch.rs[2]),
                 "s"(ch.re[0]), "s"(ch.re[1]), "s"(ch.re[2]), "s"(ch.n_kblocks), "s"(ch.sink_shift), "s"(ch.t_row));
    asm volatile("" ::"s"(p.q), "s"(p.k_cache), "s"(p.v_cache), "s"(p.head_stride), "s"(p.out), "s"(p.out_frag), "s"(p.t_table), "s"(p.row_cs), "s"(p.col_cs));
    const int xcd = blockIdx.x & 7;
    int head = -1, tile = 0, ci = -1;
    const int idx = blockIdx.x >> 3;
    if (p.n_groups == 0) {
        const int total = p.n_tiles * p.H;
        const int item = ((xcd * total + 7) >> 3) + idx;
        if (item < (((xcd + 1) * total + 7) >> 3)) {
            head = item / p.n_tiles;
            tile = item % p.n_tiles;
        }
    } else {
        if (!attn_placed_tile(p, xcd, idx, head, ci, tile)) head = -1;
    }
    if (head < 0) return;                        // uniform over the workgroup
    if (p.n_chunks > 1) {
        if (ci < 0)
            for (ci = 0; ci + 1 < p.n_chunks && tile >= p.chunk[ci + 1].tile_begin;) ++ci;
        ch = p.chunk[ci];
    }
    const int row0 = ch.q_begin + (tile - ch.tile_begin) * (256 / G);
    s16_shift_table(p, ch, shift_cs);
    if constexpr (G > 1) {
        __shared__ float2 ml[8][2][16];          // (reference, row sum) per wave, query block and column
        constexpr int NW = 8 / G, PER_WAVE = D / 8 / G;
        const int q0 = row0 + wave % NW * 32;
        S16Touch touch;
        if constexpr (!QSCALE) touch = s16_take_turns<D, G>(ch, p.H, row0, tile, idx, p.n_groups == 0 ? p.n_tiles * p.H : 0);
        s16_groups<D, QSCALE, SCHED, G>(p, ch, tid, head, q0, 0, 1, lds, shift_cs, ml, S16Unsplit{}, touch);
        if (q0 >= ch.q_end) return;
#pragma unroll
        for (int i = 0; i < PER_WAVE; ++i) {
            const int u = wave / NW * PER_WAVE + i, row = q0 + 16 * (u & 1) + n;
            float m, l;
            f32x4 o;
            s16_add_groups<D, G>(tid, lds, ml, u, false, m, l, o);
            if (row < ch.q_end) s16_store_unit<D, LSE>(p, head, row, u >> 1, g, o, m, l);
        }
        return;
    }
    const int row_block = ((wave & 3) << 1) | (wave >> 2);      // waves w and w + 4 (one SIMD) take neighbouring blocks
    const int q0 = row0 + row_block * 32;
    S16State<D> st;
    s16_whole<D, QSCALE, SCHED>(p, ch, tid, head, q0, 0, ch.n_kblocks, lds, st, shift_cs, S16Unsplit{});
    if (q0 >= ch.q_end) return;

    // out[row][head][16 dq + 4 g + j] = O^T block (dq, qb) register j, divided by the row sum
#pragma unroll
    for (int qb = 0; qb < 2; ++qb) {
        float l = st.l[qb];
        l += __shfl_xor(l, 16);
        l += __shfl_xor(l, 32);
        const float inv = 1.0f / l;
        const int row = q0 + 16 * qb + n;
        if (row < ch.q_end) {
            if (p.out_frag != nullptr) {         // uniform: the output projection's operand, 1 KB per store instruction
                const int n_ksteps = p.H * (D / 32);
#pragma unroll
                for (int t = 0; t < D / 32; ++t) {
                    const f32x4 a = st.o[2 * t][qb], b = st.o[2 * t + 1][qb];
                    const u32x4 w = {s16_pack_bf16(a[0] * inv, a[1] * inv), s16_pack_bf16(a[2] * inv, a[3] * inv),
                                     s16_pack_bf16(b[0] * inv, b[1] * inv), s16_pack_bf16(b[2] * inv, b[3] * inv)};
                    *reinterpret_cast<u32x4*>(p.out_frag + op_frag_offset(row, head * (D / 32) + t, g, n_ksteps)) = w;
                }
                continue;
            }
            uint16_t* dst = p.out + (int64_t(row) * p.H + head) * D + g * 4;
#pragma unroll
            for (int dq = 0; dq < D / 16; ++dq) {
                const f32x4 o = st.o[dq][qb];
                u32x2 w = {s16_pack_bf16(o[0] * inv, o[1] * inv), s16_pack_bf16(o[2] * inv, o[3] * inv)};
                *reinterpret_cast<u32x2*>(dst + dq * 16) = w;
            }
            if constexpr (LSE) {                 // for the backward pass of the train-time rule (see attn_stream.hip)
                if (p.lse != nullptr && g == 0)
                    p.lse[int64_t(head) * p.lse_stride + row] = st.m[qb] + __builtin_amdgcn_logf(l);
                if (p.out32 != nullptr) {
                    float* d32 = p.out32 + (int64_t(row) * p.H + head) * D + g * 4;
#pragma unroll
                    for (int dq = 0; dq < D / 16; ++dq) *reinterpret_cast<f32x4*>(d32 + dq * 16) = st.o[dq][qb] * inv;
                }
            }
        }
    }
}

// ---- the launches of tiles whose keys are split: several workgroups per tile, one share of its keys each, and their merge, with
// the tile's rows in slices
struct S16SplitTile {
    SplitPlace at;                               // (part: split, or slice of the merge)
    AttnChunk ch;
    int row0, splits, slice_rows, rows;
};
template <int G>
__device__ __forceinline__ S16SplitTile s16_split_tile(const AttnParams& p) {
    S16SplitTile t;
    t.ch = p.chunk[0];                           // (in one go, as above)
    asm volatile("" ::"s"(t.ch.q_begin), "s"(t.ch.q_end), "s"(t.ch.tile_begin), "s"(t.ch.n_ranges), "s"(t.ch.rs[0]), "s"(t.ch.rs[1]), "s"(t.ch.rs[2]),
                 "s"(t.ch.re[0]), "s"(t.ch.re[1]), "s"(t.ch.re[2]), "s"(t.ch.n_kblocks), "s"(t.ch.sink_shift), "s"(t.ch.t_row));
    asm volatile("" ::"s"(p.q), "s"(p.k_cache), "s"(p.v_cache), "s"(p.head_stride), "s"(p.out), "s"(p.t_table), "s"(p.row_cs), "s"(p.col_cs), "s"(p.splits), "s"(p.per_tile),
                 "s"(p.pool), "s"(p.token));
    t.at = split_place(p);
    if (p.n_chunks > 1) {
        int ci = 0;
        while (ci + 1 < p.n_chunks && t.at.tile >= p.chunk[ci + 1].tile_begin) ++ci;
        t.ch = p.chunk[ci];
    }
    t.row0 = t.ch.q_begin + (t.at.tile - t.ch.tile_begin) * (256 / G);
    t.splits = min(p.splits, max(1, t.ch.n_kblocks / G));                        // no more than the chunk has keys for
    t.slice_rows = 16 * p.slice_blocks;
    t.rows = min(256 / G, t.ch.q_end - t.row0);
    return t;
}
// Share `share` of the tile: false if the gate stopped it, else what the wave's unit i = 0 .. PER_WAVE - 1 is (s16_share_unit).
template <int D, int SCHED, int G, typename Gate>
__device__ __forceinline__ bool s16_share(const AttnParams& p, const S16SplitTile& t, int tid, int q0, int share, char* lds, const float2* shift_cs,
                                          float2 (*ml)[2][16], S16State<D>& st, Gate gate) {
    if constexpr (G > 1) return s16_groups<D, false, SCHED, G>(p, t.ch, tid, t.at.head, q0, share, t.splits, lds, shift_cs, ml, gate, S16Touch{});
    if (!s16_whole<D, false, SCHED>(p, t.ch, tid, t.at.head, q0, t.ch.n_kblocks * share / t.splits, t.ch.n_kblocks * (share + 1) / t.splits, lds, st, shift_cs, gate))
        return false;
#pragma unroll
    for (int qb = 0; qb < 2; ++qb) {
        st.l[qb] += __shfl_xor(st.l[qb], 16);
        st.l[qb] += __shfl_xor(st.l[qb], 32);
    }
    return true;
}
template <int D, int G>
__device__ __forceinline__ void s16_share_unit(int tid, const char* lds, const float2 (*ml)[2][16], const S16State<D>& st, int i, int u, float& m, float& l, f32x4& o) {
    if constexpr (G > 1) {
        s16_add_groups<D, G>(tid, lds, ml, u, true, m, l, o);    // a share may hold no key with weight, a tile does (or is NaN)
    } else {
        m = st.m[i & 1];
        l = st.l[i & 1];
        o = st.o[i >> 1][i & 1];
    }
}
template <int G>
__device__ __forceinline__ int s16_row_block(int wave) { return G > 1 ? wave % (8 / G) : ((wave & 3) << 1) | (wave >> 2); }    // (as in the kernel above)

// One share of a tile whose partial results are not all there, added to the sums in a space of the pool; the last one stores the rows.
template <int D, bool LSE, int SCHED, int G>
__device__ __forceinline__ bool s16_next_share(const AttnParams& p, char* lds, const float2* shift_cs, float2 (*ml)[2][16], int space, int share,
                                               float (&m_sum)[2], float (&l_sum)[2]) {
    constexpr int DQ = D / 16, NW = 8 / G, PER_WAVE = 2 * DQ / G;
    int tid = threadIdx.x;
    asm volatile("" : "+v"(tid));                // (as attn_params_again)
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int lane = tid & 63, n = lane & 15, g = lane >> 4;
    const S16SplitTile t = s16_split_tile<G>(p);
    const int row_block = s16_row_block<G>(wave), q0 = t.row0 + row_block * 32, u0 = G > 1 ? wave / NW * PER_WAVE : 0;
    S16State<D> st;
    s16_share<D, SCHED, G>(p, t, tid, q0, share, lds, shift_cs, ml, st, S16NextShare{});
    if (q0 < t.ch.q_end) {
        float a[2] = {}, b[2] = {};
#pragma unroll
        for (int i = 0; i < PER_WAVE; ++i) {
            const int u = u0 + i, dq = u >> 1, row = q0 + 16 * (u & 1) + n;
            float m, l;
            f32x4 o;
            s16_share_unit<D, G>(tid, lds, ml, st, i, u, m, l, o);
            f32x4* at = reinterpret_cast<f32x4*>(p.pool->o[space]) + ((row_block * 2 + (u & 1)) * DQ + dq) * 64 + lane;
            if (i < 2) split_weights(m_sum[i], l_sum[i], m, l, a[i], b[i]);
            const f32x4 before = share > 0 ? *at : f32x4{0.f, 0.f, 0.f, 0.f};
            o = split_add(before, a[i & 1], o, b[i & 1]);
            if (share + 1 < t.splits) *at = o;
            else if (row < t.ch.q_end) s16_store_unit<D, LSE>(p, t.at.head, row, dq, g, o, m_sum[i & 1], l_sum[i & 1]);
            asm volatile("" ::: "memory");       // one unit's sums in registers at a time
        }
    }
    __syncthreads();                             // the groups' sums have been read, and the sums over shares too
    return share + 1 < t.splits;
}

// The gate of a workgroup that needs a slot: it claims one with its first loads, looks at the answer behind them, and leaves if
// there is none, since what it would compute is the merge's then.  us a call of 1560 rows x 12 x 128, four streams making such
// calls: 320 where workgroups looked for a slot when they had their result, 209 to 230 so; one stream 167 either way.
struct S16Claim {
    static constexpr bool STOPS = true;
    using Again = S16Barrier<2>;
    const AttnParams& p;
    int* slot;
    int item, readers;                           // readers 0: needs none
    unsigned long long seen;                     // thread 0: what the claim of the first candidate found
    __device__ __forceinline__ bool operator()() const {
        unsigned long long found = seen;
        asm volatile("" : "+v"(found));          // looked at here: the compiler would compare it, and wait for it, where it was asked for
        if (threadIdx.x == 0 && readers > 0) *slot = found == 0 ? split_candidate(item, 0) : split_claim(p.pool, item, p.token, readers, 1);
        __syncthreads();
        return readers == 0 || __builtin_amdgcn_readfirstlane(*slot) >= 0;
    }
};
template <int D, bool LSE, int SCHED, int G>
__global__ __launch_bounds__(S16_THREADS) __attribute__((amdgpu_waves_per_eu(2, 2))) void ll_attn_split16_kernel(const AttnParams p) {
    constexpr int DQ = D / 16, NW = 8 / G, PER_WAVE = 2 * DQ / G;
    extern __shared__ __attribute__((aligned(16))) char lds[];
    __shared__ float2 shift_cs[64];
    __shared__ float2 ml[G > 1 ? 8 : 1][2][16];
    __shared__ int slot_lds;
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int lane = tid & 63, n = lane & 15, g = lane >> 4;
    const S16SplitTile t = s16_split_tile<G>(p);
    if (t.at.item < 0 || t.at.part >= t.splits) return;          // uniform, as all of this
    const int readers = t.splits > 1 ? (t.rows + t.slice_rows - 1) / t.slice_rows : 0;
    S16Claim claim{p, &slot_lds, t.at.item, readers, 0};
    s16_shift_table(p, t.ch, shift_cs);          // (before the claim: its load would wait for that)
    if (tid == 0 && readers > 0) claim.seen = split_try(p.pool, t.at.item, 0, p.token, readers);
    const int row_block = s16_row_block<G>(wave), q0 = t.row0 + row_block * 32, u0 = G > 1 ? wave / NW * PER_WAVE : 0;
    S16State<D> st;
    if (!s16_share<D, SCHED, G>(p, t, tid, q0, t.at.part, lds, shift_cs, ml, st, claim) || q0 >= t.ch.q_end) return;
    float m, l;
    f32x4 o;
    if (readers == 0) {                          // (a loop of its own: the units' reads from LDS overlap)
#pragma unroll
        for (int i = 0; i < PER_WAVE; ++i) {
            const int u = u0 + i, row = q0 + 16 * (u & 1) + n;
            s16_share_unit<D, G>(tid, lds, ml, st, i, u, m, l, o);
            if (row < t.ch.q_end) s16_store_unit<D, LSE>(p, t.at.head, row, u >> 1, g, o, m, l);
        }
        return;
    }
    const int slot = __builtin_amdgcn_readfirstlane(slot_lds);
#pragma unroll
    for (int i = 0; i < PER_WAVE; ++i) {
        const int u = u0 + i, blk = row_block * 2 + (u & 1);
        s16_share_unit<D, G>(tid, lds, ml, st, i, u, m, l, o);
        reinterpret_cast<f32x4*>(p.pool->o[slot])[(blk * DQ + (u >> 1)) * 64 + lane] = o;
        if (u < 2 && g == 0) p.pool->ml[slot][blk * 16 + n] = make_float2(m, l);
    }
}

template <int D, bool LSE, int SCHED, int G>
__global__ __launch_bounds__(S16_THREADS) __attribute__((amdgpu_waves_per_eu(2, 2))) void ll_attn_merge16_kernel(const AttnParams p) {
    extern __shared__ __attribute__((aligned(16))) char lds[];
    __shared__ float2 shift_cs[64];
    __shared__ float2 ml[G > 1 ? 8 : 1][2][16];
    __shared__ int slots[MAX_SPLITS];
    const int tid = threadIdx.x;
    const S16SplitTile t = s16_split_tile<G>(p);
    const int slice = t.at.part, first = slice * p.slice_blocks;
    // (one share: its workgroup has stored the finished rows, maybe over the queries)
    if (t.at.item < 0 || t.splits == 1 || slice * t.slice_rows >= t.rows) return;
    if (s16_merge<D, LSE>(p, t.ch, tid, t.at.head, t.at.tile, t.splits, t.row0 + slice * t.slice_rows, first, min(p.slice_blocks, 16 / G - first), slots)) return;
    // a partial result is missing: the first slice's workgroup takes the tile's shares one after another
    if (slice > 0) return;
    s16_shift_table(p, t.ch, shift_cs);
    if (tid == 0) slots[0] = split_take_space(p.pool, blockIdx.x);
    __syncthreads();
    const int space = __builtin_amdgcn_readfirstlane(slots[0]);
    float m_sum[2] = {-INFINITY, -INFINITY}, l_sum[2] = {0.f, 0.f};             // over the shares, by query block
    int share = 0;
    while (__builtin_amdgcn_readfirstlane(s16_next_share<D, LSE, SCHED, G>(attn_params_again(), lds, shift_cs, ml, space, share, m_sum, l_sum))) ++share;
    if (tid == 0) split_leave_space(p.pool, space);
}

// Default schedule: exponentials of the second query block behind the S^T slots, and the reference kept fixed with
// the second, maximum-following pass as the fallback (SCHED 9).  The *_tracked variants follow the maximum throughout;
// the *_qrope variants (SCHED bit 4) take unrotated queries and turn them on load.
constexpr int S16_DEFAULT = 9, S16_TRACKED = 1;
#define S16_KERNEL(D, QS, LSE, SCHED, G) ll_attn_stream16_kernel<D, QS, LSE, SCHED, G>
#define S16_BY_GROUPS(kernel, D, LSE, SCHED) \
    {kernel<D, LSE, SCHED, 1>, kernel<D, LSE, SCHED, 2>, kernel<D, LSE, SCHED, 4>, D == 64 ? kernel<D, LSE, SCHED, (D == 64 ? 8 : 4)> : nullptr}
#define S16_SPLIT(D, LSE, SCHED) S16_BY_GROUPS(ll_attn_split16_kernel, D, LSE, SCHED), S16_BY_GROUPS(ll_attn_merge16_kernel, D, LSE, SCHED)
#define S16_ENTRY(name, D, QS, LSE, SCHED, ...)                                                                       \
    {name, D, 256, 8 * 2 * KBLOCK * D * 2, S16_KERNEL(D, QS, LSE, SCHED, 1), S16_THREADS, KBLOCK,                     \
     {S16_KERNEL(D, QS, LSE, SCHED, 2), S16_KERNEL(D, QS, LSE, SCHED, 4),                                             \
      D == 64 ? S16_KERNEL(D, QS, LSE, SCHED, (D == 64 ? 8 : 4)) : nullptr}, __VA_ARGS__}
// (the tracked variants are there to be compared with, one key group)
#define S16_ENTRY_WHOLE(name, D, QS, LSE, SCHED) \
    {name, D, 256, 8 * 2 * KBLOCK * D * 2, S16_KERNEL(D, QS, LSE, SCHED, 1), S16_THREADS, KBLOCK, {}}
const AttnVariant kStream16Variants[] = {
    S16_ENTRY("d128_stream16", 128, false, false, S16_DEFAULT, S16_SPLIT(128, false, S16_DEFAULT)),
    S16_ENTRY("d64_stream16", 64, false, false, S16_DEFAULT, S16_SPLIT(64, false, S16_DEFAULT)),
    S16_ENTRY("d128_stream16_qscale", 128, true, false, S16_DEFAULT, {}, {}),
    S16_ENTRY("d64_stream16_qscale", 64, true, false, S16_DEFAULT, {}, {}),
    S16_ENTRY("d128_stream16_lse", 128, false, true, S16_DEFAULT, S16_SPLIT(128, true, S16_DEFAULT)),
    S16_ENTRY("d64_stream16_lse", 64, false, true, S16_DEFAULT, S16_SPLIT(64, true, S16_DEFAULT)),
    S16_ENTRY_WHOLE("d128_stream16_tracked", 128, false, false, S16_TRACKED),
    S16_ENTRY_WHOLE("d64_stream16_tracked", 64, false, false, S16_TRACKED),
    S16_ENTRY("d128_stream16_qrope", 128, false, false, S16_DEFAULT | 16, S16_SPLIT(128, false, S16_DEFAULT | 16)),
    S16_ENTRY("d64_stream16_qrope", 64, false, false, S16_DEFAULT | 16, S16_SPLIT(64, false, S16_DEFAULT | 16)),
};
#undef S16_ENTRY
#undef S16_ENTRY_WHOLE
#undef S16_KERNEL
#undef S16_SPLIT
#undef S16_BY_GROUPS
const int kNumStream16Variants = sizeof(kStream16Variants) / sizeof(kStream16Variants[0]);

}  // namespace ll
