// ll_sink_window_attn / ll_recache_prefill on the GPU: flash-style attention of a
// chunk's rotated queries over the live token-slot ranges of the layer's cache
// (paper Sec. 3.3: sink + short window + current chunk; no mask inside the set).
//
// Formulation per wave: S^T = K Q^T and O^T = V^T P^T with the 32x32x16 bf16 MFMA, so
// that every lane owns ONE query column.  Row max and row sum of the softmax are then
// plain in-lane reductions over accumulator registers; the two lane halves of a query
// are reconciled only when the running reference maximum has to move.  The K and V
// tiles come from HBM already in MFMA-fragment order (see kernels.h), go through LDS
// as straight 16-byte copies and are shared by all waves of the workgroup.
//
// Softmax is computed in fp32 in the log2 domain: p = 2^(s*c - m), c = log2(e)/sqrt(D).
// m is a per-query reference that is raised only when a new score exceeds it by more
// than RESCALE_SLACK (then O and the row sum are rescaled); the final division by the
// row sum makes the result independent of the reference chosen.
#include "kernels.h"
#include "lds_plan.h"
#include "split.h"

#include <algorithm>
#include <atomic>
#include <vector>

namespace ll {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
typedef unsigned u32x2 __attribute__((ext_vector_type(2)));

constexpr float RESCALE_SLACK = 6.0f;     // log2 units: p stays below 2^6 between rescales

__device__ inline unsigned pack_bf16(float a, float b) {
    f32x2 v = {a, b};
    return __builtin_bit_cast(unsigned, __builtin_convertvector(v, bf16x2));
}

// D: head_dim.  QB: 32-query blocks per wave.  NW: waves per workgroup.  KT: kblocks per tile.
// OCC: waves per SIMD the register allocation must leave room for (several small workgroups per CU).
template <int D, int QB, int NW, int KT, int OCC = 1>
__global__ __launch_bounds__(NW * 64) __attribute__((amdgpu_waves_per_eu(OCC, 8))) void ll_attn_kernel(const AttnParams p) {
    constexpr int KS = D / 16;                  // MFMA k-steps of the QK^T product
    constexpr int DB = D / 32;                  // 32-row blocks of O^T
    constexpr int KB_BYTES = KBLOCK * D * 2;    // one kblock of K (or of V)
    constexpr int TILE_BYTES = KT * KB_BYTES;
    constexpr int NT = NW * 64;
    constexpr int QT = NW * QB * 32;            // query rows per workgroup
    constexpr int CPT = TILE_BYTES / 16 / NT;   // 16-byte chunks per thread per tile (K, same for V)
    static_assert(TILE_BYTES % (16 * NT) == 0, "tile must split evenly over the threads");

    extern __shared__ __attribute__((aligned(16))) char lds[];   // [2][K tile | V tile]

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int col = lane & 31, half = lane >> 5;

    // Workgroup -> (head, query tile).  Consecutive workgroup ids go round-robin over the
    // 8 XCDs; give each XCD a contiguous run of (head, tile) items so that workgroups that
    // stream the same head's K/V share one L2.
    const int total = p.n_tiles * p.H;
    const int per_xcd = (total + 7) >> 3;
    const int item = (blockIdx.x & 7) * per_xcd + (blockIdx.x >> 3);
    if (item >= total) return;
    const int head = item / p.n_tiles;
    const int tile = item % p.n_tiles;
    int ci = 0;
    while (ci + 1 < p.n_chunks && tile >= p.chunk[ci + 1].tile_begin) ++ci;
    const AttnChunk& ch = p.chunk[ci];
    const int q0 = ch.q_begin + (tile - ch.tile_begin) * QT + wave * (QB * 32);

    // Q^T fragments: lane (col, half) holds features 16*ks + 8*half + 0..7 of query q0 + 32n + col.
    bf16x8 qf[QB][KS];
#pragma unroll
    for (int n = 0; n < QB; ++n) {
        const int row = min(q0 + n * 32 + col, ch.q_end - 1);
        const uint16_t* src = p.q + (int64_t(row) * p.H + head) * D + half * 8;
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) qf[n][ks] = *reinterpret_cast<const bf16x8*>(src + ks * 16);
    }

    f32x16 o[QB][DB];
    float mref[QB], lsum[QB];
#pragma unroll
    for (int n = 0; n < QB; ++n) {
        mref[n] = -INFINITY;
        lsum[n] = 0.f;
#pragma unroll
        for (int db = 0; db < DB; ++db)
#pragma unroll
            for (int r = 0; r < 16; ++r) o[n][db][r] = 0.f;
    }

    const char* kbase = reinterpret_cast<const char*>(p.k_cache + head * p.head_stride);
    const char* vbase = reinterpret_cast<const char*>(p.v_cache + head * p.head_stride);
    const float c = p.scale_log2e;

    // Tile iterator over the ranges.
    int n_tiles_total = 0;
    for (int r = 0; r < ch.n_ranges; ++r)
        n_tiles_total += ((ch.re[r] + KBLOCK - 1) / KBLOCK - ch.rs[r] / KBLOCK + KT - 1) / KT;
    int rng = 0;
    int kb = ch.rs[0] / KBLOCK;                                   // first kblock of the current tile
    int kb_end = (ch.re[0] + KBLOCK - 1) / KBLOCK;                // end kblock of the current range

    u32x4 kreg[CPT], vreg[CPT];
    auto fetch = [&](int kblk) {
        const char* ks = kbase + int64_t(kblk) * KB_BYTES;
        const char* vs = vbase + int64_t(kblk) * KB_BYTES;
#pragma unroll
        for (int i = 0; i < CPT; ++i) {
            kreg[i] = *reinterpret_cast<const u32x4*>(ks + (tid + i * NT) * 16);
            vreg[i] = *reinterpret_cast<const u32x4*>(vs + (tid + i * NT) * 16);
        }
    };
    auto stash = [&](int buf) {
        char* kd = lds + buf * (2 * TILE_BYTES);
        char* vd = kd + TILE_BYTES;
#pragma unroll
        for (int i = 0; i < CPT; ++i) {
            *reinterpret_cast<u32x4*>(kd + (tid + i * NT) * 16) = kreg[i];
            *reinterpret_cast<u32x4*>(vd + (tid + i * NT) * 16) = vreg[i];
        }
    };

    fetch(kb);
    stash(0);
    __syncthreads();

    for (int it = 0; it < n_tiles_total; ++it) {
        // position of this tile, and of the next one
        const int cur_kb = kb, cur_end = kb_end, cur_rs = ch.rs[rng], cur_re = ch.re[rng];
        kb += KT;
        if (kb >= kb_end && rng + 1 < ch.n_ranges) {
            ++rng;
            kb = ch.rs[rng] / KBLOCK;
            kb_end = (ch.re[rng] + KBLOCK - 1) / KBLOCK;
        }
        const bool more = it + 1 < n_tiles_total;
        if (more) fetch(kb);

        const char* kt = lds + (it & 1) * (2 * TILE_BYTES);
        const char* vt = kt + TILE_BYTES;
#pragma unroll
        for (int kbi = 0; kbi < KT; ++kbi) {
            const int kabs = cur_kb + kbi;
            if (kabs >= cur_end) break;                           // tile reaches past its range
            const int key0 = kabs * KBLOCK;
            const bool edge = key0 < cur_rs || key0 + KBLOCK > cur_re;

            // S^T = K Q^T for 32 keys x (QB*32) queries
            f32x16 s[QB];
#pragma unroll
            for (int n = 0; n < QB; ++n)
#pragma unroll
                for (int r = 0; r < 16; ++r) s[n][r] = 0.f;
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) {
                const bf16x8 a = *reinterpret_cast<const bf16x8*>(kt + kbi * KB_BYTES + ks * 1024 + lane * 16);
#pragma unroll
                for (int n = 0; n < QB; ++n)
                    s[n] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, qf[n][ks], s[n], 0, 0, 0);
            }
            // register r of a lane is key key0 + 16*(r/8) + 8*half + r%8
            unsigned live = 0xFFFFu;                              // bit r: key of register r is in range
            if (edge) {
                live = 0;
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    const int key = key0 + 16 * (r >> 3) + 8 * half + (r & 7);
                    if (key >= cur_rs && key < cur_re) live |= 1u << r;
                }
#pragma unroll
                for (int n = 0; n < QB; ++n)
#pragma unroll
                    for (int r = 0; r < 16; ++r)
                        if (!((live >> r) & 1)) s[n][r] = -INFINITY;
            }

            unsigned pb[QB][2][4];                                // P^T fragments, bf16 pairs
#pragma unroll
            for (int n = 0; n < QB; ++n) {
                float mx = s[n][0];
#pragma unroll
                for (int r = 1; r < 16; ++r) mx = fmaxf(mx, s[n][r]);
                mx *= c;
                if (__any(mx > mref[n] + RESCALE_SLACK)) {
                    const float both = fmaxf(mx, __shfl_xor(mx, 32));
                    const float mnew = fmaxf(mref[n], both);
                    const float alpha = (mref[n] == -INFINITY) ? 0.f : __builtin_amdgcn_exp2f(mref[n] - mnew);
                    mref[n] = mnew;
                    lsum[n] *= alpha;
#pragma unroll
                    for (int db = 0; db < DB; ++db)
#pragma unroll
                        for (int r = 0; r < 16; ++r) o[n][db][r] *= alpha;
                }
                float pr[16];
                float acc = 0.f;
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    pr[r] = __builtin_amdgcn_exp2f(__builtin_fmaf(s[n][r], c, -mref[n]));
                    acc += pr[r];
                }
                lsum[n] += acc;
#pragma unroll
                for (int t = 0; t < 2; ++t)
#pragma unroll
                    for (int e = 0; e < 4; ++e) pb[n][t][e] = pack_bf16(pr[8 * t + 2 * e], pr[8 * t + 2 * e + 1]);
            }

            // O^T += V^T P^T
#pragma unroll
            for (int t = 0; t < 2; ++t) {
#pragma unroll
                for (int db = 0; db < DB; ++db) {
                    u32x4 av = *reinterpret_cast<const u32x4*>(vt + kbi * KB_BYTES + (db * 2 + t) * 1024 + lane * 16);
                    if (edge) {                                   // dead slots may hold anything, even NaN
#pragma unroll
                        for (int e = 0; e < 4; ++e) {
                            const unsigned b0 = (live >> (8 * t + 2 * e)) & 1, b1 = (live >> (8 * t + 2 * e + 1)) & 1;
                            av[e] &= (b0 ? 0x0000FFFFu : 0u) | (b1 ? 0xFFFF0000u : 0u);
                        }
                    }
                    const bf16x8 a = __builtin_bit_cast(bf16x8, av);
#pragma unroll
                    for (int n = 0; n < QB; ++n) {
                        u32x4 bv = {pb[n][t][0], pb[n][t][1], pb[n][t][2], pb[n][t][3]};
                        o[n][db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, __builtin_bit_cast(bf16x8, bv), o[n][db], 0, 0, 0);
                    }
                }
            }
        }

        if (more) stash((it + 1) & 1);
        __syncthreads();
    }

    // out[row][head][32*db + 8*g + 4*half + i] = O^T register 4*g + i, divided by the row sum
#pragma unroll
    for (int n = 0; n < QB; ++n) {
        const float l = lsum[n] + __shfl_xor(lsum[n], 32);
        const float inv = 1.0f / l;
        const int row = q0 + n * 32 + col;
        if (row < ch.q_end) {
            if (p.out_frag != nullptr) {         // uniform: the output projection's operand (kernels.h)
                // features 32 db + 4 G + e and 32 db + 16 + 4 G + e of lane group G are registers 4 g + e of this
                // lane half for g = 0, 2 (G = half) and g = 1, 3 (G = half + 2)
                const int n_ksteps = p.H * DB;
#pragma unroll
                for (int db = 0; db < DB; ++db)
#pragma unroll
                    for (int hi = 0; hi < 2; ++hi) {
                        const int g0 = hi, g1 = hi + 2;
                        const u32x4 w = {pack_bf16(o[n][db][4 * g0] * inv, o[n][db][4 * g0 + 1] * inv),
                                         pack_bf16(o[n][db][4 * g0 + 2] * inv, o[n][db][4 * g0 + 3] * inv),
                                         pack_bf16(o[n][db][4 * g1] * inv, o[n][db][4 * g1 + 1] * inv),
                                         pack_bf16(o[n][db][4 * g1 + 2] * inv, o[n][db][4 * g1 + 3] * inv)};
                        *reinterpret_cast<u32x4*>(p.out_frag + op_frag_offset(row, head * DB + db, half + 2 * hi, n_ksteps)) = w;
                    }
                continue;
            }
            uint16_t* dst = p.out + (int64_t(row) * p.H + head) * D + half * 4;
#pragma unroll
            for (int db = 0; db < DB; ++db)
#pragma unroll
                for (int g = 0; g < 4; ++g) {
                    u32x2 w = {pack_bf16(o[n][db][4 * g] * inv, o[n][db][4 * g + 1] * inv),
                               pack_bf16(o[n][db][4 * g + 2] * inv, o[n][db][4 * g + 3] * inv)};
                    *reinterpret_cast<u32x2*>(dst + db * 32 + g * 8) = w;
                }
        }
    }
}

#define LL_VARIANT(D, QB, NW, KT)                                                              \
    { "d" #D "_q" #QB "x" #NW "_k" #KT, D, NW * QB * 32, 2 * 2 * KT * KBLOCK * D * 2,          \
      ll_attn_kernel<D, QB, NW, KT>, NW * 64, KBLOCK }

static const AttnVariant kSimpleVariants[] = {
    LL_VARIANT(128, 2, 4, 2),   // 1: 256 queries, 64-key tiles
    LL_VARIANT(128, 2, 4, 4),   // 2: 256 queries, 128-key tiles
    LL_VARIANT(128, 1, 4, 2),   // 3: 128 queries
    LL_VARIANT(128, 1, 8, 2),   // 4: 256 queries, 8 waves
    LL_VARIANT(64, 2, 4, 2),    // 5
    LL_VARIANT(64, 1, 4, 2),    // 6
    // 128 queries per workgroup and room for 2 or 3 workgroups per CU: for short key sets (cross-attention over a
    // prompt), where a workgroup's life is mostly the load of its queries and the store of its outputs
    { "d128_q1x4_k2_occ2", 128, 128, 2 * 2 * 2 * KBLOCK * 128 * 2, ll_attn_kernel<128, 1, 4, 2, 2>, 256, KBLOCK },   // 7
    { "d128_q1x4_k1_occ3", 128, 128, 2 * 2 * 1 * KBLOCK * 128 * 2, ll_attn_kernel<128, 1, 4, 1, 3>, 256, KBLOCK },   // 8
    { "d64_q1x4_k2_occ2", 64, 128, 2 * 2 * 2 * KBLOCK * 64 * 2, ll_attn_kernel<64, 1, 4, 2, 2>, 256, KBLOCK },       // 9
    { "d64_q1x4_k1_occ3", 64, 128, 2 * 2 * 1 * KBLOCK * 64 * 2, ll_attn_kernel<64, 1, 4, 1, 3>, 256, KBLOCK },       // 10
};
constexpr int kNumSimple = sizeof(kSimpleVariants) / sizeof(kSimpleVariants[0]);
static_assert(kNumSimple == 10, "attn_variant_short_keys names table positions 8 and 10");

// variant ids: 1..kNumSimple are the kernels of this file, then the software-pipelined kernels, then the
// kernels of the 8-bit cache, then the software-pipelined kernels on 16x16x32 MFMAs
static const AttnVariant* variant(int v) {
    if (v >= 1 && v <= kNumSimple) return &kSimpleVariants[v - 1];
    v -= kNumSimple;
    if (v >= 1 && v <= kNumStreamVariants) return &kStreamVariants[v - 1];
    v -= kNumStreamVariants;
    if (v >= 1 && v <= kNumFp8Variants) return &kFp8Variants[v - 1];
    v -= kNumFp8Variants;
    if (v >= 1 && v <= kNumStream16Variants) return &kStream16Variants[v - 1];
    return nullptr;
}
static int first_stream16() { return kNumSimple + kNumStreamVariants + kNumFp8Variants + 1; }
static bool is_stream16(int v) { return v >= first_stream16() && v < first_stream16() + kNumStream16Variants; }
int attn_variant_count() { return kNumSimple + kNumStreamVariants + kNumFp8Variants + kNumStream16Variants; }
const char* attn_variant_name(int v) { return variant(v) ? variant(v)->name : nullptr; }
// the software-pipelined kernels are the default: for the bf16 cache the form built on 16x16x32 MFMAs (faster than the
// 32x32x16 form at every shape measured: 3 to 5 % at head_dim 128, 1 % at 64)
int attn_variant_default(int D, int kblock) {
    if (kblock == KBLOCK8) return kNumSimple + kNumStreamVariants + (D == 128 ? 1 : 2);
    return first_stream16() + (D == 128 ? 0 : 1);
}
bool attn_variant_supports(int v, int D, int kblock) { return variant(v) && variant(v)->D == D && variant(v)->kblock == kblock; }
// only the software-pipelined bf16 kernels take queries turned back for the sink range (AttnChunk::sink_shift)
bool attn_variant_sink_shift(int v) {
    return (v > kNumSimple && v <= kNumSimple + 2) || (is_stream16(v) && (v < first_stream16() + 2 || (v >= first_stream16() + 6 && v < first_stream16() + 8)));
}
// the software-pipelined kernel that multiplies the queries by AttnParams::scale_log2e itself
int attn_variant_qscale(int D) { return first_stream16() + (D == 128 ? 2 : 3); }
int attn_variant_lse(int D) { return first_stream16() + (D == 128 ? 4 : 5); }
int attn_variant_qrope(int D) { return first_stream16() + (D == 128 ? 8 : 9); }
// the 128-query kernel that leaves room for three workgroups per CU (short key sets, many query tiles)
int attn_variant_short_keys(int D) { return D == 128 ? 8 : 10; }
bool attn_variant_out_frag(int v) { return (v >= 1 && v <= kNumSimple) || is_stream16(v); }
bool attn_variant_applies_scale(int v) {
    return (v >= 1 && v <= kNumSimple) || v == kNumSimple + 3 || v == kNumSimple + 4 || v == first_stream16() + 2 || v == first_stream16() + 3;
}

// Into how many key groups (as a power of two) the workgroups of a launch deal their tiles' keys.  The chip holds one
// workgroup per CU.  With whole-key tiles of 256 rows a launch of few rows and heads leaves most of the 256 CUs idle
// while the others walk all its keys; G groups give G times as many workgroups of 1 / G of the steps each.  What the
// groups cost is LDS and L2 traffic: a kblock that goes into LDS serves 256 / G rows, so a step takes longer, the more
// so the more workgroups run.  A step's length relative to one group's, with n workgroups at work, as measured at
// 4 to 24 heads and 180 to 1560 rows over 2 to 634 kblocks (us per step with one group: 0.56 at head_dim 128, 0.41
// at 64):  a_G + n / b_G.  A workgroup also takes about ten steps' time before its first step and after its last (its
// arguments, the first loads, the results' way out), which every round of workgroups pays.  At 1170 rows x 183 kblocks x
// 12 heads x 128: 114 us with one group, 71 with two, 54 with four.  (A cache asks for each chunk as a launch of its own,
// api.cpp: build_attn; a clip or a prompt for the launch it makes.)
template <typename Rows, typename Kblocks>
static int key_groups_log2(const AttnVariant& v, int H, int n_chunks, Rows rows, Kblocks kblocks) {
    constexpr int CUS = 256, AROUND = 10;
    if (v.kblock == KBLOCK8) return 0;           // (no key groups there)
    struct Step { double a, b; };
    static constexpr Step steps128[4] = {{1.0, 1300}, {1.1, 900}, {1.35, 650}, {0, 1}};
    static constexpr Step steps64[4] = {{1.0, 1300}, {1.05, 1300}, {1.2, 1500}, {1.6, 800}};
    int best = 0;
    double best_cost = 0, bar = 1;
    for (int lg = 0; lg < 4; ++lg) {
        if (lg > 0 && v.grouped[lg - 1] == nullptr) continue;
        const int qtile = v.qtile >> lg;
        int64_t tiles = 0, work = 0, longest = 0;
        for (int c = 0; c < n_chunks; ++c) {
            const int64_t t = (rows(c) + qtile - 1) / qtile * int64_t(H);
            const int64_t len = (kblocks(c) + (1 << lg) - 1) >> lg;
            tiles += t;
            work += t * len;
            longest = std::max(longest, len);
        }
        const Step& s = (v.D == 128 ? steps128 : steps64)[lg];
        const double step = s.a + double(std::min<int64_t>(tiles, CUS)) / s.b, one = longest * step + AROUND;
        // equal workgroups run in whole rounds; of unequal ones the last to finish is half a workgroup behind the mean
        double cost = one;
        if (tiles > CUS)
            cost = n_chunks == 1 ? double((tiles + CUS - 1) / CUS) * one : (work * step + double(tiles) * AROUND) / CUS + 0.5 * one;
        // with half the chip at work as it is, a win has to be clear of what the model leaves out (short last tiles are
        // cheaper than whole ones, a round of new workgroups starts cold): 16 frames of 513 tokens x 17 x 128 as a clip
        // were predicted 4 % faster with two groups and ran 11 % slower (the margin is taken from two such clips)
        if (lg == 0 && tiles >= CUS / 2) bar = 0.87;
        if (lg == 0 || cost < bar * best_cost) {
            best = lg;
            best_cost = cost;
            bar = lg == 0 ? bar : 1;
        }
    }
    return best;
}
int attn_key_groups(int variant, int H, int n_chunks, const int* rows, const int* kblocks) {
    return 1 << key_groups_log2(*ll::variant(variant), H, n_chunks, [&](int c) { return rows[c]; }, [&](int c) { return kblocks[c]; });
}

// The same where tiles may also be dealt to several workgroups, merged by a second kernel (split.h).  What a launch
// takes is modelled in us: a round of workgroups takes its steps, each the longer the more workgroups run (LDS and L2
// traffic), and the way in and out; a merge, its launch and the partial results' way through memory.
struct SplitModel {
    struct { double step, busy; } whole[4], split[4];            // by log2 of the groups; 0: no such kernel
    double around, around_split, merge, per_split, per_mb;       // a round's way in and out, without and with splits
};
// bf16 cache: fitted to 350 timings of 26 shapes (1 to 24 heads, 96 to 4680 rows, 30 to 732 kblocks; 6 % off in the mean; the
// pair it picks was 1 % slower than the best).  The groups alone stay as above, and a split has to be 10 % cheaper than they
// are, 15 % where half the chip is at work without one.  us without and with splits at head_dim 128: 190 rows x 143 kblocks x 4
// heads 34 and 19 (4 groups x 9), 720 x 143 x 5 40 and 24 (4 x 4), 1560 x 634 x 12 206 and 165 (1 x 3), 4680 x 732 x 2 163
// and 104 (1 x 6); 1170 x 183 x 12 takes none (50).
static constexpr SplitModel kSplitModel[2] = {
    {{{0.52, 0.31}, {0.63, 0.21}, {0.82, 0.14}, {0, 0}}, {{0.52, 0.31}, {0.63, 0.21}, {0.82, 0.14}, {0, 0}}, 7.1, 7.1, 3.7, 0.22, 0.25},
    {{{0.38, 0.14}, {0.41, 0.10}, {0.47, 0.05}, {0.42, 0.39}}, {{0.38, 0.14}, {0.41, 0.10}, {0.47, 0.05}, {0.42, 0.39}}, 5.0, 5.0, 3.7, 0.22, 0.26}};
// 8-bit cache: no key groups, but workgroups of half and a quarter of the waves, which keep every row's bits (a wave that
// has its SIMD for itself takes two thirds of the time), and splits, whose steps take longer (weights of two terms).  430
// timings of 27 shapes (6 % off in the mean; the pick 2 % slower than the best, 4 % over the eleven of
// profiles/attn_split_times.txt).  Narrow tiles have to be 5 % cheaper than wide ones, splits 10 %.  us at head_dim 128, 256-row
// tiles and pick: 980 rows x 50 kblocks of 64 x 2 heads 50 and 29 (128-row tiles, 10 splits; 27 with 8), 300 x 22 x 24 30 and 20 (64), 1170 x
// 80 x 16 74 and 54 (128), 4680 x 366 x 2 285 and 108 (256, 6).
static constexpr SplitModel kSplitModel8[2] = {
    {{{0.82, 0.0}, {0.545, 0.03}, {0.494, 0.03}, {0, 0}}, {{1.23, 0.15}, {0.864, 0.03}, {0, 0}, {0, 0}}, 9.3, 6.7, 6.3, 0.58, 0.19},
    {{{0.66, 0.0}, {0.436, 0.05}, {0.373, 0.52}, {0, 0}}, {{1.00, 0.14}, {0.618, 0.46}, {0, 0}, {0, 0}}, 8.7, 3.3, 8.0, 0.26, 0.18}};

AttnSplit attn_split(int variant, int H, int n_chunks, const int* rows, const int* kblocks) {
    const AttnVariant& v = *ll::variant(variant);
    const bool fp8 = v.kblock == KBLOCK8;
    const int unsplit = key_groups_log2(v, H, n_chunks, [&](int c) { return rows[c]; }, [&](int c) { return kblocks[c]; });
    AttnSplit best{1 << unsplit, 1};
    if (v.split[0] == nullptr) return best;
    constexpr int CUS = 256;
    const SplitModel& m = (fp8 ? kSplitModel8 : kSplitModel)[v.D == 128 ? 0 : 1];
    int most_kblocks = 0;
    for (int c = 0; c < n_chunks; ++c) most_kblocks = std::max(most_kblocks, kblocks[c]);
    auto tiles_of = [&](int lg) {
        int64_t n = 0;
        for (int c = 0; c < n_chunks; ++c) n += (int64_t(rows[c]) + (v.qtile >> lg) - 1) / (v.qtile >> lg) * H;
        return n;
    };
    auto cost = [&](int lg, int splits) {
        const int keys_lg = fp8 ? 0 : lg;                        // groups that share a tile's keys
        const int64_t slots = fp8 && v.D == 64 && lg > 0 ? 2 * CUS : CUS;          // workgroups the chip holds
        int64_t n = 0, steps = 0, longest = 0;
        for (int c = 0; c < n_chunks; ++c) {
            const int shares = std::min(splits, std::max(1, kblocks[c] >> keys_lg)) << keys_lg;
            const int64_t t = (int64_t(rows[c]) + (v.qtile >> lg) - 1) / (v.qtile >> lg) * H * (shares >> keys_lg), len = (kblocks[c] + shares - 1) / shares;
            n += t;
            steps += t * len;
            longest = std::max(longest, len);
        }
        const auto& k = (splits == 1 ? m.whole : m.split)[lg];
        const double around = splits == 1 ? m.around : m.around_split;
        const double step = k.step * (1 + k.busy * double(std::min(n, slots)) / CUS), one = double(longest) * step + around;
        const double run = n <= slots ? one : n_chunks == 1 ? double((n + slots - 1) / slots) * one : (double(steps) * step + double(n) * around) / double(slots) + 0.5 * one;
        return run + (splits == 1 ? 0 : m.merge + m.per_split * splits + m.per_mb * 1e-6 * double(n) * (v.qtile >> lg) * v.D * 4);
    };
    double best_cost = cost(unsplit, 1), bar = tiles_of(unsplit) >= CUS / 2 && !fp8 ? 0.85 : 0.9;
    for (int lg = 1; fp8 && lg < 4; ++lg)
        if (m.whole[lg].step > 0 && cost(lg, 1) < (best.groups == 1 ? 0.95 : 1) * best_cost) {
            best_cost = cost(lg, 1);
            best = {1 << lg, 1};
        }
    best_cost *= bar;
    for (int lg = 0; lg < 4; ++lg) {
        if (m.split[lg].step <= 0) continue;
        const int64_t tiles = tiles_of(lg);
        for (int splits = 2; splits <= MAX_SPLITS && tiles * splits <= SPLIT_SLOTS && (fp8 ? splits : splits << lg) <= most_kblocks; ++splits) {
            if (m.around_split + m.merge + m.per_split * splits >= best_cost) break;         // (no cost of more splits is less)
            const double c = cost(lg, splits);
            if (c < best_cost) {
                best_cost = c;
                best = {1 << lg, splits};
            }
        }
    }
    return best;
}
// Whether a re-prefill launch of the 8-bit cache that takes no splits has its tiles in 64 rows and their keys dealt to four groups of
// two waves (attn_fp8.hip) instead of the narrow tiles that attn_split picks.  In one round of workgroups the longest share is a quarter of the
// longest key set, at two waves per SIMD instead of one; us a layer of a re-prefill, cache write included, without and with:
// 10 frames of 299 tokens x 5 heads x 128 (250 tiles) 46.3 -> 35.2, x 64 40 -> 27, 13 of 190 x 4 x 128 38 -> 30, 10 of 96 x 3 x 128 23.5 ->
// 22.5.  More tiles than CUs walk as many steps either way and read more of L2 (300 tiles 49 and 49, 450 52 and 56, 1200 96 and
// 116), and six kblocks leave a share little to walk (17.6 and 18.7).  In long key sets most rows' references move on the way, and a share
// does not know of those before it: its weights, no further from the exact ones, are rounded otherwise than the whole tile's (outputs
// 1.8 % of the 2-norm apart at 47 kblocks, 3.0 % at 131, two separate roundings 3.7 %), so those keep their tiles.
bool attn_takes_group8(int variant, AttnSplit split, int H, int n_chunks, const int* rows, const int* kblocks) {
    if (split.splits > 1 || ll::variant(variant)->grouped[2] == nullptr) return false;
    int64_t tiles = 0;
    int longest = 0;
    for (int c = 0; c < n_chunks; ++c) {
        tiles += int64_t(rows[c] + 63) / 64 * H;
        longest = std::max(longest, kblocks[c]);
    }
    return tiles <= 256 && longest >= 7 && longest <= 64;
}
// A launch of whole-key tiles of one length that fills some rounds of workgroups and a small part of one more: the tiles per head to
// take out of it and how many splits a launch of their own deals their keys to (0 tiles: none).  What that last round takes with
// and without, by the model above; it has to save 15 us.  us a clip's forward pass
// (layout included): 21 frames of 1560 tokens x 12 heads x 128 (1596 tiles, 60 of them in a seventh round) 3996 -> 3517, 21 of 390 x 8
// (280) 289 -> 219, 18 of 600 x 6 (270) 407 -> 294, 15 of 1560 x 4 (380) 996 -> 873, 20 of 200 x 15 (300) 163 -> 147.
// Only where all chunks are alike: a clip whose last chunk is shorter keeps the one launch (20 frames of 1560 x 12 x 128 in chunks of three
// take 3750 to 3950 us).
// (equal key sets that begin at other places of their first kblocks differ by one or two)
static bool same_length(int a, int b) { return std::abs(a - b) <= 2 && std::min(a, b) >= 16; }
AttnTail attn_tail(int variant, AttnSplit split, int H, int n_chunks, const int* rows, const int* kblocks) {
    const AttnVariant& v = *ll::variant(variant);
    constexpr int CUS = 256;
    if (split.groups > 1 || split.splits > 1) return {0, 1};
    int tiles = 0;
    for (int c = 0; c < n_chunks; ++c) {
        if (!same_length(kblocks[c], kblocks[0])) return {0, 1};
        tiles += (rows[c] + v.qtile - 1) / v.qtile;
    }
    const int full = tiles * H / CUS * CUS, per_head = (tiles * H - full + H - 1) / H, n = per_head * H;
    if (v.split[0] == nullptr || full == 0 || per_head == 0 || per_head >= tiles) return {0, 1};
    const SplitModel& m = kSplitModel[v.D == 128 ? 0 : 1];
    auto steps = [&](int workgroups, int length) { return length * m.split[0].step * (1 + m.split[0].busy * double(workgroups) / CUS) + m.around_split; };
    AttnTail best{0, 1};
    double most = 15;
    for (int splits = 2; splits <= MAX_SPLITS && n * splits <= CUS && splits <= kblocks[0]; ++splits) {
        const double saved = steps(n, kblocks[0]) - steps(n * splits, (kblocks[0] + splits - 1) / splits) -
                             (m.merge + m.per_split * splits + m.per_mb * 1e-6 * double(n) * splits * v.qtile * v.D * 4);
        if (saved > most) {
            most = saved;
            best = {per_head, splits};
        }
    }
    return best;
}
static __device__ SplitPool split_pool;
// its address on the current device (looked up on the first call per device; threads may do that at the same time)
hipError_t split_pool_address(SplitPool** pool) {
    constexpr int MAX_DEVICES = 64;
    static std::atomic<SplitPool*> known[MAX_DEVICES];
    int dev = -1;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < MAX_DEVICES && (*pool = known[dev].load(std::memory_order_relaxed)) != nullptr) return hipSuccess;
    void* at = nullptr;
    e = hipGetSymbolAddress(&at, HIP_SYMBOL(split_pool));
    if (e != hipSuccess) return e;
    *pool = static_cast<SplitPool*>(at);
    if (dev < MAX_DEVICES) known[dev].store(*pool, std::memory_order_relaxed);
    return hipSuccess;
}

// A call whose splits were launched and whose merge could not be: nobody is to read its partial results.  Gives back the slots
// that have its token (a word with a token is the call's own) once its stream is through; waits for that, as only this case may.
static void split_forget(SplitPool* pool, unsigned long long token, hipStream_t s) {
    unsigned long long owner[SPLIT_SLOTS];
    const unsigned long long nobody = 0;
    if (hipStreamSynchronize(s) != hipSuccess || hipMemcpy(owner, pool->owner, sizeof(owner), hipMemcpyDeviceToHost) != hipSuccess) return;
    for (int i = 0; i < SPLIT_SLOTS; ++i)
        if (owner[i] >> 24 == token) (void)hipMemcpy(&pool->owner[i], &nobody, sizeof(nobody), hipMemcpyHostToDevice);
}

constexpr int GROUPED_LDS_BYTES = 130 * 1024;    // GroupRing: 128 KB / G at most per group (the groups' results fit too), and what is touched
static_assert(4 * GroupRing<128, 4>::BYTES + 8 * GroupRing<128, 4>::LDS_TOUCH <= GROUPED_LDS_BYTES, "rings and what is touched");

hipError_t launch_attn(const AttnParams& p_in, int variant, hipStream_t s) {
    if (!attn_variant_supports(variant, p_in.D, p_in.kblock)) return hipErrorInvalidValue;
    AttnParams p = p_in;
    const AttnVariant& v = *ll::variant(variant);
    const int KB = p.kblock;
    for (int c = 0; c < p.n_chunks; ++c) {
        AttnChunk& ch = p.chunk[c];
        ch.n_kblocks = 0;
        for (int r = 0; r < ch.n_ranges; ++r) ch.n_kblocks += (ch.re[r] + KB - 1) / KB - ch.rs[r] / KB;
        if (ch.n_kblocks < 1) return hipErrorInvalidValue;
    }
    if (p.keys_reside && attn_resident_fits(p.D, p.chunk[0].n_kblocks) &&
        resident_fills_chip(p.H, p.chunk[0].q_end, p.chunk[0].n_kblocks)) {
        ResidentParams r{};
        r.q = p.q; r.out = p.out; r.out_frag = p.out_frag;
        r.k_cache = p.k_cache; r.v_cache = p.v_cache; r.head_stride = p.head_stride;
        r.H = p.H; r.n_rows = p.chunk[0].q_end; r.n_keys = p.chunk[0].re[0];
        r.scale_log2e = p.scale_log2e;
        return launch_attn_resident(r, p.D, s);
    }
    if (p.key_groups == 0) {
        int rows[MAX_ATTN_CHUNKS], kblocks[MAX_ATTN_CHUNKS];
        for (int c = 0; c < p.n_chunks; ++c) {
            rows[c] = p.chunk[c].q_end - p.chunk[c].q_begin;
            kblocks[c] = p.chunk[c].n_kblocks;
        }
        p.key_groups = attn_key_groups(variant, p.H, p.n_chunks, rows, kblocks);
        p.splits = 1;
        if (p.may_split) {
            const AttnSplit split = attn_split(variant, p.H, p.n_chunks, rows, kblocks);
            p.key_groups = split.groups;
            p.splits = split.splits;
            const AttnTail tail = p.may_split_tail ? attn_tail(variant, split, p.H, p.n_chunks, rows, kblocks) : AttnTail{0, 1};
            if (tail.tiles > 0) {                // the last tiles of the last chunks in a launch of their own
                AttnParams t = p, rest = p;
                t.key_groups = rest.key_groups = 1;
                t.splits = tail.splits;
                rest.splits = 1;
                t.n_chunks = 0;
                for (int left = tail.tiles; left > 0;) {
                    AttnChunk& last = rest.chunk[rest.n_chunks - 1];
                    AttnChunk& moved = t.chunk[t.n_chunks++] = last;
                    const int tiles = (last.q_end - last.q_begin + v.qtile - 1) / v.qtile;
                    if (tiles <= left) {
                        --rest.n_chunks;
                    } else {
                        moved.q_begin = last.q_end = last.q_begin + (tiles - left) * v.qtile;
                    }
                    left -= tiles;
                }
                const hipError_t e = launch_attn(rest, variant, s);
                return e != hipSuccess ? e : launch_attn(t, variant, s);
            }
            if (p.may_group8 && attn_takes_group8(variant, split, p.H, p.n_chunks, rows, kblocks)) p.key_groups = 8;
        }
    }
    int log_g = 0;
    while ((1 << log_g) < p.key_groups) ++log_g;
    if (log_g > 3) return hipErrorInvalidValue;
    const bool fp8 = v.kblock == KBLOCK8;
    const int qtile = v.qtile >> (fp8 ? std::min(log_g, 2) : log_g);             // (8 there: 64 rows, four key groups)
    p.n_tiles = 0;
    for (int c = 0; c < p.n_chunks; ++c) {
        p.chunk[c].tile_begin = p.n_tiles;
        p.n_tiles += (p.chunk[c].q_end - p.chunk[c].q_begin + qtile - 1) / qtile;
    }
    const int total = p.n_tiles * p.H;
    if (total <= 0) return hipSuccess;
    p.splits = std::max(1, p.splits);
    if (p.splits > MAX_SPLITS || (p.splits > 1 && (v.split[log_g] == nullptr || int64_t(total) * p.splits > SPLIT_SLOTS))) return hipErrorInvalidValue;
    p.per_tile = p.splits;
    p.merge = 0;
    p.slice_blocks = 16 >> log_g;
    int grid = ((total * p.splits + 7) / 8) * 8;           // the kernels spread their workgroups over the 8 XCDs
    if (p.splits > 1) {
        static std::atomic<unsigned long long> calls{0};
        p.token = calls.fetch_add(1, std::memory_order_relaxed) % (SPLIT_TOKENS - 1) + 1;
        hipError_t e = split_pool_address(&p.pool);
        if (e != hipSuccess) return e;
        // the merge in one round of workgroups: each takes its part of a tile's 16-row blocks (of the 8-bit kernel's 32-row ones)
        const int blocks = 16 >> log_g, least = p.kblock == KBLOCK8 ? 2 : 1, slices = std::max(1, std::min(blocks / least, 256 / total));
        p.slice_blocks = (blocks / least + slices - 1) / slices * least;
    }
    p.n_groups = 0;
    const int groups = p.H * p.n_chunks;
    // (every kernel but the simple ones reads the placement; a launch of one round, or of tiles of one length, is better dealt out
    // evenly: whole groups can give one XCD more tiles than the others; 500 tiles of a clip of 15 x 390 rows x 20 x 64 289 us -> 222)
    bool one_length = true;
    for (int c = 1; c < p.n_chunks; ++c) one_length = one_length && same_length(p.chunk[c].n_kblocks, p.chunk[0].n_kblocks);
    if (variant > kNumSimple && p.splits == 1 && p.n_chunks > 1 && !one_length && total > 256 && groups >= 16 && groups <= MAX_XCD_GROUPS) {
        // Tiles of different chunks differ in length, and the hardware binds workgroup b to XCD b % 8: hand each
        // XCD whole (head, chunk) groups so that all carry the same number of kblock steps (longest group to the
        // least loaded XCD), and let each start with its longest tiles.
        struct Group { int id, tiles, len; };
        std::vector<Group> all;
        for (int h = 0; h < p.H; ++h)
            for (int c = 0; c < p.n_chunks; ++c) {
                const int tiles = (c + 1 < p.n_chunks ? p.chunk[c + 1].tile_begin : p.n_tiles) - p.chunk[c].tile_begin;
                all.push_back({h * p.n_chunks + c, tiles, p.chunk[c].n_kblocks});
            }
        std::stable_sort(all.begin(), all.end(), [](const Group& a, const Group& b) {
            return int64_t(a.tiles) * a.len > int64_t(b.tiles) * b.len;
        });
        std::vector<Group> per_xcd[8];
        int64_t load[8] = {};
        for (const Group& g : all) {
            const int x = int(std::min_element(load, load + 8) - load);
            per_xcd[x].push_back(g);
            load[x] += int64_t(g.tiles) * g.len;
        }
        int n = 0, most_tiles = 0;
        for (int x = 0; x < 8; ++x) {
            std::stable_sort(per_xcd[x].begin(), per_xcd[x].end(), [](const Group& a, const Group& b) { return a.len > b.len; });
            p.xcd_first[x] = uint16_t(n);
            int tiles = 0;
            for (const Group& g : per_xcd[x]) {
                tiles += g.tiles;
                p.xcd_group[n++] = uint32_t(tiles) << 16 | uint32_t(g.id / p.n_chunks) << 8 | uint32_t(g.id % p.n_chunks);
            }
            most_tiles = std::max(most_tiles, tiles);
        }
        p.xcd_first[8] = uint16_t(n);
        if (most_tiles < 65536) {                              // (the words' 16 bits)
            p.n_groups = n;
            grid = 8 * most_tiles;
        }
    }
    if (variant > 64) return hipErrorInvalidValue;
    const int lds_bytes = log_g == 0 || fp8 ? v.lds_bytes : GROUPED_LDS_BYTES;
    const dim3 threads(fp8 && log_g < 3 ? v.threads >> log_g : v.threads);
    static bool attr_set[64][12] = {};
    auto prepare = [&](void (*kernel)(const AttnParams), int which) {            // which: one of the variant's kernels
        if (kernel == nullptr) return hipErrorInvalidValue;
        if (attr_set[variant - 1][which]) return hipSuccess;
        const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize, lds_bytes);
        attr_set[variant - 1][which] = e == hipSuccess;
        return e;
    };
    auto launch = [&](void (*kernel)(const AttnParams), int blocks) {
        return launch_kernel(reinterpret_cast<const void*>(kernel), dim3(blocks), threads, &p, lds_bytes, s);
    };
    if (p.splits == 1) {
        void (*const kernel)(const AttnParams) = log_g == 0 ? v.kernel : v.grouped[log_g - 1];
        const hipError_t e = prepare(kernel, log_g);
        return e != hipSuccess ? e : launch(kernel, grid);
    }
    hipError_t e = prepare(v.split[log_g], 4 + log_g);
    if (e == hipSuccess) e = prepare(v.merge[log_g], 8 + log_g);
    if (e == hipSuccess) e = launch(v.split[log_g], grid);
    if (e != hipSuccess) return e;
    p.merge = 1;
    p.per_tile = ((16 >> log_g) + p.slice_blocks - 1) / p.slice_blocks;
    e = launch(v.merge[log_g], (total * p.per_tile + 7) / 8 * 8);
    if (e != hipSuccess) split_forget(p.pool, p.token, s);
    return e;
}

}  // namespace ll
