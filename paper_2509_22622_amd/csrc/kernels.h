// Interface between the C-ABI host code and the gfx950 kernels, and the HBM layout
// of the rolling KV cache.
//
// Layout (per layer, per head; all bf16).  Token slots are grouped into "kblocks" of
// 32 slots.  Each kblock is stored as the exact register image the 32x32x16 bf16 MFMA
// wants, so a tile moves HBM -> LDS -> VGPR as straight 16-byte copies:
//   K kblock  [D/8 chunks][32 rows][8 elems]   row i holds key slot 32*b + swap23(i),
//             (swap23 exchanges bits 2 and 3) so that the S^T = K Q^T accumulator
//             registers of a lane hold 8 consecutive keys per half -- the order the
//             P^T operand of the second MFMA needs, with no cross-lane movement.
//   V kblock  [D/32 d-blocks][2 key halves t][2 lane halves h][32 d][8 keys]
//             = V^T fragments: element e of lane (h, dd) is key 32*b + 16*t + 8*h + e
//             at feature 32*db + dd.
// A head's K region is `kblocks_alloc` kblocks long, followed by its V region.
#pragma once
#include <hip/hip_runtime.h>
#include <cmath>
#include <cstdint>

namespace ll {

constexpr int KBLOCK = 32;          // key slots per kblock
constexpr int PAD_KBLOCKS = 8;      // readable padding after the last kblock of a head
constexpr int MAX_RANGES = 3;
constexpr int MAX_ATTN_CHUNKS = 24; // query chunks per attention launch
constexpr int MAX_APPEND_FRAMES = 16; // frames per cache-write launch (its argument block carries a rotary table per frame)
constexpr int FEW_APPEND_FRAMES = 8;  // up to here the launch takes the shorter argument block
constexpr int MAX_CHUNK_FRAMES = 32;  // largest chunk (ll_chunk_append splits longer runs of frames into several launches)
constexpr int MAX_T_PAIRS = 24;       // frame-axis rotary pairs: 22 at head_dim 128, 12 at 64
constexpr int MAX_XCD_GROUPS = 256; // (head, chunk) groups an attention launch can place on the XCDs one by one
__host__ __device__ inline int swap23(int i) {
    return (i & ~12) | ((i & 4) << 1) | ((i & 8) >> 1);
}
// Element offset (in bf16 units) of (slot-in-kblock k, feature d) inside a K kblock.
__host__ __device__ inline int k_elem_offset(int k, int d) {
    return (((d >> 3) * 32 + swap23(k)) << 3) + (d & 7);
}
// Element offset of (slot-in-kblock k, feature d) inside a V kblock.
__host__ __device__ inline int v_elem_offset(int k, int d) {
    const int t = k >> 4, h = (k >> 3) & 1, e = k & 7;
    return ((((((d >> 5) * 2 + t) * 2 + h) * 32) + (d & 31)) << 3) + e;
}

// ---- 8-bit (E4M3) cache.  One byte per element, kblocks of 64 slots, stored as the register image of the
// 32x32x64 fp8 MFMA (lane = 32 * k-half + row holds 32 consecutive contraction elements of its k-half), in
// 1 KB pieces [64 lanes][16 bytes] so that HBM -> LDS -> VGPR are straight 16-byte copies:
//   K kblock  [2 row blocks R][D/64 feature halves dh][2 pieces c][lane (h, r)][16]
//             lane (h, r) of piece (R, dh, c) holds key 32R + r, features 64dh + 32h + 16c + 0..15.
//   V kblock  [D/32 d-blocks db][2 pieces R][lane (h, dd)][16]
//             byte 4g + j of lane (h, dd) of piece (db, R) holds key 32R + 8g + 4h + j at feature 32db + dd:
//             the keys whose scores the S^T accumulator registers 4g + j of a lane in half h hold, so the
//             softmax weights go from accumulator to the second MFMA's operand without leaving the lane.
constexpr int KBLOCK8 = 64;
__host__ __device__ inline int k8_byte_offset(int k, int d, int D) {
    const int R = k >> 5, r = k & 31, dh = d >> 6, h = (d >> 5) & 1, c = (d >> 4) & 1;
    return ((((R * (D >> 6) + dh) * 2 + c) * 64 + h * 32 + r) << 4) + (d & 15);
}
__host__ __device__ inline int v8_byte_offset(int k, int d) {
    const int R = k >> 5, r = k & 31, h = (r >> 2) & 1;
    return ((((d >> 5) * 2 + R) * 64 + h * 32 + (d & 31)) << 4) + 4 * (r >> 3) + (r & 3);
}

struct RopeTables {            // device pointers into the cache buffer's tail
    const double* inv_freq_t;  // [n_t]      frame-axis frequencies theta^(-2i/d_t)
    const float2* row_cs;      // [grid_h][n_h]  (cos, sin) of y * freq
    const float2* col_cs;      // [grid_w][n_w]  (cos, sin) of x * freq
    int n_t, n_h, n_w;
};

struct AppendHead {
    const uint16_t* q; const uint16_t* k; const uint16_t* v;   // [n_frames*P, H, D]; q null (bf16 cache only): K, V only
    uint16_t* q_out;                                            // same shape; rotated q times q_scale
    float q_scale;                                              // log2(e) / sqrt(D), folded into q_out
    uint16_t* k_cache; uint16_t* v_cache;                       // layer base (head 0)
    int64_t head_stride;                                        // elements between heads
    RopeTables rope;
    int H, D, P, grid_w;
    int n_frames;
    // no rotary step at all (every pair passes unchanged; q, where given, only takes q_scale): the tables are not read then
    int identity;
    // When set (bf16 cache): t_cs[0 .. n_frames) is also stored there, [n_frames][MAX_T_PAIRS], for the attention
    // kernels that turn the queries themselves (AttnParams::t_table).
    float2* t_table_out;
    // 8-bit cache (all null / unused for the bf16 cache): byte pointers, head_stride in bytes
    uint8_t* q8_out; uint8_t* k8_cache; uint8_t* v8_cache;
    float k_mul, v_mul;                                         // 2^-k_exp, 2^-v_exp (q_scale carries 2^k_exp)
};
// The kernels' arguments for up to N frames.  A re-prefill of 9 to 16 frames is one launch, not two; a chunk's few frames keep
// the block of 8, 1.6 KB shorter and half the tables for a workgroup to fetch first.  us a call: 10 frames of 299 tokens x 5 x
// 128 with an 8-bit cache 52.7 -> 46.4, 9 of 126 x 2 x 128 31.0 -> 26.7, three layers' 10 of 132 x 13 x 128 128.5 -> 117.0.
template <int N>
struct AppendArgs : AppendHead {
    // (cos, sin) of frame * frequency for every frame-axis pair of every frame, computed on the host in double
    // (set_frame_rotation): the kernels run no trigonometry.
    float2 t_cs[N][MAX_T_PAIRS];
    int64_t slot[N];                                            // first token slot
    int seg_begin[N + 1];                                       // prefix sum of segments (the part of a frame in 32 slots)
};
using AppendParams = AppendArgs<MAX_APPEND_FRAMES>;
using FewAppendParams = AppendArgs<FEW_APPEND_FRAMES>;

// Fill p.t_cs for frames with absolute indices frames[0 .. n_frames) from the host copy of the frame-axis frequencies (p.rope.n_t).
template <int N>
inline void set_frame_rotation(AppendArgs<N>& p, const int64_t* frames, const double* inv_freq_t_host) {
    for (int i = 0; i < p.n_frames; ++i)
        for (int j = 0; j < p.rope.n_t && j < MAX_T_PAIRS; ++j) {
            const double a = double(frames[i]) * inv_freq_t_host[j];
            p.t_cs[i][j] = make_float2(float(std::cos(a)), float(std::sin(a)));
        }
}

// One rotary pair (re, im) turned by w = (cos, sin) and scaled, in fp32.  Every kernel that turns a query or an 8-bit key
// goes through here, and the bf16 keys through rope_turn_key, with the contraction into fused multiply-adds fixed by hand:
// left to the compiler it flips with edits elsewhere in the kernel, and some results then round to the neighbouring value.
__device__ __forceinline__ void rope_turn_scaled(float re, float im, float2 w, float scale, float& o_re, float& o_im) {
    const float t = im * w.y, u = im * w.x;
    o_re = __builtin_fmaf(re, w.x, -t) * scale;
    o_im = __builtin_fmaf(re, w.y, u) * scale;
}
// (the other product of the imaginary part is the rounded one here: these are the bits cached keys have always had)
__device__ __forceinline__ void rope_turn_key(float re, float im, float2 w, float& o_re, float& o_im) {
    const float t = im * w.y, u = re * w.y;
    o_re = __builtin_fmaf(re, w.x, -t);
    o_im = __builtin_fmaf(im, w.x, u);
}

struct AttnChunk {
    int q_begin, q_end;          // query rows [q_begin, q_end) of the q tensor
    int tile_begin;              // first query tile of this chunk in the launch  (filled in by launch_attn)
    int n_ranges;
    int rs[MAX_RANGES], re[MAX_RANGES];   // key token-slot ranges
    int n_kblocks;               // kblocks the ranges touch        (filled in by launch_attn)
    // Sink at a fixed rotary distance (0 = off): range 0 is exactly the sink, and its scores are taken with the
    // queries turned back by sink_shift frames on the frame axis of the rotary embedding.
    int sink_shift;
    // Queries given before the rotary embedding (AttnParams::t_table set): row r of the chunk is token (r - q_begin)
    // % P of the frame whose frame-axis (cos, sin) are row t_row + (r - q_begin) / P of the table.
    int t_row;
};

struct AttnParams {
    const uint16_t* q; uint16_t* out;     // [rows, H, D]
    // When set, the output goes here instead, in the fragment order of the output projection (op_frag_offset with
    // H * D / 32 k-steps, the heads side by side); honoured by the kernels attn_variant_out_frag names.  Chunk 0 must
    // start at row 0.
    uint16_t* out_frag;
    const uint16_t* k_cache; const uint16_t* v_cache;   // layer base (head 0)
    int64_t head_stride;
    int H, D;
    float scale_log2e;           // factor still to apply to q.k in the log2 domain (1 when q is pre-scaled); only
                                 // the simple kernels and the *_qscale kernels apply it
    int n_chunks, n_tiles;       // n_tiles = query tiles over all chunks (filled in by launch_attn)
    // Placement on the 8 XCDs (filled in by launch_attn; workgroup b runs on XCD b % 8).  n_groups == 0: the
    // (head, tile) items are split into 8 contiguous runs.  Otherwise (launches of several chunks, whose tiles
    // differ in length) XCD x runs the (head, chunk) groups xcd_group[xcd_first[x] .. xcd_first[x + 1]) in that
    // order, all tiles of a group on one XCD; a group's word is end << 16 | head << 8 | chunk, end counting the XCD's tiles
    // up to and with the group's.
    int n_groups;
    // 8-bit cache: E4M3 queries and cache (byte pointers, head_stride in bytes), factor 2^v_exp on the output
    const uint8_t* q8; const uint8_t* k8_cache; const uint8_t* v8_cache;
    float out_scale;
    int kblock;                  // key slots per kblock: 32 (bf16 cache) or 64 (8-bit cache)
    const double* inv_freq_t;    // frame-axis rotary frequencies [n_t] (used when a chunk has a sink_shift)
    int n_t;
    int key_groups;              // key groups per tile (AttnVariant::grouped); 0: chosen for the launch,
    bool may_split;              // and splits with them
    bool may_group8;             // 8-bit cache: and tiles of 64 rows in four key groups
    bool may_split_tail;         // and splits for the tiles of the last round alone (queries rotated already, whole chunks or not)
    // A tile's keys dealt to `splits` workgroups, whose partial results a second kernel merges (split.h);
    // chunks of fewer kblocks take fewer.  The rest is filled in by launch_attn.
    int splits;
    int merge;                   // this launch is the merge: a workgroup takes slice_blocks 16-row blocks of a tile
    int slice_blocks;
    int per_tile;                // workgroups per tile: splits, or slices of the merge
    unsigned long long token;
    struct SplitPool* pool;
    bool keys_reside;            // the one key range may be brought into LDS whole where it fits (attn_resident.hip)
    float* lse;                  // *_lse kernels: log2 of each row's sum of 2^score, [H][lse_stride] (null otherwise)
    int64_t lse_stride;
    float* out32;                // *_lse kernels: the output once more in fp32, [rows, H, D] (null: not wanted)
    // *_qrope kernels: q holds the queries as the model's projection made them; a wave turns its rows on load
    // (3D rotary embedding, the same arithmetic as the cache-write kernel) and scales them by q_scale.
    const float2* t_table;       // frame-axis (cos, sin), [frames of the call][MAX_T_PAIRS], written by the cache write
    const float2* row_cs; const float2* col_cs;   // as in RopeTables
    int P, grid_w;
    float q_scale;
    uint16_t xcd_first[9];
    uint32_t xcd_group[MAX_XCD_GROUPS];
    AttnChunk chunk[MAX_ATTN_CHUNKS];
};

// The kernel's arguments read anew: nothing that was computed from them before can be kept in registers for what follows.
// For the body of a loop that nearly always runs once, so that a kernel with it needs the registers of one without.
__device__ __forceinline__ const AttnParams& attn_params_again() {
    auto at = __builtin_amdgcn_kernarg_segment_ptr();
    asm volatile("" : "+s"(at));
    return *(const AttnParams*)(at);
}

// Which group of its XCD's list a workgroup's tile belongs to, found by a wave with one load, an entry a lane, instead of a walk
// along the groups of three scalar loads each, cold in the first round of workgroups.  us a re-prefill with the walk and so: 7
// frames of 140 tokens x 16 x 128 in chunks of two 36.6 and 34.4, 7 of 232 x 10 x 64 (two layers) 69.1 and 66.2, 1560 tokens x 12
// x 128 level.  (The walk along a launch's chunks where nothing is placed stays: over two to four chunks, whose scalar loads
// share cache lines with the other arguments', it takes 0.3 us less than a vector load.)
// (idx: the workgroup's number on its XCD; false past the end of the list)
__device__ __forceinline__ bool attn_placed_tile(const AttnParams& p, int xcd, int idx, int& head, int& chunk, int& tile) {
    const int lane = threadIdx.x & 63, first = p.xcd_first[xcd], n = p.xcd_first[xcd + 1] - first;
    int passed = 0;                              // tiles of the groups looked at so far
    for (int base = 0; base < n; base += 64) {
        const unsigned word = p.xcd_group[first + min(base + lane, n - 1)];
        const int k = __builtin_popcountll(__ballot(base + lane < n && idx >= int(word >> 16)));
        if (k > 0) passed = int(unsigned(__builtin_amdgcn_readlane(int(word), k - 1)) >> 16);
        if (k < 64 && base + k < n) {
            const int group = __builtin_amdgcn_readlane(int(word), k);
            head = (group >> 8) & 255;
            chunk = group & 255;
            tile = p.chunk[chunk].tile_begin + idx - passed;
            return true;
        }
    }
    return false;
}

// A workgroup's place in a launch of split tiles, or of their merge: heads, splits (slices of the merge), tiles; a split's tiles side
// by side, they share its keys.  item < 0: none.
struct SplitPlace { int item, head, part, tile; };
__device__ __forceinline__ SplitPlace split_place(const AttnParams& p) {
    const int xcd = blockIdx.x & 7, per_head = p.n_tiles * p.per_tile, total = per_head * p.H;
    const int item = ((xcd * total + 7) >> 3) + (blockIdx.x >> 3);
    if (item >= (((xcd + 1) * total + 7) >> 3)) return {-1, 0, 0, 0};
    const int head = item / per_head, in_head = item - head * per_head, part = in_head / p.n_tiles;
    return {item, head, part, in_head - part * p.n_tiles};
}

struct ReadFrameParams {
    const uint16_t* k_cache; const uint16_t* v_cache; int64_t head_stride;
    uint16_t* k_out; uint16_t* v_out;     // [P, H, D], either may be null
    int H, D, P; int64_t slot;
    const uint8_t* k8_cache; const uint8_t* v8_cache;   // 8-bit cache: codes go to k8_out / v8_out
    uint8_t* k8_out; uint8_t* v8_out;
};

// ---- backward pass of the train-time rule (attn_bwd.hip)
constexpr int MAX_BWD_GROUPS = 32;
struct BwdGroup {                // column tiles that share one set of streamed rows
    int c_begin, c_end;          // columns: query rows (dQ kernel) or clip-token indices of keys (dK/dV kernel)
    int tile_begin;              // first tile of the group in the launch (filled in by launch_bwd_*)
    int n_ranges;
    int rs[2], re[2];            // streamed rows: key token slots (dQ kernel), query rows (dK/dV kernel: one range)
};
struct BwdParams {
    const uint16_t* q;                                  // dQ kernel: rotated, scaled queries, [rows, H, D]
    const float* lse; const float* delta;               // [H][row_stride]
    int64_t row_stride;
    // streamed fragment regions (head 0; element strides between heads): two K-style, two V^T-style
    const uint16_t* s_k1; const uint16_t* s_k2; const uint16_t* s_t1; const uint16_t* s_t2;
    int64_t hs_k1, hs_k2, hs_t1, hs_t2;
    // K-style regions holding the columns' own rows: K' and V, and the token slot of clip token 0 (dK/dV kernel); dO in c_k2,
    // row 0 at slot 0 (dQ kernel: the caller's dO is not read here, dV of the same launch may be written over it)
    const uint16_t* c_k1; const uint16_t* c_k2;
    int64_t hc_k1, hc_k2, col_slot0;
    float* g1;                   // fp32 [rows, H, D]: Gq (dQ kernel) or Gk (dK/dV kernel)
    uint16_t* dv;                // dK/dV kernel: bf16 [rows, H, D]
    int H, D, n_groups;
    int n_tiles;                 // filled in by launch_bwd_*
    BwdGroup group[MAX_BWD_GROUPS];
};
// Both kinds in one launch; the placement on the XCDs is filled in by launch_bwd_both (attn_bwd.hip).
constexpr int MAX_BWD_UNITS = 640;
struct BwdBothParams {
    BwdParams dq, dkv;
    int n_units;
    uint16_t xcd_first[9];
    uint16_t xcd_unit[MAX_BWD_UNITS];            // head * (groups of both kinds) + group, the dK/dV kind's first
};
static_assert(sizeof(BwdBothParams) <= 4096, "kernel arguments");
struct BwdFinishParams {
    const float* gq; const float* gk;                   // [n_frames * P, H, D]
    uint16_t* dq; uint16_t* dk;
    RopeTables rope;
    int H, D, P, grid_w, n_frames;
    int64_t frame0;              // absolute index of the first frame
    float q_mul, k_mul;          // 1/sqrt(D), ln 2
};
// The operands of a training step as MFMA fragments (clip_layout.hip): rows [0, rows) of x and y [rows, H, D], both ways round each.
struct ClipLayoutParams {
    const uint16_t* x; const uint16_t* y;
    uint16_t* x_k; uint16_t* y_k; uint16_t* x_t; uint16_t* y_t;  // K-style and V^T-style regions (head 0)
    int64_t head_stride;
    int H, rows;
    // forward (out32 null): x holds keys before the rotary embedding, and rows from q_row0 on are the clip's, whose queries q
    // [rows - q_row0, H, D] go to q_out rotated and scaled.  Row r belongs to frame r / P of the list of resident frames: the
    // first n_sink_outside are the sink's, the others follow ctx_start.
    const uint16_t* q; uint16_t* q_out;
    int q_row0;
    float q_scale;
    RopeTables rope;
    int P, grid_w, n_sink_outside;
    int64_t ctx_start;
    // backward: x holds q', y dO; delta[head * row_stride + row] = dO . O
    const float* out32; float* delta;
    int64_t row_stride;
};
hipError_t launch_clip_layout(const ClipLayoutParams& p, int D, hipStream_t s);
hipError_t launch_bwd_both(const BwdParams& dq, const BwdParams& dkv, hipStream_t s);
hipError_t launch_bwd_dq(const BwdParams& p, hipStream_t s);
hipError_t launch_bwd_dkv(const BwdParams& p, hipStream_t s);
hipError_t launch_bwd_finish(const BwdFinishParams& p, hipStream_t s);

// One attention kernel instantiation.
struct AttnVariant {
    const char* name;
    int D, qtile, lds_bytes;
    void (*kernel)(const AttnParams);
    int threads;
    int kblock;                  // 32: bf16 cache, 64: 8-bit cache
    // The same work with the keys of a tile dealt to G = 2, 4, 8 groups of the workgroup's waves (qtile / G rows per
    // workgroup); null where there is no such kernel.  8-bit cache: the first two have 1 / G of the waves instead, which all
    // walk all keys; the third 64 rows, whose keys are dealt to four groups of two waves.
    void (*grouped[3])(const AttnParams);
    // The kernels of launches with AttnParams::splits > 1 and of their merges, by log2 of G (null: no splits)
    void (*split[4])(const AttnParams);
    void (*merge[4])(const AttnParams);
};
extern const AttnVariant kStreamVariants[];
extern const int kNumStreamVariants;
extern const AttnVariant kFp8Variants[];
extern const int kNumFp8Variants;
extern const AttnVariant kStream16Variants[];   // the software-pipelined kernels on 16x16x32 MFMAs (attn_stream16.hip)
extern const int kNumStream16Variants;

// Attention variants (query rows per workgroup differ).
int attn_variant_count();
const char* attn_variant_name(int v);
int attn_variant_default(int D, int kblock);
bool attn_variant_supports(int v, int D, int kblock);
// the key groups a launch of these chunks takes with the variant: 1, 2, 4 or 8
int attn_key_groups(int v, int H, int n_chunks, const int* rows, const int* kblocks);
// the same where tiles may also be dealt to several workgroups: for one streamed chunk, or for a launch of several
struct AttnSplit { int groups, splits; };
AttnSplit attn_split(int v, int H, int n_chunks, const int* rows, const int* kblocks);
// where that is `split`: whether an 8-bit re-prefill's tiles go to four key groups, and how many tiles a head of a clip's forward
// pass go out in a launch of their own, with how many splits (0 and 1: none)
bool attn_takes_group8(int v, AttnSplit split, int H, int n_chunks, const int* rows, const int* kblocks);
struct AttnTail { int tiles, splits; };
AttnTail attn_tail(int v, AttnSplit split, int H, int n_chunks, const int* rows, const int* kblocks);
bool attn_variant_sink_shift(int v);          // the variant honours AttnChunk::sink_shift
int attn_variant_lse(int D);                   // the variant that also writes AttnParams::lse
int attn_variant_qscale(int D);                // the variant for queries not yet scaled (honours scale_log2e)
int attn_variant_short_keys(int D);            // small workgroups, three per CU: for short key sets
int attn_variant_qrope(int D);                 // the variant that turns the queries itself (AttnParams::t_table)
bool attn_variant_applies_scale(int v);        // the variant multiplies the scores (or queries) by scale_log2e itself
bool attn_variant_out_frag(int v);             // the variant honours AttnParams::out_frag

// Output projection y = x w^T (out_proj.hip): x [M, K] and w [N, K] in fragment order, y [M, N] bf16 row-major.
// Fragment order: 16 rows x 32 contraction indices form one 1 KB fragment, ready to be an operand of a 16x16x32 MFMA:
// lane 16 g + r holds, for row 16 b + r, the indices 32 ks + 4 g + 0..3 and 32 ks + 16 + 4 g + 0..3 (the pairing the
// attention kernels' accumulators give for free); the fragments of a row block b lie side by side in ks.  The
// offset, in elements, of the 8 values of (row, k-step ks, lane group g) in a tensor of n_ksteps = K / 32 k-steps:
__host__ __device__ inline int64_t op_frag_offset(int row, int ks, int g, int n_ksteps) {
    return ((int64_t(row >> 4) * n_ksteps + ks) * 64 + 16 * g + (row & 15)) * 8;
}
// x_frag holds ceil(M / 16) row blocks (rows past M in the last one may hold anything); N a multiple of 16, K of 64.
struct OutProjParams { const uint16_t* x_frag; const uint16_t* w_frag; uint16_t* y; int M, N, K; };
hipError_t launch_out_proj(const OutProjParams& p, hipStream_t s);
// w [N, K] bf16 row-major ([output feature][input feature]) -> fragment order, same size
hipError_t launch_pack_out_weight(const uint16_t* w, uint16_t* w_frag, int N, int K, hipStream_t s);

// Attention over one key range that starts at slot 0 and fits into LDS whole (attn_resident.hip).
struct ResidentParams {
    const uint16_t* q; uint16_t* out; uint16_t* out_frag;        // as in AttnParams; rows [0, n_rows)
    const uint16_t* k_cache; const uint16_t* v_cache;
    int64_t head_stride;
    int H, n_rows, n_keys;
    float scale_log2e;           // factor to apply to the scores
    int n_kblocks, parts;        // workgroups per head (filled in by launch_attn_resident)
};
bool attn_resident_fits(int D, int n_kblocks);
hipError_t launch_attn_resident(const ResidentParams& p, int D, hipStream_t s);

// A launch with its arguments by pointer (they are 2 to 3 KB).  A failure is the caller's to report: it does not stay behind as the
// thread's last error, for a later call of somebody else's to find.
inline hipError_t launch_kernel(const void* kernel, dim3 grid, dim3 block, const void* args, size_t lds_bytes, hipStream_t s) {
    void* list[] = {const_cast<void*>(args)};
    const hipError_t e = hipLaunchKernel(kernel, grid, block, list, lds_bytes, s);
    if (e != hipSuccess) (void)hipGetLastError();
    return e;
}
hipError_t launch_append(const AppendParams& p, hipStream_t s);
hipError_t launch_append(const FewAppendParams& p, hipStream_t s);
hipError_t launch_append8(const AppendParams& p, hipStream_t s);
hipError_t launch_append8(const FewAppendParams& p, hipStream_t s);
hipError_t launch_read_frame8(const ReadFrameParams& p, hipStream_t s);
hipError_t launch_attn(const AttnParams& p, int variant, hipStream_t s);
hipError_t launch_read_frame(const ReadFrameParams& p, hipStream_t s);
// diagnostic (probe_kernels.hip): sink holds workgroups * 512 floats, counters two 64-bit words; `companion` is the
// kind of instruction issued `per_mfma` (1 or 2) times behind every MFMA
enum ProbeCompanion {
    PROBE_NONE = 0, PROBE_ADD = 1, PROBE_EXP = 2, PROBE_CVT_BF16 = 3, PROBE_DOT2_BF16 = 4, PROBE_MAX3 = 5,
    PROBE_LDS_READ = 6, PROBE_SHAPE_16X16X32 = 7,  // 7: no companion, 16x16x32 MFMAs instead of 32x32x16
    // fp8 32x32x64 MFMAs (E4M3 operands): alone, with what the 8-bit attention kernel issues per MFMA (4 exp2, 4 adds,
    // 2 conversions, 2 max3, two 16-byte LDS reads), with its vector part only, with its LDS part only
    PROBE_FP8_NONE = 8, PROBE_FP8_MIX = 9, PROBE_FP8_VALU = 10, PROBE_FP8_LDS = 11
};
hipError_t launch_probe_mfma(float* sink, unsigned long long* counters, int workgroups, int iters, int random_operands,
                             int companion, int per_mfma, hipStream_t s);

}  // namespace ll
