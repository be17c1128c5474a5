// Output projection of the cross-attention block: y = x w^T with x [M, K] the heads' attention outputs side by side
// (K = H * D), w [N, K] the layer's output weight as a linear layer stores it ([output feature][input feature]),
// y [M, N]; bf16 in and out, fp32 accumulation.  A dense contraction: MFMA-bound (roofline of the bf16 matrix pipe).
//
// Why its own kernel and not an epilogue inside the attention kernel: the projection sums over ALL heads of a token,
// while attention's unit of work is one head (its K/V stream is what a workgroup shares).  A workgroup that held a
// token's all-head output would have to stream the whole weight (4.7 MB at 12 heads x 128) for a few dozen rows; one
// that kept its head would have to add its share into y across workgroups.  So the call runs the attention kernel
// first and this kernel behind it on the same stream.  What the two share is the operand layout: the attention
// kernel's epilogue writes its output as ready-made MFMA fragments (kernels.h: op_frag_offset), which is the order its
// accumulator registers already have, and the weight is packed into the same order once, when the model is loaded.
//
// Why fragments and not row-major operands (measured on this chip): a row-major fragment is 16 rows x 64 bytes, rows
// H * D * 2 bytes apart, and every load instruction gathers 16 separate pieces; L2 delivers 7.7-7.9 TB/s for such
// gathers against 13.8 TB/s for contiguous 1 KB fragments.  The row-major form of this kernel spent its time there
// (6.3 TB/s, whatever the staging: registers, direct-to-LDS loads, whole cache lines, staggered walks).
//
// Formulation, as in the attention kernels: the transposed product y^T = w x^T on 16x16x32 MFMAs.
//   A: w fragment (n block, k-step), B: x fragment (m block, k-step), same order of the 32 contraction indices in both
//   C: lane (g, c) register j = y[m0 + c][n0 + 4 g + j]: four neighbouring output features, one 8-byte store.
// A workgroup of 8 waves (two per SIMD) owns a tile of y, 256 x 128 where there are rows enough (each wave 64 x 64: 16
// accumulator blocks; smaller tiles below, at launch_out_proj), and walks K in steps of 64 through a ring of three LDS
// stages filled by direct-to-LDS loads two steps ahead: a step is 48 fragments (16 of w, 32 of x), six loads per wave, and
// 32 MFMAs per wave; one barrier per step (steps of 32 through six stages take the same time).  Every w fragment
// is read from LDS by four waves, every x fragment by two.
#include "kernels.h"

#include <algorithm>

namespace ll {

typedef __bf16 op_bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 op_bf16x2 __attribute__((ext_vector_type(2)));
typedef float op_f32x4 __attribute__((ext_vector_type(4)));
typedef float op_f32x2 __attribute__((ext_vector_type(2)));
typedef unsigned op_u32x4 __attribute__((ext_vector_type(4)));
typedef unsigned op_u32x2 __attribute__((ext_vector_type(2)));

constexpr int OP_WAVES = 8;
// A tile shape: BM x BN outputs per workgroup, WM x WN waves, K in steps of BK through STAGES stages.
template <int BM_, int BN_, int BK_, int STAGES_, int WM_, int WN_>
struct OpTile {
    static constexpr int BM = BM_, BN = BN_, BK = BK_, STAGES = STAGES_, WM = WM_, WN = WN_;
    static constexpr int SUBS = BK / 32;                        // k-steps of 32 per stage
    static constexpr int WFRAGS = BN / 16 * SUBS;               // 1 KB fragments per stage: of w,
    static constexpr int FRAGS = WFRAGS + BM / 16 * SUBS;       // then of x
    static constexpr int STAGE_BYTES = FRAGS * 1024, LDS_BYTES = STAGES * STAGE_BYTES;
    static constexpr int LPW = FRAGS / OP_WAVES;                // fragments a wave loads per stage
    static constexpr int MB = BM / 16 / WM, NB = BN / 16 / WN;  // 16 x 16 blocks of a wave
    static_assert(WM * WN == OP_WAVES && FRAGS % OP_WAVES == 0 && STAGES * LPW < 64 && LDS_BYTES <= 160 * 1024 && MB >= 1 && NB >= 1, "tile of the output projection");
};

// s_waitcnt that only waits for vector-memory loads: at most N outstanding
template <int N>
__device__ __forceinline__ void op_wait_vmcnt() {
    __builtin_amdgcn_s_waitcnt((N & 0xF) | ((N >> 4) << 14) | (0x7 << 4) | (0xF << 8));
}

// LDS reads the compiler does not see (attn_stream.hip): `dst` is pending until op_lds_wait, which waits for all of them.
__device__ __forceinline__ void op_lds_read(op_u32x4& dst, unsigned addr, int offset) {
    asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(dst) : "v"(addr), "n"(offset));
}
template <int N>
__device__ __forceinline__ void op_lds_wait(op_u32x4 (&x)[N]) {
    asm volatile("s_waitcnt lgkmcnt(0)" : "+v"(x[0]));
#pragma unroll
    for (int i = 1; i < N; ++i) asm volatile("" : "+v"(x[i]));   // arrived too: ties the register to this point
}

// The streamed fragments' base and offset stay in scalar registers, as in attn_bwd.hip (offsets are in bounds by construction).
__device__ __forceinline__ __amdgpu_buffer_rsrc_t op_region(const uint16_t* base) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t*>(base), 0, 0x7FFFFFFF, 0x00020000);   // raw buffer of dwords
}
__device__ __forceinline__ void op_load_lds16(__amdgpu_buffer_rsrc_t r, char* to, int lane_off, int uniform_off) {
    __builtin_amdgcn_raw_ptr_buffer_load_lds(r, (__attribute__((address_space(3))) void*)(to), 16, lane_off, uniform_off, 0, 0);
}

template <typename Tile>
__global__ __launch_bounds__(64 * OP_WAVES) __attribute__((amdgpu_waves_per_eu(2, 2)))
void ll_out_proj_kernel(const OutProjParams p) {
    constexpr int OP_BM = Tile::BM, OP_BN = Tile::BN, OP_BK = Tile::BK, OP_STAGES = Tile::STAGES;
    constexpr int OP_SUBS = Tile::SUBS, OP_WFRAGS = Tile::WFRAGS, OP_STAGE_BYTES = Tile::STAGE_BYTES, OP_LPW = Tile::LPW;
    constexpr int MB = Tile::MB, NB = Tile::NB;
    extern __shared__ __attribute__((aligned(16))) char lds[];
    const int lane = threadIdx.x & 63, r = lane & 15, g = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int wm = wave % Tile::WM, wn = wave / Tile::WM;
    // Workgroup b runs on XCD b % 8, each with its own L2: every XCD takes one contiguous run of tiles, weight blocks
    // fastest, so that the tiles it has in flight share a few row blocks of x (read once per XCD, then from its L2 for
    // every weight block) and walk the weight together.
    const int n_nt = (p.N + OP_BN - 1) / OP_BN, n_mt = (p.M + OP_BM - 1) / OP_BM;
    const int total = n_nt * n_mt, xcd = blockIdx.x & 7;
    const int tile = ((xcd * total + 7) >> 3) + (blockIdx.x >> 3);
    if (tile >= (((xcd + 1) * total + 7) >> 3)) return;          // uniform over the workgroup
    const int mt = tile / n_nt, nt = tile % n_nt;
    const int m0 = mt * OP_BM, n0 = nt * OP_BN;
    const int KT = p.K / OP_BK, n_ksteps = p.K / 32;
    const int last_mb = (p.M - 1) >> 4, last_nb = (p.N >> 4) - 1;

    // the fragments this wave loads per stage: fragments wave + 8 l of [w: (n block, sub-step) | x: (m block, sub-step)];
    // the two sub-steps of a block are neighbours in memory.  Blocks past the end of a tensor are clamped to its last
    // block (their products are never stored).  Base and offset stay in scalar registers (offsets are those within a tile).
    const __amdgpu_buffer_rsrc_t w_from = op_region(p.w_frag + int64_t(n0 >> 4) * n_ksteps * 512), x_from = op_region(p.x_frag + int64_t(m0 >> 4) * n_ksteps * 512);
    int src[OP_LPW];
#pragma unroll
    for (int l = 0; l < OP_LPW; ++l) {
        const int f = wave + OP_WAVES * l;                       // wave-uniform
        const int blk = f < OP_WFRAGS ? min(f / OP_SUBS, last_nb - (n0 >> 4)) : min((f - OP_WFRAGS) / OP_SUBS, last_mb - (m0 >> 4));
        src[l] = (blk * n_ksteps + f % OP_SUBS) * 1024;
    }
    static_assert(OP_WFRAGS % OP_WAVES == 0, "a load is of w or of x, whatever the wave");
    auto issue = [&](int kt, int to, int l) {
        const int kc = min(kt, KT - 1);          // past the end the last step is fetched again, never used
        op_load_lds16(OP_WAVES * l < OP_WFRAGS ? w_from : x_from, lds + to * OP_STAGE_BYTES + (wave + OP_WAVES * l) * 1024, lane * 16,
                      src[l] + kc * OP_SUBS * 1024);
    };

    op_f32x4 acc[NB][MB];                        // [n block][m block]
#pragma unroll
    for (int a = 0; a < NB; ++a)
#pragma unroll
        for (int b = 0; b < MB; ++b) acc[a][b] = op_f32x4{0.f, 0.f, 0.f, 0.f};

    // Fragment i of k-step `sub` of a stage: the wave's NB of w, then its MB of x.  Two register sets: while the MFMAs of one k-step
    // run from the one, the next k-step's fragments are read into the other (by hand: the compiler would put the reads in
    // front of the MFMAs that use them, and the two waves of a SIMD would wait for LDS at the same time).
    constexpr int NFR = NB + MB, NMFMA = NB * MB;
    op_u32x4 fr[2][NFR];
    const unsigned lds_lane = (unsigned)(size_t)(__attribute__((address_space(3))) char*)lds + lane * 16;
    const unsigned w_at = lds_lane + wn * NB * OP_SUBS * 1024, x_at = lds_lane + (OP_WFRAGS + wm * MB * OP_SUBS) * 1024;
    auto read_frag = [&](op_u32x4& dst, unsigned stage_at, int sub, int i) {
        if (i < NB) op_lds_read(dst, w_at + stage_at, (i * OP_SUBS + sub) * 1024);
        else op_lds_read(dst, x_at + stage_at, ((i - NB) * OP_SUBS + sub) * 1024);
    };
#pragma unroll
    for (int j = 0; j < OP_STAGES; ++j)
#pragma unroll
        for (int l = 0; l < OP_LPW; ++l) issue(j, j, l);
    op_wait_vmcnt<(OP_STAGES - 1) * OP_LPW>();
    asm volatile("s_barrier" ::: "memory");
#pragma unroll
    for (int i = 0; i < NFR; ++i) read_frag(fr[0][i], 0, 0, i);
    int stage = 0;                               // kt mod OP_STAGES
    static_assert(OP_SUBS == 2, "the register sets alternate within a step");
    for (int kt = 0; kt < KT; ++kt) {
        const int next = stage + 1 == OP_STAGES ? 0 : stage + 1;
#pragma unroll
        for (int sub = 0; sub < OP_SUBS; ++sub) {
            op_lds_wait(fr[sub]);
            if (sub == OP_SUBS - 1) {
                // every read of this step's stage has returned here, and this wave's loads of the next step have landed: behind
                // the barrier that holds for every wave, the stage is loaded anew and the next one read
                op_wait_vmcnt<(OP_STAGES - 2) * OP_LPW>();
                asm volatile("s_barrier" ::: "memory");
            }
            const unsigned from = unsigned(sub == OP_SUBS - 1 ? next : stage) * OP_STAGE_BYTES;
#pragma unroll
            for (int m = 0; m < NMFMA; ++m) {
                const int a = m / MB, b = m % MB;
                acc[a][b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(op_bf16x8, fr[sub][a]),
                                                                    __builtin_bit_cast(op_bf16x8, fr[sub][NB + b]), acc[a][b], 0, 0, 0);
                // the reads of the next k-step, spread over the first half of this one's MFMAs
#pragma unroll
                for (int i = 0; i < NFR; ++i)
                    if (i * ((NMFMA + 1) / 2) / NFR == m) read_frag(fr[1 - sub][i], from, 1 - sub, i);
                if (sub == OP_SUBS - 1)
#pragma unroll
                    for (int l = 0; l < OP_LPW; ++l)
                        if (l * NMFMA / OP_LPW == m) issue(kt + OP_STAGES, stage, l);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
        stage = next;
    }
    op_lds_wait(fr[0]);                          // no load may still be writing registers or LDS past this point
    op_wait_vmcnt<0>();

#pragma unroll
    for (int b = 0; b < MB; ++b) {
        const int row = m0 + (wm * MB + b) * 16 + r;
        if (row >= p.M) continue;
#pragma unroll
        for (int a = 0; a < NB; ++a) {
            const int col = n0 + (wn * NB + a) * 16 + 4 * g;
            if (col >= p.N) continue;            // N is a multiple of 16: a group of four is inside or outside
            const op_f32x2 lo = {acc[a][b][0], acc[a][b][1]}, hi = {acc[a][b][2], acc[a][b][3]};
            const op_u32x2 o = {__builtin_bit_cast(unsigned, __builtin_convertvector(lo, op_bf16x2)),
                                __builtin_bit_cast(unsigned, __builtin_convertvector(hi, op_bf16x2))};
            *reinterpret_cast<op_u32x2*>(p.y + int64_t(row) * p.N + col) = o;
        }
    }
}

// One thread per 16-byte unit of the packed weight: lane (g, r) of fragment (n block, k-step) takes
// w[16 nb + r][32 ks + 4 g + 0..3] and w[16 nb + r][32 ks + 16 + 4 g + 0..3].
__global__ __launch_bounds__(256) void ll_pack_out_weight_kernel(const uint16_t* w, uint16_t* w_frag, int N, int K) {
    const int64_t unit = int64_t(blockIdx.x) * 256 + threadIdx.x;
    const int n_ksteps = K / 32;
    if (unit >= int64_t(N / 16) * n_ksteps * 64) return;
    const int lane = int(unit & 63), r = lane & 15, g = lane >> 4;
    const int ks = int((unit >> 6) % n_ksteps), nb = int((unit >> 6) / n_ksteps);
    const uint16_t* row = w + int64_t(16 * nb + r) * K + 32 * ks + 4 * g;
    const op_u32x2 lo = *reinterpret_cast<const op_u32x2*>(row), hi = *reinterpret_cast<const op_u32x2*>(row + 16);
    *reinterpret_cast<op_u32x4*>(w_frag + unit * 8) = op_u32x4{lo[0], lo[1], hi[0], hi[1]};
}

hipError_t launch_pack_out_weight(const uint16_t* w, uint16_t* w_frag, int N, int K, hipStream_t s) {
    if (N < 16 || N % 16 != 0 || K < 32 || K % 32 != 0) return hipErrorInvalidValue;
    const int64_t units = int64_t(N / 16) * (K / 32) * 64;
    if ((units + 255) / 256 > 0x7FFFFFFF) return hipErrorInvalidValue;
    hipLaunchKernelGGL(ll_pack_out_weight_kernel, dim3(unsigned((units + 255) / 256)), dim3(256), 0, s, w, w_frag, N, K);
    return hipGetLastError();
}

template <typename Tile>
static hipError_t launch_tile(const OutProjParams& p, hipStream_t s) {
    const int64_t tiles = int64_t((p.M + Tile::BM - 1) / Tile::BM) * ((p.N + Tile::BN - 1) / Tile::BN);
    if (tiles > 0x7FFFFFFF) return hipErrorInvalidValue;
    static bool attr_set = false;
    if (!attr_set) {
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(ll_out_proj_kernel<Tile>),
                                           hipFuncAttributeMaxDynamicSharedMemorySize, Tile::LDS_BYTES);
        if (e != hipSuccess) return e;
        attr_set = true;
    }
    hipLaunchKernelGGL(ll_out_proj_kernel<Tile>, dim3(unsigned((tiles + 7) / 8 * 8)), dim3(64 * OP_WAVES), Tile::LDS_BYTES, s, p);
    return hipGetLastError();
}

using OpTile256x128 = OpTile<256, 128, 64, 3, 4, 2>;
using OpTile128x128 = OpTile<128, 128, 64, 3, 4, 2>;
using OpTile128x64 = OpTile<128, 64, 64, 5, 4, 2>;
using OpTile64x64 = OpTile<64, 64, 64, 6, 4, 2>;

// Time of a launch in us, fitted to 224 timings (60 to 23400 rows, 64 to 3072 features): rounds of workgroups over the CUs, each
// `around` and a walk over K whose step takes `alone` with few workgroups on the chip and `more` longer with all CUs at work.
// The tile it picks was the fastest or within 3 % of it at all 56 shapes.
template <typename Tile>
static double tile_us(const OutProjParams& p, double launch, double around, double alone, double more) {
    const int64_t tiles = int64_t((p.M + Tile::BM - 1) / Tile::BM) * ((p.N + Tile::BN - 1) / Tile::BN);
    return launch + double((tiles + 255) / 256) * (around + (p.K / Tile::BK) * (alone + more * double(std::min<int64_t>(tiles, 256)) / 256));
}

// The largest tile asks least of L2 and LDS and is the best one where there are enough of them; a launch of few rows leaves
// most CUs idle with it while the others walk all of K at 0.9 us a step.  The sums run over K in the same order in every tile
// shape: the results do not depend on it.  us with 256 x 128 tiles and with the tile taken, 12 heads x 128: 60 rows 23 -> 7,
// 300 22 -> 8, 1200 23 -> 11, 2400 25 -> 17, 4680 28 (228 tiles) either way.
//
// What a step of 256 x 128 costs: 128 KB of fragment reads and 48 KB of ring writes through LDS (1400 clocks) beside 1024 clocks
// of MFMAs.  With each k-step's reads in front of its own MFMAs they added up: 32 us at 4680 rows; read a k-step ahead, by
// hand, 28 (4680 x 3072 104 -> 92, 23400 x 1536 141 -> 128, 2400 x 2432 43 -> 37).
// With the loads dealt out between the MFMAs instead of six in a row behind the barrier, with the attention in front of it: 4680 x 3072
// 128.7 -> 125.6, 4680 x 1536 35.5 -> 34.5 (16 tokens) and 47.2 -> 46.5 (512).  What bounds it now is L2: 228 tiles x 24 steps x 48 KB at
// 12.8 TB/s while the steps run, 10.9 over a call; four waves of 128 x 64, which read two thirds as much of LDS, take the same time.
hipError_t launch_out_proj(const OutProjParams& p, hipStream_t s) {
    if (p.M < 1 || p.N < 16 || p.N % 16 != 0 || p.K < 64 || p.K % 64 != 0) return hipErrorInvalidValue;   // K = H * D, D 64 or 128
    const double t0 = tile_us<OpTile256x128>(p, 2.3, 3.85, 0.626, 0.257), t1 = tile_us<OpTile128x128>(p, 2.0, 2.36, 0.367, 0.136);
    const double t2 = tile_us<OpTile128x64>(p, 1.7, 2.13, 0.216, 0.098), t3 = tile_us<OpTile64x64>(p, 1.8, 1.38, 0.151, 0.103);
    const double best = std::min(std::min(t0, t1), std::min(t2, t3));
    if (best == t0) return launch_tile<OpTile256x128>(p, s);
    if (best == t1) return launch_tile<OpTile128x128>(p, s);
    if (best == t2) return launch_tile<OpTile128x64>(p, s);
    return launch_tile<OpTile64x64>(p, s);
}

}  // namespace ll
