// The operands of a training step (ll_clip_*), laid out as MFMA fragments: every tensor that some product contracts over its
// rows and another over its features is needed both ways round (kernels.h: K-style, V^T-style kblocks).
//   forward:  k, v of all resident frames -> region pairs A (K' K-style, V^T) and B (V K-style, K'^T), K' = k after the rotary
//             embedding; the clip's q -> rotated, scaled, row-major
//   backward: q' and dO of the clip -> region pairs Cq (q' K-style, dO^T) and Cd (dO K-style, q'^T), and delta = rowsum(dO O)
// All frames of a step lie in one linear region, so a kblock is 32 consecutive rows whatever frames they belong to, and one
// launch serves them all.
//
// Memory bound: one pass over the inputs, one over the regions.  A workgroup takes one kblock of one head: all its loads
// first (16 bytes a lane), rows of both tensors into LDS, four images out of it in 16-byte stores.  The frame axis's
// (cos, sin) are computed by a few lanes while the loads are on their way, as in the gradients' last kernel.  This took the place of
// five cache writes of eight frames each, a read-back of K' and a second pair of writes (forward), and of two writes and a
// kernel for delta (backward).  us a step: 21 frames of 1560 tokens x 12 x 128 17130 -> 16820; 15 of 140 x 3 x 64 96 -> 77; 19 of
// 99 x 9 x 128 190 -> 146; every bit as before.
#include "kernels.h"

namespace ll {

typedef unsigned short u16x8 __attribute__((ext_vector_type(8)));
typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));

__device__ inline float cl_f32(unsigned short b) { return __uint_as_float(unsigned(b) << 16); }
__device__ inline unsigned cl_pack(float a, float b) { return __builtin_bit_cast(unsigned, __builtin_convertvector(f32x2{a, b}, bf16x2)); }

template <int D, bool BACKWARD>
__global__ __launch_bounds__(256) void ll_clip_layout_kernel(const ClipLayoutParams p) {
    constexpr int CH = D / 8;                 // 16-byte chunks per (row, head)
    constexpr int ROW = D + 8;                // padded LDS row (elements)
    constexpr int ITEMS = 32 * CH / 256;
    __shared__ __attribute__((aligned(16))) unsigned short x_rows[32 * ROW];
    __shared__ __attribute__((aligned(16))) unsigned short y_rows[32 * ROW];
    __shared__ float2 t_cs[BACKWARD ? 1 : 32 * MAX_T_PAIRS];

    const int tid = threadIdx.x;
    const int kb = blockIdx.x / p.H, head = blockIdx.x - kb * p.H;
    const int row0 = kb * KBLOCK, n_rows = min(KBLOCK, p.rows - row0);
    // position (frame, token) of the first row; P >= 1, so a kblock touches at most 32 frames
    const int pos0 = BACKWARD ? 0 : row0 / p.P, tok0 = row0 - pos0 * p.P;
    const int y0 = BACKWARD ? 0 : tok0 / p.grid_w;

    u16x8 xv[ITEMS], yv[ITEMS], qv[ITEMS];
    f32x4 o0[ITEMS], o1[ITEMS];
    float2 cs[ITEMS][4];
    int frame[ITEMS];                         // of the row, counted from the kblock's first
#pragma unroll
    for (int it = 0; it < ITEMS; ++it) {
        const int item = tid + 256 * it, ti = item / CH, c = item % CH;
        xv[it] = yv[it] = qv[it] = u16x8{};
        frame[it] = 0;
        if (ti >= n_rows) continue;
        const int64_t src = (int64_t(row0 + ti) * p.H + head) * D + c * 8;
        xv[it] = *reinterpret_cast<const u16x8*>(p.x + src);
        yv[it] = *reinterpret_cast<const u16x8*>(p.y + src);
        if constexpr (BACKWARD) {
            o0[it] = *reinterpret_cast<const f32x4*>(p.out32 + src);
            o1[it] = *reinterpret_cast<const f32x4*>(p.out32 + src + 4);
        } else {
            if (row0 + ti >= p.q_row0) qv[it] = *reinterpret_cast<const u16x8*>(p.q + src - int64_t(p.q_row0) * p.H * D);
            int tok = tok0 + ti;
            if (p.P >= KBLOCK) {              // one wrap at most
                if (tok >= p.P) { tok -= p.P; frame[it] = 1; }
            } else {
                frame[it] = tok / p.P;
                tok -= frame[it] * p.P;
            }
            int y, x;
            if (p.grid_w >= KBLOCK && frame[it] == 0) {          // the same for the grid's rows
                y = y0;
                x = tok - y0 * p.grid_w;
                if (x >= p.grid_w) { x -= p.grid_w; ++y; }
            } else {
                y = tok / p.grid_w;
                x = tok - y * p.grid_w;
            }
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int pi = c * 4 + e;
                cs[it][e] = make_float2(1.f, 0.f);
                if (pi >= p.rope.n_t)
                    cs[it][e] = pi < p.rope.n_t + p.rope.n_h ? p.rope.row_cs[y * p.rope.n_h + (pi - p.rope.n_t)]
                                                             : p.rope.col_cs[x * p.rope.n_w + (pi - p.rope.n_t - p.rope.n_h)];
            }
        }
    }
    if constexpr (!BACKWARD) {
        const int n_frames = (tok0 + n_rows - 1) / p.P + 1;
        for (int i = tid; i < n_frames * p.rope.n_t; i += 256) {
            const int f = i / p.rope.n_t, pi = i - f * p.rope.n_t, pos = pos0 + f;
            const int64_t at = pos < p.n_sink_outside ? pos : p.ctx_start + (pos - p.n_sink_outside);
            double sn, cn;
            sincos(double(at) * p.rope.inv_freq_t[pi], &sn, &cn);
            t_cs[f * MAX_T_PAIRS + pi] = make_float2(float(cn), float(sn));
        }
        __syncthreads();
    }
#pragma unroll
    for (int it = 0; it < ITEMS; ++it) {
        const int item = tid + 256 * it, ti = item / CH, c = item % CH;
        u32x4 x = __builtin_bit_cast(u32x4, xv[it]);
        if constexpr (BACKWARD) {
            // (the lanes of a row are neighbours; summed in the order a kernel of its own for delta had)
            float acc = 0.f;
            if (ti < n_rows) {
#pragma unroll
                for (int e = 0; e < 4; ++e) acc += o0[it][e] * cl_f32(yv[it][e]) + o1[it][e] * cl_f32(yv[it][e + 4]);
            }
#pragma unroll
            for (int m = CH / 2; m >= 1; m >>= 1) acc += __shfl_xor(acc, m);
            if (ti < n_rows && c == 0) p.delta[head * p.row_stride + row0 + ti] = acc;
        } else {
            u32x4 qo;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int pi = c * 4 + e;
                const float2 w = pi < p.rope.n_t ? t_cs[frame[it] * MAX_T_PAIRS + pi] : cs[it][e];
                float re, im;
                rope_turn_scaled(cl_f32(qv[it][2 * e]), cl_f32(qv[it][2 * e + 1]), w, p.q_scale, re, im);
                qo[e] = cl_pack(re, im);
                rope_turn_key(cl_f32(xv[it][2 * e]), cl_f32(xv[it][2 * e + 1]), w, re, im);
                x[e] = cl_pack(re, im);
            }
            if (ti < n_rows && row0 + ti >= p.q_row0)
                *reinterpret_cast<u32x4*>(p.q_out + (int64_t(row0 + ti - p.q_row0) * p.H + head) * D + c * 8) = qo;
            if (ti >= n_rows) x = u32x4{};    // rows past the last hold zeros
        }
        *reinterpret_cast<u32x4*>(x_rows + ti * ROW + c * 8) = x;
        *reinterpret_cast<u16x8*>(y_rows + ti * ROW + c * 8) = yv[it];
    }
    __syncthreads();

    const int64_t at = head * p.head_stride + int64_t(kb) * (KBLOCK * D);
    // K-style image: unit u is (chunk, row); the row holds key swap23(row)
#pragma unroll
    for (int it = 0; it < ITEMS; ++it) {
        const int u = tid + 256 * it, from = swap23(u & 31) * ROW + (u >> 5) * 8;
        *reinterpret_cast<u16x8*>(p.x_k + at + u * 8) = *reinterpret_cast<const u16x8*>(x_rows + from);
        *reinterpret_cast<u16x8*>(p.y_k + at + u * 8) = *reinterpret_cast<const u16x8*>(y_rows + from);
    }
    // V^T-style image: unit (db, t, h, dd) holds rows 16 t + 8 h + e, e = 0..7, of feature 32 db + dd; a thread builds the units
    // of two neighbouring features from eight 4-byte LDS reads
    for (int up = tid; up < 16 * CH; up += 256) {
        const int ddp = up & 15, hh = (up >> 4) & 1, t = (up >> 5) & 1, db = up >> 6;
        const int from = (16 * t + 8 * hh) * ROW + 32 * db + 2 * ddp, u = ((db * 2 + t) * 2 + hh) * 32 + 2 * ddp;
#pragma unroll
        for (int which = 0; which < 2; ++which) {
            const unsigned short* rows = which == 0 ? x_rows : y_rows;
            uint16_t* dst = (which == 0 ? p.x_t : p.y_t) + at + u * 8;
            unsigned w[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) w[e] = *reinterpret_cast<const unsigned*>(rows + from + e * ROW);
            u32x4 lo, hi;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                lo[e] = __builtin_amdgcn_perm(w[2 * e + 1], w[2 * e], 0x05040100u);    // low halves: the first feature
                hi[e] = __builtin_amdgcn_perm(w[2 * e + 1], w[2 * e], 0x07060302u);    // high halves: the second
            }
            *reinterpret_cast<u32x4*>(dst) = lo;
            *reinterpret_cast<u32x4*>(dst + 8) = hi;
        }
    }
}

hipError_t launch_clip_layout(const ClipLayoutParams& p, int D, hipStream_t s) {
    if (p.rows <= 0) return hipSuccess;
    const int64_t grid = (int64_t(p.rows) + KBLOCK - 1) / KBLOCK * p.H;
    if (grid > 0x7FFFFFFF || (p.out32 == nullptr && p.rope.n_t > MAX_T_PAIRS)) return hipErrorInvalidValue;
    const dim3 blocks{unsigned(grid)}, threads(256);
    if (D == 128 && p.out32) hipLaunchKernelGGL((ll_clip_layout_kernel<128, true>), blocks, threads, 0, s, p);
    else if (D == 128) hipLaunchKernelGGL((ll_clip_layout_kernel<128, false>), blocks, threads, 0, s, p);
    else if (D == 64 && p.out32) hipLaunchKernelGGL((ll_clip_layout_kernel<64, true>), blocks, threads, 0, s, p);
    else if (D == 64) hipLaunchKernelGGL((ll_clip_layout_kernel<64, false>), blocks, threads, 0, s, p);
    else return hipErrorInvalidValue;
    return hipGetLastError();
}

}  // namespace ll
