// ll_chunk_append for the 8-bit (E4M3) cache: the same 3D rotary embedding as append_kernel.hip (see there for
// the convention), then conversion of the rotated keys, the values and the rotated, pre-scaled queries to E4M3
// and the write of K and V into the ring slots in the fragment layout of the 32x32x64 fp8 MFMA (kernels.h).
// Memory bound; one pass over q, k, v.
//
// Quantisation: e4m3(x) = nearest E4M3 value, ties to even, after clamping |x| to 448 (the hardware conversion
// turns anything beyond 464 into NaN, so the clamp comes first).  K8 = e4m3(K' * 2^-k_exp),
// V8 = e4m3(V * 2^-v_exp), Q8 = e4m3(q' * log2(e)/sqrt(D) * 2^k_exp): the product Q8 . K8 needs no rescaling
// and 2^v_exp is applied once to the attention output.
//
// Work split: one workgroup per (32-slot segment of a frame, head), heads fastest as in append_kernel.hip; a segment is the part
// of one frame that falls into one half (row block R) of a kblock.  The workgroup builds the segment's share of the half's K
// and V images in LDS and stores whole 16-byte units where the segment covers them, single bytes at a frame boundary
// inside a unit.  As in append_kernel.hip a workgroup is a handful of memory round trips long, so its arguments are fetched in
// one go and every load is issued before the first value is touched; the V image is built two features at a time from
// one LDS read per key and byte permutes.  Half a kblock and not a whole one: two (head_dim 64: one) items a thread instead of
// four halve the chain of conversions between the round trips.  us with whole and half kblocks: 4680 rows x 12 x 128 19.4 and
// 16.7 (64.8 MB: 3.9 TB/s, a copy here takes 13), 2392 rows x 5 x 128 9.4 and 8.5, 598 rows 8.2 and 6.1 (all 2990 in one launch now: 10.2).
#include "kernels.h"

namespace ll {

typedef unsigned short u16x8 __attribute__((ext_vector_type(8)));
typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
typedef unsigned u32x2 __attribute__((ext_vector_type(2)));

__device__ inline float a8_bf16_to_f32(unsigned short b) { return __uint_as_float(unsigned(b) << 16); }
__device__ inline float a8_clamp(float x) { return fminf(fmaxf(x, -448.0f), 448.0f); }
// four floats -> four E4M3 bytes (byte 0 = a)
__device__ inline unsigned a8_pack4(float a, float b, float c, float d) {
    int w = __builtin_amdgcn_cvt_pk_fp8_f32(a8_clamp(a), a8_clamp(b), 0, false);
    w = __builtin_amdgcn_cvt_pk_fp8_f32(a8_clamp(c), a8_clamp(d), w, true);
    return unsigned(w);
}

template <int D, int FRAMES>
__global__ __launch_bounds__(256) void ll_append8_kernel(const AppendArgs<FRAMES> p) {
    constexpr int CH = D / 8;                 // 8-element chunks per (token, head) row
    constexpr int VROW = D + 16;              // padded LDS row of V bytes
    constexpr int HALF = KBLOCK8 / 2;
    constexpr int ITEMS = HALF * CH / 256;    // (token, chunk) items per thread
    __shared__ float2 t_cs[64];
    __shared__ __attribute__((aligned(16))) unsigned char k_img[HALF * D];
    __shared__ __attribute__((aligned(16))) unsigned char v_rows[HALF * VROW];

    const int tid = threadIdx.x;
    const int head = blockIdx.x % p.H;
    const int gseg = blockIdx.x / p.H;
    int begin[FRAMES];
    int64_t slots[FRAMES];
#pragma unroll
    for (int i = 0; i < FRAMES; ++i) {
        begin[i] = p.seg_begin[i];
        slots[i] = p.slot[i];
        asm volatile("" ::"s"(begin[i]), "s"(slots[i]));
    }
    asm volatile("" ::"s"(p.q), "s"(p.k), "s"(p.v), "s"(p.k8_cache), "s"(p.v8_cache), "s"(p.head_stride), "s"(p.rope.row_cs), "s"(p.rope.col_cs));
    int fi = 0, begin_fi = 0;
    int64_t slot0 = slots[0];
#pragma unroll
    for (int i = 1; i < FRAMES; ++i)
        if (i < p.n_frames && gseg >= begin[i]) {
            fi = i;
            begin_fi = begin[i];
            slot0 = slots[i];
        }
    const int seg = gseg - begin_fi;
    const int64_t hb = slot0 / HALF + seg;                         // half kblock this segment is in
    const int64_t s_begin = max(slot0, hb * HALF);
    const int64_t s_end = min(slot0 + p.P, (hb + 1) * HALF);
    const int k_lo = int(s_begin - hb * HALF);                     // slots [k_lo, k_hi) of the half
    const int k_hi = int(s_end - hb * HALF);
    const int ntok = k_hi - k_lo;
    const int tok0 = int(s_begin - slot0);                         // token inside the frame
    const int n_t = p.rope.n_t, n_h = p.rope.n_h;
    const int64_t row0 = int64_t(fi) * p.P + tok0;                 // first input row
    const int y0 = tok0 / p.grid_w, x0 = tok0 - y0 * p.grid_w;     // grid position of the segment's first token

    // ---- every load first
    u16x8 qv[ITEMS], kv[ITEMS], vv[ITEMS];
    float2 cs[ITEMS][4];
    bool live[ITEMS];
#pragma unroll
    for (int it = 0; it < ITEMS; ++it) {
        const int item = tid + 256 * it;
        const int ti = item / CH, c = item % CH;
        live[it] = ti < ntok;
        qv[it] = kv[it] = vv[it] = u16x8{};
#pragma unroll
        for (int e = 0; e < 4; ++e) cs[it][e] = make_float2(1.f, 0.f);
        if (live[it]) {
            const int64_t src = ((row0 + ti) * p.H + head) * D + c * 8;
            qv[it] = *reinterpret_cast<const u16x8*>(p.q + src);
            kv[it] = *reinterpret_cast<const u16x8*>(p.k + src);
            vv[it] = *reinterpret_cast<const u16x8*>(p.v + src);
            const int dy = (x0 + ti) / p.grid_w, y = y0 + dy, x = x0 + ti - dy * p.grid_w;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int pi = c * 4 + e;
                if (pi >= n_t)
                    cs[it][e] = *(pi < n_t + n_h ? p.rope.row_cs + (y * n_h + (pi - n_t)) : p.rope.col_cs + (x * p.rope.n_w + (pi - n_t - n_h)));
            }
        }
    }
    if (tid < n_t) t_cs[tid] = p.t_cs[fi][tid];                  // frame-axis (cos, sin), made on the host in double
    __syncthreads();

#pragma unroll
    for (int it = 0; it < ITEMS; ++it) {
        if (!live[it]) continue;
        const int item = tid + 256 * it;
        const int ti = item / CH, c = item % CH;
        const int64_t src = ((row0 + ti) * p.H + head) * D + c * 8;
        float qo[8], ko[8];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int pi = c * 4 + e;
            float2 w = cs[it][e];
            if (pi < n_t) w = t_cs[pi];
            const float qr = a8_bf16_to_f32(qv[it][2 * e]), qi = a8_bf16_to_f32(qv[it][2 * e + 1]);
            const float kr = a8_bf16_to_f32(kv[it][2 * e]), ki = a8_bf16_to_f32(kv[it][2 * e + 1]);
            rope_turn_scaled(qr, qi, w, p.q_scale, qo[2 * e], qo[2 * e + 1]);
            rope_turn_scaled(kr, ki, w, p.k_mul, ko[2 * e], ko[2 * e + 1]);
        }
        const u32x2 q8 = {a8_pack4(qo[0], qo[1], qo[2], qo[3]), a8_pack4(qo[4], qo[5], qo[6], qo[7])};
        const u32x2 k8 = {a8_pack4(ko[0], ko[1], ko[2], ko[3]), a8_pack4(ko[4], ko[5], ko[6], ko[7])};
        float vf[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) vf[e] = a8_bf16_to_f32(vv[it][e]) * p.v_mul;
        const u32x2 v8 = {a8_pack4(vf[0], vf[1], vf[2], vf[3]), a8_pack4(vf[4], vf[5], vf[6], vf[7])};
        *reinterpret_cast<u32x2*>(p.q8_out + src) = q8;
        *reinterpret_cast<u32x2*>(k_img + k8_byte_offset(k_lo + ti, c * 8, D)) = k8;     // 8 features stay together
        *reinterpret_cast<u32x2*>(v_rows + (k_lo + ti) * VROW + c * 8) = v8;
    }
    __syncthreads();

    const int R = int(hb & 1);
    unsigned char* kdst = p.k8_cache + head * p.head_stride + hb * (HALF * D);                    // row block R's pieces side by side
    unsigned char* vdst = p.v8_cache + head * p.head_stride + (hb >> 1) * (KBLOCK8 * D) + R * 1024;   // piece (db, R) at db * 2 KB
    // K image: unit u = (piece, lane); lane = 32h + r holds key r of the half
    for (int u = tid; u < HALF * D / 16; u += 256) {
        const int key = u & 31;
        if (key >= k_lo && key < k_hi)
            *reinterpret_cast<u32x4*>(kdst + u * 16) = *reinterpret_cast<const u32x4*>(k_img + u * 16);
    }
    // V image: unit (db, h, dd); byte 4g + j holds key 8g + 4h + j of the half at feature 32db + dd.  A thread builds the units of
    // two neighbouring features.
    constexpr int FPT = 2;
    for (int uq = tid; uq < HALF * D / 16 / FPT; uq += 256) {
        const int u = uq * FPT, dd = u & 31, hh = (u >> 5) & 1, db = u >> 6;
        const int d = 32 * db + dd;
        const int first = 4 * hh;                               // keys first + 8g + j
        unsigned char* dst = vdst + db * 2048 + (hh * 32 + dd) * 16;
        u32x4 o[FPT];                                           // [feature][g]
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            unsigned w[4];                                      // one key each, its features (rows outside: not used)
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                w[j] = *reinterpret_cast<const unsigned short*>(v_rows + (first + 8 * g + j) * VROW + d);
            }
            const unsigned a = __builtin_amdgcn_perm(w[1], w[0], 0x05010400u), b = __builtin_amdgcn_perm(w[3], w[2], 0x05010400u);
            o[0][g] = __builtin_amdgcn_perm(b, a, 0x05040100u);
            o[1][g] = __builtin_amdgcn_perm(b, a, 0x07060302u);
        }
        if (first >= k_lo && first + 28 <= k_hi) {
#pragma unroll
            for (int f = 0; f < FPT; ++f) *reinterpret_cast<u32x4*>(dst + f * 16) = o[f];
        } else {
#pragma unroll
            for (int f = 0; f < FPT; ++f)
#pragma unroll
                for (int g = 0; g < 4; ++g)
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        const int kk = first + 8 * g + j;
                        if (kk >= k_lo && kk < k_hi) dst[f * 16 + 4 * g + j] = (unsigned char)(o[f][g] >> (8 * j));
                    }
        }
    }
}

template <int FRAMES>
static hipError_t launch(const AppendArgs<FRAMES>& p, hipStream_t s) {
    const int nseg = p.seg_begin[p.n_frames];
    if (nseg <= 0) return hipSuccess;
    if (p.n_frames > FRAMES || p.rope.n_t > MAX_T_PAIRS) return hipErrorInvalidValue;
    if (int64_t(nseg) * p.H > 0x7FFFFFFF) return hipErrorInvalidValue;
    if (p.D != 128 && p.D != 64) return hipErrorInvalidValue;
    void (*const kernel)(const AppendArgs<FRAMES>) = p.D == 128 ? ll_append8_kernel<128, FRAMES> : ll_append8_kernel<64, FRAMES>;
    return launch_kernel(reinterpret_cast<const void*>(kernel), dim3(unsigned(nseg) * unsigned(p.H)), dim3(256), &p, 0, s);
}
hipError_t launch_append8(const AppendParams& p, hipStream_t s) { return launch(p, s); }
hipError_t launch_append8(const FewAppendParams& p, hipStream_t s) { return launch(p, s); }

// Copy one frame's K and V codes out of the cache layout into [P, H, D] bytes.
__global__ __launch_bounds__(256) void ll_read_frame8_kernel(const ReadFrameParams p) {
    const int64_t n = int64_t(p.P) * p.H * p.D;
    for (int64_t i = blockIdx.x * 256LL + threadIdx.x; i < n; i += int64_t(gridDim.x) * 256) {
        const int d = int(i % p.D);
        const int head = int((i / p.D) % p.H);
        const int64_t tok = i / (int64_t(p.D) * p.H);
        const int64_t slot = p.slot + tok;
        const int64_t base = head * p.head_stride + (slot / KBLOCK8) * (KBLOCK8 * p.D);
        const int k = int(slot % KBLOCK8);
        if (p.k8_out) p.k8_out[i] = p.k8_cache[base + k8_byte_offset(k, d, p.D)];
        if (p.v8_out) p.v8_out[i] = p.v8_cache[base + v8_byte_offset(k, d)];
    }
}

hipError_t launch_read_frame8(const ReadFrameParams& p, hipStream_t s) {
    hipLaunchKernelGGL(ll_read_frame8_kernel, dim3(512), dim3(256), 0, s, p);
    return hipGetLastError();
}

}  // namespace ll
