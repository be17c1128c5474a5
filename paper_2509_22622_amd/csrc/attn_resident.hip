// Attention of many query rows over a key set that fits into a CU's LDS whole (cross-attention over a prompt of up to
// 256 tokens at head_dim 128, 512 at 64): the same 16x16x32 MFMA formulation, fragments and cache layout as
// attn_stream16.hip.
//
// What bounds it: the queries in and the outputs out.  At 226 tokens x 23400 rows x 12 heads x 128 these are 144 MB
// (29 us at a copy's rate) next to some 16 us of matrix time.  A kernel that streams the keys through a ring for every
// tile of 256 rows spends most of a tile's life loading queries, filling the ring and storing outputs, one after the
// other.  Here a workgroup brings the keys and values of one head into LDS once and its eight waves then go through
// their rows on their own: blocks of 32 rows, no barrier, no ring, the next block's queries on their way while this
// block is computed, and the waves of a CU in different phases.  Measured against the streaming kernels, us:
// 226 tokens x 23400 rows x 12 x 128 75 -> 55 (16 tokens, all memory: 47 -> 36, 4.0 TB/s), x 24 heads 137 -> 101;
// 1200 rows x 77 tokens x 24 x 64 10 -> 7.  Rows that went to memory in the lanes' own order (64-byte loads, 32-byte stores) took
// 46 us at 16 tokens.  The fragments' reads were then left to the compiler, which put each in front of its MFMAs
// (no room for more beside the next queries), and the matrix work did not hide under the memory's; by hand, in turn on one card (they
// differ by 8 %): 226 tokens x 23400 x 12 x 128 48.0 -> 47.1, 20000 x 400 x 12 x 64 39.6 -> 37.8, 9000 x 500 x 6 x 64 15.4 -> 14.8.
#include "kernels.h"

#include <algorithm>

namespace ll {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
typedef unsigned u32x2 __attribute__((ext_vector_type(2)));

constexpr int RES_WAVES = 8, RES_THREADS = 64 * RES_WAVES;
constexpr int RES_KEY_BYTES = 128 * 1024;        // keys and values; 16 rows per wave come on top: 160 KB at head_dim 128
constexpr float RES_SLACK = 6.0f;                // log2 units: weights stay below 2^6 between rescales

__device__ __forceinline__ unsigned res_pack_bf16(float a, float b) {
    f32x2 v = {a, b};
    return __builtin_bit_cast(unsigned, __builtin_convertvector(v, bf16x2));
}

// LDS reads the compiler does not see (attn_stream.hip): `dst` is pending until res_lds_wait<N>(dst) with N reads issued after it
__device__ __forceinline__ void res_lds_read(u32x4& dst, unsigned addr, int offset) {
    asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(dst) : "v"(addr), "n"(offset));
}
template <int N>
__device__ __forceinline__ void res_lds_wait(u32x4& x) {
    asm volatile("s_waitcnt lgkmcnt(%1)" : "+v"(x) : "n"(N));
}

// FRAG: the output goes out in the output projection's fragment order (AttnParams::out_frag)
template <int D, bool FRAG>
__global__ __launch_bounds__(RES_THREADS) __attribute__((amdgpu_waves_per_eu(2, 2))) void ll_attn_resident_kernel(const ResidentParams p) {
    constexpr int KS = D / 16, NV = D / 16, NQ = D / 32, NF = KS + NV;
    constexpr int KB_BYTES = KBLOCK * D * 2, STAGE_BYTES = 2 * KB_BYTES;      // [K kblock | V kblock]
    extern __shared__ __attribute__((aligned(16))) char lds[];
    const int tid = threadIdx.x, lane = tid & 63, n = lane & 15, g = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int head = blockIdx.x % p.H, part = blockIdx.x / p.H;               // workgroups of all heads walk the same rows
    const int T = p.n_kblocks, tail = p.n_keys - (T - 1) * KBLOCK;            // keys in the last kblock
    const int n_blocks = (p.n_rows + 31) >> 5;
    const int lo = int(int64_t(n_blocks) * part / p.parts), hi = int(int64_t(n_blocks) * (part + 1) / p.parts);

    {
        const char* kbase = reinterpret_cast<const char*>(p.k_cache + head * p.head_stride);
        const char* vbase = reinterpret_cast<const char*>(p.v_cache + head * p.head_stride);
        // K fragments are permuted on the way, as in attn_stream16.hip: lane (c, m, r) fetches stored row
        // (r & 7) + 8 m + 16 (r >> 3) of 16-byte chunk c
        const int hc = lane >> 5, m = (lane >> 4) & 1, r = lane & 15;
        const unsigned k_off = unsigned(hc * 32 + (r & 7) + 8 * m + 16 * (r >> 3)) * 16u, v_off = lane * 16u;
        for (int f = wave; f < T * NF; f += RES_WAVES) {
            const int kb = f / NF, fr = f % NF;
            const char* src = (fr < KS ? kbase + fr * 1024 + k_off : vbase + (fr - KS) * 1024 + v_off) + int64_t(kb) * KB_BYTES;
            __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)(src),
                                             (__attribute__((address_space(3))) void*)(lds + kb * STAGE_BYTES + fr * 1024), 16, 0, 0);
        }
    }
    // Rows come and go as whole rows (a load or store instruction covers 64 / CH of them), so that memory sees full
    // lines; between that order and the lanes' own (row n, features 32 s + 8 g ..) they pass through 16 rows of LDS of the
    // wave's own, chunk c of row r at place c ^ r (no bank conflicts).
    constexpr int CH = D / 8, RPI = 64 / CH;     // 16-byte chunks per row, rows per instruction
    char* turn = lds + T * STAGE_BYTES + wave * (16 * D * 2);
    const int line_row = lane / CH, line_c = lane % CH;
    auto place = [&](int row, int c) { return turn + row * (D * 2) + ((c ^ row) & (CH - 1)) * 16; };
    u32x4 q_next[2][NQ];
    auto fetch = [&](int b) {
#pragma unroll
        for (int qb = 0; qb < 2; ++qb)
#pragma unroll
            for (int i = 0; i < NQ; ++i) {
                const int row = min(32 * b + 16 * qb + i * RPI + line_row, p.n_rows - 1);
                q_next[qb][i] = *reinterpret_cast<const u32x4*>(p.q + (int64_t(row) * p.H + head) * D + line_c * 8);
            }
    };
    fetch(min(lo + wave, n_blocks - 1));
    __builtin_amdgcn_s_waitcnt((0x7 << 4) | (0xF << 8));                      // vmcnt(0): what this wave brings into LDS has landed
    __syncthreads();
    if (tail < KBLOCK) {                         // slots past the last key may hold anything, even NaN
        uint16_t* v_last = reinterpret_cast<uint16_t*>(lds + (T - 1) * STAGE_BYTES + KB_BYTES);
        for (int i = tid; i < KBLOCK * D; i += RES_THREADS)
            if (i / D >= tail) v_last[v_elem_offset(i / D, i % D)] = 0;
        __syncthreads();
    }

    const char* lane_lds = lds + g * 512 + n * 16;
    auto frag = [&](int kb, int kind, int f) {   // as attn_stream16.hip reads them
        return *reinterpret_cast<const bf16x8*>(lane_lds + kb * STAGE_BYTES + kind * KB_BYTES + (f >> 1) * 2048 + (f & 1) * 256);
    };
    auto col_max = [&](float x) {
        x = fmaxf(x, __shfl_xor(x, 16));
        return fmaxf(x, __shfl_xor(x, 32));
    };

    const float c = p.scale_log2e;               // applied to the scores in fp32: the queries are not rounded again
    bf16x8 qf[2][NQ];
    auto take_queries = [&]() {
#pragma unroll
        for (int qb = 0; qb < 2; ++qb) {
#pragma unroll
            for (int i = 0; i < NQ; ++i) *reinterpret_cast<u32x4*>(place(i * RPI + line_row, line_c)) = q_next[qb][i];
#pragma unroll
            for (int s = 0; s < NQ; ++s) qf[qb][s] = *reinterpret_cast<const bf16x8*>(place(n, 4 * s + g));
        }
    };
    take_queries();
    for (int b = lo + wave; b < hi; b += RES_WAVES) {
        fetch(min(b + RES_WAVES, n_blocks - 1));

        f32x4 o[NV][2];
        float lsum[2], mref[2];                  // row sums, references (log2 domain)
#pragma unroll
        for (int qb = 0; qb < 2; ++qb) {
            lsum[qb] = 0.f;
#pragma unroll
            for (int f = 0; f < NV; ++f) o[f][qb] = f32x4{0.f, 0.f, 0.f, 0.f};
        }
        auto scores = [&](int kb, f32x4 (&s)[2][2]) {
#pragma unroll
            for (int k = 0; k < KS; ++k) {
                const bf16x8 a = frag(kb, 0, k);
#pragma unroll
                for (int qb = 0; qb < 2; ++qb) {
                    if (k < 2) s[k & 1][qb] = f32x4{0.f, 0.f, 0.f, 0.f};
                    s[k & 1][qb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, qf[qb][k >> 1], s[k & 1][qb], 0, 0, 0);
                }
            }
        };
        auto mask_tail = [&](f32x4 (&s)[2][2]) {                  // register j of group m is key 8 g + 4 m + j
#pragma unroll
            for (int m = 0; m < 2; ++m)
#pragma unroll
                for (int qb = 0; qb < 2; ++qb) {
                    const f32x4 x = s[m][qb];
                    const int left = tail - 8 * g - 4 * m;
                    s[m][qb] = f32x4{left > 0 ? x[0] : -INFINITY, left > 1 ? x[1] : -INFINITY,
                                     left > 2 ? x[2] : -INFINITY, left > 3 ? x[3] : -INFINITY};
                }
        };
        auto max_s = [&](const f32x4 (&s)[2][2], int qb) {
            float m = fmaxf(fmaxf(s[0][qb][0], s[0][qb][1]), s[0][qb][2]);
            m = fmaxf(fmaxf(m, s[0][qb][3]), s[1][qb][0]);
            m = fmaxf(fmaxf(m, s[1][qb][1]), s[1][qb][2]);
            return fmaxf(m, s[1][qb][3]);
        };
        auto weights = [&](const f32x4 (&s)[2][2], int qb, int w, u32x4 (&pb)[2]) {
            const float e0 = __builtin_amdgcn_exp2f(__builtin_fmaf(s[w >> 1][qb][2 * (w & 1)], c, -mref[qb]));
            const float e1 = __builtin_amdgcn_exp2f(__builtin_fmaf(s[w >> 1][qb][2 * (w & 1) + 1], c, -mref[qb]));
            lsum[qb] += e0;
            lsum[qb] += e1;
            pb[qb][w] = res_pack_bf16(e0, e1);
        };

        // A kblock is KS + NV fragments, two MFMAs each: those of keys kb + 1, with the weights of kb behind them, then those of
        // values kb, with the maximum over the new scores.  The fragments are read by hand, AHEAD before their MFMAs, into a
        // ring of four buffers.
        f32x4 sA[2][2], sB[2][2];
        scores(0, sA);
        if (T == 1 && tail < KBLOCK) mask_tail(sA);
#pragma unroll
        for (int qb = 0; qb < 2; ++qb) mref[qb] = col_max(max_s(sA, qb)) * c;     // the first kblock holds a live key: finite
        float mx[2];                             // largest score of the kblock to come among this lane's keys
        // (before that kblock's weights: the reference follows where a score exceeds it by far)
        auto follow = [&]() {
            if (__any(mx[0] * c > mref[0] + RES_SLACK || mx[1] * c > mref[1] + RES_SLACK)) {
#pragma unroll
                for (int qb = 0; qb < 2; ++qb) {
                    const float m = fmaxf(mref[qb], col_max(mx[qb]) * c);
                    const float alpha = __builtin_amdgcn_exp2f(mref[qb] - m);
                    mref[qb] = m;
                    lsum[qb] *= alpha;
#pragma unroll
                    for (int f = 0; f < NV; ++f) o[f][qb] *= alpha;
                }
            }
        };
        constexpr int AHEAD = 3, RING = 4, NFR = KS + NV;
        u32x4 fr[RING];
        u32x4 pb[2];
        // fragment j of kblock kb's NFR, from NFR on those of the next one; `at`: this lane's place in kblock kb
        auto read = [&](int j, unsigned at) {
            const int next = j / NFR, f = j % NFR < KS ? j % NFR : j % NFR - KS;
            res_lds_read(fr[j % RING], at + (next + (j % NFR < KS ? 1 : 0)) * STAGE_BYTES, (j % NFR < KS ? 0 : KB_BYTES) + (f >> 1) * 2048 + (f & 1) * 256);
        };
        static_assert(NFR % RING == 0 && STAGE_BYTES + KB_BYTES < 65536, "a fragment's buffer does not depend on the kblock");
        unsigned at = (unsigned)(size_t)(__attribute__((address_space(3))) const char*)lane_lds;
        auto step = [&](f32x4 (&cur)[2][2], f32x4 (&nxt)[2][2]) {
#pragma unroll
            for (int j = 0; j < NFR; ++j) {
                read(j + AHEAD, at);
                res_lds_wait<AHEAD>(fr[j % RING]);
                const bf16x8 a = __builtin_bit_cast(bf16x8, fr[j % RING]);
#pragma unroll
                for (int qb = 0; qb < 2; ++qb) {
                    if (j < KS) nxt[j & 1][qb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, qf[qb][j >> 1], j < 2 ? f32x4{0.f, 0.f, 0.f, 0.f} : nxt[j & 1][qb], 0, 0, 0);
                    else o[j - KS][qb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, __builtin_bit_cast(bf16x8, pb[qb]), o[j - KS][qb], 0, 0, 0);
                }
                if (j < KS) {
#pragma unroll
                    for (int w = j * 8 / KS; w < (j + 1) * 8 / KS; ++w) weights(cur, w / 4, w % 4, pb);
                } else if (j >= NFR - 2) {
                    mx[j - (NFR - 2)] = max_s(nxt, j - (NFR - 2));
                }
                __builtin_amdgcn_sched_barrier(0);
            }
            at += STAGE_BYTES;
        };
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");        // nothing else is counted from here on
        __builtin_amdgcn_sched_barrier(0);
        if (T > 1) {
#pragma unroll
            for (int j = 0; j < AHEAD; ++j) read(j, at);
            step(sA, sB);
            int kb = 1;
            for (; kb + 2 < T; kb += 2) {        // (the two score sets swap roles)
                follow();
                step(sB, sA);
                follow();
                step(sA, sB);
            }
            if (kb + 1 < T) {
                follow();
                step(sB, sA);
            } else {
#pragma unroll
                for (int m = 0; m < 2; ++m)
#pragma unroll
                    for (int qb = 0; qb < 2; ++qb) sA[m][qb] = sB[m][qb];
            }
#pragma unroll
            for (int j = 0; j < AHEAD; ++j) res_lds_wait<0>(fr[j]);               // (read for a kblock past the last: not used)
            if (tail < KBLOCK) {
                mask_tail(sA);
#pragma unroll
                for (int qb = 0; qb < 2; ++qb) mx[qb] = max_s(sA, qb);
            }
            follow();
        }
#pragma unroll
        for (int w = 0; w < 8; ++w) weights(sA, w / 4, w % 4, pb);
#pragma unroll
        for (int f = 0; f < NV; ++f) {
            const bf16x8 a = frag(T - 1, 1, f);
#pragma unroll
            for (int qb = 0; qb < 2; ++qb)
                o[f][qb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, __builtin_bit_cast(bf16x8, pb[qb]), o[f][qb], 0, 0, 0);
        }

        // the next block's queries are waited for before the stores are issued: one counter counts both, in order
        take_queries();
        __builtin_amdgcn_sched_barrier(0);

        // out[row][head][16 dq + 4 g + j] = O^T block (dq, qb) register j, divided by the row sum
#pragma unroll
        for (int qb = 0; qb < 2; ++qb) {
            float l = lsum[qb];
            l += __shfl_xor(l, 16);
            l += __shfl_xor(l, 32);
            const float inv = 1.0f / l;
            if constexpr (FRAG) {                // 1 KB per store instruction as it is
                const int row = 32 * b + 16 * qb + n;
                if (row >= p.n_rows) continue;
#pragma unroll
                for (int t = 0; t < D / 32; ++t) {
                    const f32x4 x = o[2 * t][qb] * inv, y = o[2 * t + 1][qb] * inv;
                    const u32x4 w = {res_pack_bf16(x[0], x[1]), res_pack_bf16(x[2], x[3]), res_pack_bf16(y[0], y[1]), res_pack_bf16(y[2], y[3])};
                    *reinterpret_cast<u32x4*>(p.out_frag + op_frag_offset(row, head * (D / 32) + t, g, p.H * (D / 32))) = w;
                }
            } else {
#pragma unroll
                for (int dq = 0; dq < NV; ++dq) {
                    const f32x4 x = o[dq][qb] * inv;
                    const u32x2 w = {res_pack_bf16(x[0], x[1]), res_pack_bf16(x[2], x[3])};
                    *reinterpret_cast<u32x2*>(place(n, 2 * dq + (g >> 1)) + (g & 1) * 8) = w;
                }
#pragma unroll
                for (int i = 0; i < NQ; ++i) {
                    const u32x4 w = *reinterpret_cast<const u32x4*>(place(i * RPI + line_row, line_c));
                    const int row = 32 * b + 16 * qb + i * RPI + line_row;
                    if (row < p.n_rows) *reinterpret_cast<u32x4*>(p.out + (int64_t(row) * p.H + head) * D + line_c * 8) = w;
                }
            }
        }
    }
}

bool attn_resident_fits(int D, int n_kblocks) { return n_kblocks * 2 * KBLOCK * D * 2 <= RES_KEY_BYTES; }

hipError_t launch_attn_resident(const ResidentParams& p_in, int D, hipStream_t s) {
    ResidentParams p = p_in;
    p.n_kblocks = (p.n_keys + KBLOCK - 1) / KBLOCK;
    if (p.n_keys < 1 || p.n_rows < 1 || (D != 64 && D != 128) || !attn_resident_fits(D, p.n_kblocks)) return hipErrorInvalidValue;
    // one workgroup per CU, every head the same number of them, at least one block of rows each
    const int blocks = (p.n_rows + 31) / 32;
    p.parts = std::max(1, std::min(256 / p.H, blocks));
    const int lds = p.n_kblocks * 2 * KBLOCK * D * 2 + RES_WAVES * 16 * D * 2;
    static bool attr_set[2][2] = {};
    void (*const kernel)(const ResidentParams) = p.out_frag != nullptr
        ? (D == 128 ? ll_attn_resident_kernel<128, true> : ll_attn_resident_kernel<64, true>)
        : (D == 128 ? ll_attn_resident_kernel<128, false> : ll_attn_resident_kernel<64, false>);
    bool& set = attr_set[D == 128][p.out_frag != nullptr];
    if (!set) {
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize,
                                           RES_KEY_BYTES + RES_WAVES * 16 * D * 2);
        if (e != hipSuccess) return e;
        set = true;
    }
    hipLaunchKernelGGL(kernel, dim3(unsigned(p.H) * unsigned(p.parts)), dim3(RES_THREADS), lds, s, p);
    return hipGetLastError();
}

}  // namespace ll
