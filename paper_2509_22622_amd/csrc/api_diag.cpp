// Diagnostics and tuning knobs (include/longlive_diag.h): the process-wide attention-kernel variant and the probe
// that measures what the matrix pipe sustains.  Not part of the method.
#include "../../include/longlive_diag.h"

#include "api_common.h"
#include "split.h"

using namespace ll;
using namespace ll_api;

extern "C" {

ll_status ll_set_attn_variant(int variant) {
    if (variant != 0 && !attn_variant_name(variant)) return fail(LL_ERR_INVALID_ARG, "no attention variant %d", variant);
    g_variant = variant;
    return LL_OK;
}
const char* ll_attn_variant_name(int variant) { return attn_variant_name(variant); }

extern "C++" {
namespace {
ll_status check_launch(int head_dim, int heads, int n_chunks, const int* rows, const int* kblocks) {
    if ((head_dim != 64 && head_dim != 128) || heads < 1 || heads > 1024 || n_chunks < 1 || n_chunks > MAX_ATTN_CHUNKS)
        return fail(LL_ERR_INVALID_ARG, "head_dim %d, heads %d or n_chunks %d out of range", head_dim, heads, n_chunks);
    for (int c = 0; c < n_chunks; ++c)
        if (rows[c] < 1 || kblocks[c] < 1) return fail(LL_ERR_INVALID_ARG, "chunk %d has %d rows and %d kblocks", c, rows[c], kblocks[c]);
    return LL_OK;
}
}  // namespace
}  // extern "C++"

ll_status ll_attn_key_groups(int head_dim, int heads, int n_chunks, const int* rows, const int* kblocks, int* groups) {
    if (!rows || !kblocks || !groups) return fail(LL_ERR_INVALID_ARG, "null pointer");
    const ll_status bad = check_launch(head_dim, heads, n_chunks, rows, kblocks);
    if (bad != LL_OK) return bad;
    *groups = attn_key_groups(attn_variant_default(head_dim, KBLOCK), heads, n_chunks, rows, kblocks);
    return LL_OK;
}

ll_status ll_attn_split(int head_dim, int fp8, int heads, int rows, int kblocks, int* groups, int* splits) {
    if (!groups || !splits) return fail(LL_ERR_INVALID_ARG, "null pointer");
    if ((head_dim != 64 && head_dim != 128) || heads < 1 || heads > 1024 || rows < 1 || kblocks < 1)
        return fail(LL_ERR_INVALID_ARG, "head_dim %d, heads %d, rows %d or kblocks %d out of range", head_dim, heads, rows, kblocks);
    const AttnSplit s = attn_split(attn_variant_default(head_dim, fp8 ? KBLOCK8 : KBLOCK), heads, 1, &rows, &kblocks);
    *groups = s.groups;
    *splits = s.splits;
    return LL_OK;
}

ll_status ll_attn_key_groups_fp8(int head_dim, int heads, int n_chunks, const int* rows, const int* kblocks, int* groups) {
    if (!rows || !kblocks || !groups) return fail(LL_ERR_INVALID_ARG, "null pointer");
    const ll_status bad = check_launch(head_dim, heads, n_chunks, rows, kblocks);
    if (bad != LL_OK) return bad;
    const int variant = attn_variant_default(head_dim, KBLOCK8);
    *groups = attn_takes_group8(variant, attn_split(variant, heads, n_chunks, rows, kblocks), heads, n_chunks, rows, kblocks) ? 4 : 1;
    return LL_OK;
}

ll_status ll_attn_clip_tail(int head_dim, int heads, int n_chunks, const int* rows, const int* kblocks, int* tiles, int* splits) {
    if (!rows || !kblocks || !tiles || !splits) return fail(LL_ERR_INVALID_ARG, "null pointer");
    const ll_status bad = check_launch(head_dim, heads, n_chunks, rows, kblocks);
    if (bad != LL_OK) return bad;
    const int variant = attn_variant_lse(head_dim);
    const AttnTail t = attn_tail(variant, attn_split(variant, heads, n_chunks, rows, kblocks), heads, n_chunks, rows, kblocks);
    *tiles = t.tiles;
    *splits = t.splits;
    return LL_OK;
}

ll_status ll_hold_split_slots(int first, int n, int hold) {
    if (first < 0 || n < 1 || first > SPLIT_SLOTS - n) return fail(LL_ERR_INVALID_ARG, "slots [%d, %d + %d) outside [0, %d)", first, first, n, SPLIT_SLOTS);
    constexpr unsigned long long HELD = 1;       // token 0, which no call has, and one reader, who never comes
    SplitPool* pool = nullptr;
    std::vector<unsigned long long> owner(n);
    hipError_t e = split_pool_address(&pool);
    if (e == hipSuccess) e = hipDeviceSynchronize();
    if (e == hipSuccess) e = hipMemcpy(owner.data(), pool->owner + first, n * sizeof(owner[0]), hipMemcpyDeviceToHost);
    if (e != hipSuccess) return hip_fail(e, "reading the slots' owners");
    for (unsigned long long& o : owner)
        if (o == (hold ? 0 : HELD)) o = hold ? HELD : 0;
    e = hipMemcpy(pool->owner + first, owner.data(), n * sizeof(owner[0]), hipMemcpyHostToDevice);
    if (e == hipSuccess) e = hipDeviceSynchronize();
    return e == hipSuccess ? LL_OK : hip_fail(e, "writing the slots' owners");
}

ll_status ll_split_slots_taken(int* taken) {
    if (!taken) return fail(LL_ERR_INVALID_ARG, "null pointer");
    SplitPool* pool = nullptr;
    std::vector<unsigned long long> owner(SPLIT_SLOTS + SPLIT_SPACES);
    hipError_t e = split_pool_address(&pool);
    if (e == hipSuccess) e = hipDeviceSynchronize();
    if (e == hipSuccess) e = hipMemcpy(owner.data(), pool->owner, owner.size() * sizeof(owner[0]), hipMemcpyDeviceToHost);
    if (e != hipSuccess) return hip_fail(e, "reading the slots' owners");
    *taken = int(owner.size() - std::count(owner.begin(), owner.end(), 0ull));
    return LL_OK;
}

ll_status ll_probe_mfma_rate(void* dev_scratch, size_t scratch_bytes, int workgroups, int iters, int random_operands,
                             double* tflops, double* clock_ghz, void* stream) {
    return ll_probe_mfma_mix(dev_scratch, scratch_bytes, workgroups, iters, random_operands, 0, 1, tflops, clock_ghz, stream);
}

ll_status ll_probe_mfma_mix(void* dev_scratch, size_t scratch_bytes, int workgroups, int iters, int random_operands,
                            int companion, int per_mfma, double* tflops, double* clock_ghz, void* stream) {
    if (!dev_scratch || !tflops || !clock_ghz) return fail(LL_ERR_INVALID_ARG, "null pointer");
    if (workgroups < 1 || workgroups > 4096 || iters < 1 || iters > (1 << 22))
        return fail(LL_ERR_INVALID_ARG, "workgroups %d or iters %d out of range", workgroups, iters);
    if (companion < PROBE_NONE || companion > PROBE_FP8_LDS || per_mfma < 1 || per_mfma > 2)
        return fail(LL_ERR_INVALID_ARG, "companion %d (0..11) or per_mfma %d (1, 2) out of range", companion, per_mfma);
    const size_t sink_bytes = size_t(workgroups) * 512 * sizeof(float);
    if (scratch_bytes < sink_bytes + 16) return fail(LL_ERR_BUFFER_TOO_SMALL, "scratch has %zu bytes, %zu needed", scratch_bytes, sink_bytes + 16);
    hipStream_t s = static_cast<hipStream_t>(stream);
    float* sink = static_cast<float*>(dev_scratch);
    unsigned long long* counters = reinterpret_cast<unsigned long long*>(static_cast<char*>(dev_scratch) + sink_bytes);
    hipEvent_t e0 = nullptr, e1 = nullptr;
    hipError_t e = hipEventCreate(&e0);
    if (e == hipSuccess) e = hipEventCreate(&e1);
    if (e == hipSuccess) e = launch_probe_mfma(sink, counters, workgroups, iters, random_operands, companion, per_mfma, s);   // clocks settle
    if (e == hipSuccess) e = hipEventRecord(e0, s);
    if (e == hipSuccess) e = launch_probe_mfma(sink, counters, workgroups, iters, random_operands, companion, per_mfma, s);
    if (e == hipSuccess) e = hipEventRecord(e1, s);
    if (e == hipSuccess) e = hipEventSynchronize(e1);
    float ms = 0.f;
    unsigned long long host[2] = {0, 0};
    if (e == hipSuccess) e = hipEventElapsedTime(&ms, e0, e1);
    if (e == hipSuccess) e = hipMemcpy(host, counters, sizeof host, hipMemcpyDeviceToHost);
    if (e0) (void)hipEventDestroy(e0);
    if (e1) (void)hipEventDestroy(e1);
    if (e != hipSuccess) return hip_fail(e, "ll_probe_mfma_mix");
    // 8 waves per workgroup, 16 MFMAs of 32x32x16 (2 * 32 * 32 * 16 flops; 32x32x64 for the fp8 kinds) per iteration and wave
    *tflops = double(workgroups) * 8 * iters * 16 * (companion >= PROBE_FP8_NONE ? 131072.0 : 32768.0) / (double(ms) * 1e9);
    *clock_ghz = host[1] ? double(host[0]) / (double(host[1]) * 10.0) : 0.0;
    return LL_OK;
}

}  // extern "C"
