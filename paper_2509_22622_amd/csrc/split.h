// Attention launches whose tiles' keys are dealt to several workgroups: where the partial results wait for the merge.
//
// A call enqueues two kernels, the splits and the merge, and the partial results pass between them through slots of a pool
// that the library holds (one per GPU, a static array: nothing is allocated).  Calls on any number of streams and threads,
// eager or captured, share the pool, so no slot belongs to a call beforehand: a workgroup that begins its share claims
// a free slot by a compare-and-swap that leaves the call's token and its own number there, the merge finds it by them, and the
// last of its readers frees it.  A workgroup that finds its few candidates taken (several such calls at work at once) computes
// nothing, and one workgroup of the merge computes the tile's shares one after another: slower, with the same arithmetic in the
// same order, so that a result does not depend on what else the GPU is doing.  us a call without any slot and with them: 1560 rows x
// 12 x 128 415 and 167, 190 rows x 4 x 128 99 and 19, 1560 rows x 3 x 64 with an 8-bit cache 132 and 30; how many calls find
// slots: two of the first at a time, four to five of the second.
// A call's token is its own; the replays of a captured call share one, but two of them at once would write one output at once,
// which no caller may do.
// Partial results are written and read in different kernels, so kernel boundaries order them; of what happens within a kernel
// only the owner words are shared, and those are touched by device-wide atomics alone.
// The sums over a tile computed in the merge do not fit beside its scores in registers; they are kept in one of a few spaces of
// the pool, taken for that time and handed on with release and acquire (the XCDs' L2 caches do not see one another's lines).  A
// workgroup that finds all of them taken waits for one: they are held by running workgroups only, which wait for nothing.
#pragma once
#include <hip/hip_runtime.h>

namespace ll {

constexpr int SPLIT_SLOTS = 512;     // two rounds of workgroups on 256 CUs
constexpr int SPLIT_SPACES = 128;    // tiles computed in merges at one time
constexpr int SPLIT_PROBES = 4;      // slots a workgroup may take
constexpr int MAX_SPLITS = 32;
constexpr unsigned long long SPLIT_TOKENS = 1ull << 40;          // a token is 1 .. SPLIT_TOKENS - 1
static_assert(SPLIT_SLOTS <= 1 << 16, "an item has 16 bits");
struct SplitPool {                               // the slots, and behind them the spaces
    unsigned long long owner[SPLIT_SLOTS + SPLIT_SPACES];        // slot: token << 24 | item << 8 | readers left; 0: free
    float2 ml[SPLIT_SLOTS][256];                 // (reference, row sum) per row
    float o[SPLIT_SLOTS + SPLIT_SPACES][256 * 128];              // unnormalised output, in an order of the kernel's own
};

__device__ __forceinline__ int split_candidate(int item, int probe) { return (item + probe * (SPLIT_SLOTS / SPLIT_PROBES)) % SPLIT_SLOTS; }

hipError_t split_pool_address(SplitPool** pool);                 // on the current device (attn_kernel.hip)

// One more share (ms, ls, xs) of a tile added to (m, l, o): sums relative to references m; a share without any weight has
// reference -inf and sums 0.  The merge and a tile computed whole in it both add their shares with this, in order.
__device__ __forceinline__ void split_weights(float& m, float& l, float ms, float ls, float& a, float& b) {
    const float top = fmaxf(m, ms), base = top == -INFINITY ? 0.f : top;
    a = __builtin_amdgcn_exp2f(m - base);
    b = __builtin_amdgcn_exp2f(ms - base);
    l = __builtin_fmaf(ls, b, l * a);
    m = top;
}
template <typename V>
__device__ __forceinline__ V split_add(V o, float a, V xs, float b) {
#pragma unroll
    for (int e = 0; e < 4; ++e) o[e] = __builtin_fmaf(xs[e], b, o[e] * a);
    return o;
}

// A slot for workgroup `item` of the launch, to be read by `readers` workgroups of the merge: what the claim of its candidate
// `probe` found there (0: claimed), and the candidate that could be claimed from `probe` on (-1: all taken).
__device__ __forceinline__ unsigned long long split_try(SplitPool* pool, int item, int probe, unsigned long long token, int readers) {
    unsigned long long seen = 0;
    __hip_atomic_compare_exchange_strong(&pool->owner[split_candidate(item, probe)], &seen, token << 24 | unsigned(item << 8 | readers), __ATOMIC_RELAXED,
                                         __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    return seen;
}
__device__ __forceinline__ int split_claim(SplitPool* pool, int item, unsigned long long token, int readers, int probe = 0) {
    for (; probe < SPLIT_PROBES; ++probe)
        if (split_try(pool, item, probe, token, readers) == 0) return split_candidate(item, probe);
    return -1;
}
// The slot that workgroup `item` of the launch with this token claimed; -1 if none.
__device__ __forceinline__ int split_find(SplitPool* pool, int item, unsigned long long token) {
    for (int c = 0; c < SPLIT_PROBES; ++c) {
        const int i = split_candidate(item, c);
        if (__hip_atomic_load(&pool->owner[i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) >> 8 == (token << 16 | unsigned(item))) return i;
    }
    return -1;
}
// One reader is done with the slot; the last one frees it.
__device__ __forceinline__ void split_release(SplitPool* pool, int slot) {
    const unsigned long long before = __hip_atomic_fetch_add(&pool->owner[slot], ~0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if ((before & 0xFF) == 1) __hip_atomic_store(&pool->owner[slot], 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// A space, looked for from number `from` on; and back.  One thread of a workgroup, with a barrier behind the one and before the other.
__device__ __forceinline__ int split_take_space(SplitPool* pool, int from) {
    for (int i = SPLIT_SLOTS + from % SPLIT_SPACES;; i = i + 1 == SPLIT_SLOTS + SPLIT_SPACES ? SPLIT_SLOTS : i + 1) {
        unsigned long long seen = 0;
        if (__hip_atomic_compare_exchange_strong(&pool->owner[i], &seen, 1ull, __ATOMIC_ACQUIRE, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) return i;
        __builtin_amdgcn_s_sleep(8);
    }
}
__device__ __forceinline__ void split_leave_space(SplitPool* pool, int space) {
    __hip_atomic_store(&pool->owner[space], 0ull, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_AGENT);
}

}  // namespace ll
