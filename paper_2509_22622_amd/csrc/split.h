// Attention launches whose tiles' keys are dealt to several workgroups: where the partial results wait for the merge.
//
// A call enqueues two kernels, the splits and the merge, and the partial results pass between them through slots of a pool
// that the library holds (one per GPU, a static array: nothing is allocated).  Calls on any number of streams and threads,
// eager or captured, share the pool, so no slot belongs to a call beforehand: a workgroup that has a partial result claims
// a free slot by a compare-and-swap that leaves the call's token and its own number there, the merge finds it by them, and the
// last of its readers frees it.  A workgroup that finds its few candidates taken (several such calls at work at once) drops its result,
// and the merge computes the tile whole: slower, never wrong, and nobody waits for anybody.  A call's token is its own; the
// replays of a captured call share one, but two of them at once would write one output at once, which no caller may do.
// Partial results are written and read in different kernels, so kernel boundaries order them; of what happens within a kernel
// only the owner words are shared, and those are touched by device-wide atomics alone.
#pragma once
#include <hip/hip_runtime.h>

namespace ll {

constexpr int SPLIT_SLOTS = 512;     // two rounds of workgroups on 256 CUs
constexpr int SPLIT_PROBES = 4;      // slots a workgroup may take
constexpr int MAX_SPLITS = 32;
constexpr unsigned long long SPLIT_TOKENS = 1ull << 40;          // a token is 1 .. SPLIT_TOKENS - 1
static_assert(SPLIT_SLOTS <= 1 << 16, "an item has 16 bits");
struct SplitPool {
    unsigned long long owner[SPLIT_SLOTS];       // token << 24 | item << 8 | readers left; 0: free
    float2 ml[SPLIT_SLOTS][256];                 // (reference, row sum) per row
    float o[SPLIT_SLOTS][256 * 128];             // unnormalised output, in an order of the kernel's own
};

__device__ __forceinline__ int split_candidate(int item, int probe) { return (item + probe * (SPLIT_SLOTS / SPLIT_PROBES)) % SPLIT_SLOTS; }

hipError_t split_pool_address(SplitPool** pool);                 // on the current device (attn_kernel.hip)

// A slot for workgroup `item` of the launch, to be read by `readers` workgroups of the merge; -1 if its candidates are taken.
__device__ __forceinline__ int split_claim(SplitPool* pool, int item, unsigned long long token, int readers) {
    for (int c = 0; c < SPLIT_PROBES; ++c) {
        const int i = split_candidate(item, c);
        unsigned long long seen = 0;
        if (__hip_atomic_compare_exchange_strong(&pool->owner[i], &seen, token << 24 | unsigned(item << 8 | readers), __ATOMIC_RELAXED, __ATOMIC_RELAXED,
                                                 __HIP_MEMORY_SCOPE_AGENT))
            return i;
    }
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

}  // namespace ll
