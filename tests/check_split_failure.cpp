// A call with splits whose merge cannot be launched: it reports the error and gives back the slots its workgroups claimed, and
// no others.  The library as built, with stand-ins for the runtime's entry points in this program (no GPU).  argv[1]: the library.
#include <dlfcn.h>

#include <cstdio>
#include <cstdlib>
#include <cstring>

#include "../include/longlive.h"
#include "../paper_2509_22622_amd/csrc/kernels.h"
#include "../paper_2509_22622_amd/csrc/split.h"

static ll::SplitPool* pool;
static int launches, fail_at, copies;            // fail_at: the launch that fails, counted from 1
static bool in_attention;
static hipError_t last_error = hipSuccess;

extern "C" {
hipError_t hipLaunchKernel(const void*, dim3, dim3, void** args, size_t, hipStream_t) {
    if (!in_attention) return hipSuccess;
    const ll::AttnParams* p = static_cast<const ll::AttnParams*>(args[0]);
    if (!p->merge)                               // two of the workgroups have claimed their slots
        for (int item : {5, 130}) pool->owner[item] = p->token << 24 | unsigned(item << 8 | 1);
    const hipError_t e = ++launches == fail_at ? hipErrorLaunchFailure : hipSuccess;
    if (e != hipSuccess) last_error = e;
    return e;
}
hipError_t hipMemcpy(void* dst, const void* src, size_t n, hipMemcpyKind) {
    auto in_pool = [](const void* at) { return at >= pool && at < pool + 1; };
    if (!in_pool(dst) && !in_pool(src)) return hipSuccess;
    std::memcpy(dst, src, n);
    ++copies;
    return hipSuccess;
}
hipError_t hipMemset(void*, int, size_t) { return hipSuccess; }
hipError_t hipDeviceSynchronize() { return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipGetLastError() {
    const hipError_t e = last_error;
    last_error = hipSuccess;
    return e;
}
hipError_t hipGetDevice(int* d) { *d = 0; return hipSuccess; }
hipError_t hipFuncSetAttribute(const void*, hipFuncAttribute, int) { return hipSuccess; }
hipError_t hipGetSymbolAddress(void** at, const void*) { *at = pool; return hipSuccess; }
}

#define CHECK(x)                                                       \
    if (!(x)) {                                                        \
        std::printf("line %d: %s does not hold\n", __LINE__, #x);      \
        return 1;                                                      \
    }

int main(int, char** argv) {
    pool = static_cast<ll::SplitPool*>(std::calloc(1, sizeof(ll::SplitPool)));
    void* lib = dlopen(argv[1], RTLD_NOW | RTLD_LOCAL);
    CHECK(pool != nullptr && lib != nullptr);
    auto create = reinterpret_cast<decltype(&ll_cache_create)>(dlsym(lib, "ll_cache_create"));
    auto bytes = reinterpret_cast<decltype(&ll_cache_bytes)>(dlsym(lib, "ll_cache_bytes"));
    auto append = reinterpret_cast<decltype(&ll_chunk_append)>(dlsym(lib, "ll_chunk_append"));
    auto attend = reinterpret_cast<decltype(&ll_sink_window_attn)>(dlsym(lib, "ll_sink_window_attn"));
    char* const device = reinterpret_cast<char*>(0x7f0000000000);    // never touched
    ll_cache* cache = nullptr;
    CHECK(create(1, 4, 128, 190, 3, 20, 1, 10, 19, 10000.f, device, bytes(1, 4, 128, 190, 3, 20, 1), &cache) == LL_OK);
    for (int f = 0; f < 25; ++f) CHECK(append(cache, 0, f, 1, device, device, device, device, nullptr) == LL_OK);
    in_attention = true;
    last_error = hipErrorInvalidValue;           // an earlier call's: nothing here is to stumble over it
    const unsigned long long other = 1ull << 50 | 7 << 8 | 2;        // another call's
    pool->owner[6] = other;
    CHECK(attend(cache, 0, device, device, nullptr) == LL_OK);
    CHECK(launches == 2 && copies == 0);
    last_error = hipSuccess;
    pool->owner[5] = pool->owner[130] = 0;       // (the merge would have)
    launches = 0;
    fail_at = 1;
    CHECK(attend(cache, 0, device, device, nullptr) == LL_ERR_HIP);
    CHECK(launches == 1);                        // no merge without its splits
    CHECK(last_error == hipSuccess);             // reported, and not left for somebody else's call to find
    pool->owner[5] = pool->owner[130] = 0;
    launches = 0;
    fail_at = 2;
    CHECK(attend(cache, 0, device, device, nullptr) == LL_ERR_HIP);
    CHECK(launches == 2 && last_error == hipSuccess);
    CHECK(pool->owner[5] == 0 && pool->owner[130] == 0 && pool->owner[6] == other);
    std::printf("slots given back\n");
    return 0;
}
