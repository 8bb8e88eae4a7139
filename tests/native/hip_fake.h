// The HIP calls of the host runtime on the CPU, for tests of its error paths
// and of its memory pool: device memory is host memory, every launch, copy and
// clear that does not wait makes the device busy until a synchronisation, and
// single calls or whole budgets of memory can be made to fail.
#pragma once
#include <hip/hip_runtime.h>

#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>

namespace fake {

bool busy = false;              // work queued and not waited for
int step = 0;                   // the test's own step, for its messages
long calls = 0, fail_at = -1;   // the call with this number fails
size_t in_use[2] = {0, 0};      // bytes of device memory, of pinned memory
size_t budget[2] = {SIZE_MAX, SIZE_MAX};
long frees[2] = {0, 0};
std::map<char*, std::pair<size_t, int>> blocks;

[[noreturn]] inline void die(const char* what) {
    std::printf("FAILED: %s (step %d, call %ld, failing call %ld)\n", what, step, calls, fail_at);
    std::fflush(stdout);
    std::_Exit(1);
}
inline void expect(bool ok, const char* what) {
    if (!ok) die(what);
}
inline hipError_t call() { return calls++ == fail_at ? hipErrorUnknown : hipSuccess; }

inline hipError_t alloc(void** p, size_t bytes, int kind) {
    *p = nullptr;
    if (call() != hipSuccess) return hipErrorOutOfMemory;
    if (bytes > budget[kind] || in_use[kind] > budget[kind] - bytes) return hipErrorOutOfMemory;
    *p = std::calloc(1, bytes ? bytes : 1);
    if (!*p) return hipErrorOutOfMemory;
    blocks[static_cast<char*>(*p)] = {bytes, kind};
    in_use[kind] += bytes;
    return hipSuccess;
}
inline hipError_t release(void* p, int kind) {
    if (!p) return hipSuccess;
    busy = false;   // freeing waits for the device
    const auto it = blocks.find(static_cast<char*>(p));
    expect(it != blocks.end() && it->second.second == kind, "freed what was not allocated");
    in_use[kind] -= it->second.first;
    frees[kind] += 1;
    blocks.erase(it);
    std::free(p);
    return hipSuccess;
}
// [p, p + bytes) lies in one live allocation
inline bool inside(const void* p, size_t bytes) {
    char* c = static_cast<char*>(const_cast<void*>(p));
    auto it = blocks.upper_bound(c);
    if (!p || it == blocks.begin()) return false;
    --it;
    return c + bytes <= it->first + it->second.first;
}

}  // namespace fake

extern "C" {
hipError_t hipMalloc(void** p, size_t n) { return fake::alloc(p, n, 0); }
hipError_t hipHostMalloc(void** p, size_t n, unsigned) { return fake::alloc(p, n, 1); }
hipError_t hipFree(void* p) { return fake::release(p, 0); }
hipError_t hipHostFree(void* p) { return fake::release(p, 1); }
hipError_t hipGetDevice(int* d) { *d = 0; return hipSuccess; }
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipGetLastError() { return fake::call(); }
hipError_t hipPeekAtLastError() { return hipSuccess; }
const char* hipGetErrorString(hipError_t) { return "injected"; }
hipError_t hipDeviceSynchronize() { fake::busy = false; return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { fake::busy = false; return fake::call(); }
hipError_t hipStreamCreateWithFlags(hipStream_t* s, unsigned) { *s = nullptr; return fake::call(); }
hipError_t hipStreamDestroy(hipStream_t) { return hipSuccess; }
hipError_t hipEventCreate(hipEvent_t* e) { *e = nullptr; return hipSuccess; }
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float* ms, hipEvent_t, hipEvent_t) { *ms = 0.0f; return hipSuccess; }
hipError_t hipPointerGetAttributes(hipPointerAttribute_t*, const void*) { return hipErrorInvalidValue; }
hipError_t hipMemcpy(void* d, const void* s, size_t n, hipMemcpyKind) {
    if (fake::call() != hipSuccess) return hipErrorUnknown;
    std::memcpy(d, s, n);
    fake::busy = false;
    return hipSuccess;
}
hipError_t hipMemcpyAsync(void* d, const void* s, size_t n, hipMemcpyKind, hipStream_t) {
    if (fake::call() != hipSuccess) return hipErrorUnknown;
    std::memcpy(d, s, n);
    fake::busy = true;
    return hipSuccess;
}
hipError_t hipMemsetAsync(void* d, int v, size_t n, hipStream_t) {
    if (fake::call() != hipSuccess) return hipErrorUnknown;
    std::memset(d, v, n);
    fake::busy = true;
    return hipSuccess;
}
}
