// Device and pinned host memory of the library's handles.
//
// Allocating and freeing the storage of a segment costs more than building
// it: 200K x 768 rows are quantised in 0.28 ms, while hipMalloc and hipFree
// of their 0.77 GB take 1.1 ms, and 20 ms once a program frees memory faster
// than the driver clears it.  Blocks of closed handles are therefore kept for
// the next ones:
//  * at most kKeepDevice bytes per GPU and kKeepHost bytes of pinned memory,
//    in at most kKeepBlocks blocks each (requests search them one by one);
//    past that the blocks kept longest are freed first; a block larger than
//    the limit is freed at once;
//  * a kept block that no request has taken since the second index release
//    after its own, or for kKeepTicks closed states, is freed, so a program
//    that has moved on to other sizes gets its memory back;
//  * when an allocation fails, every kept block of that kind is freed and the
//    allocation tried again.
// Any thread may call; the lock is held across the bookkeeping only.  A block
// must be idle when it is released (no stream uses it any more), so it may be
// handed out to any stream at once.  Its contents are not cleared.
#pragma once
#include <hip/hip_runtime.h>

#include <cstddef>

namespace eahr {

constexpr size_t kKeepDevice = size_t(4) << 30;
constexpr size_t kKeepHost = size_t(256) << 20;
constexpr size_t kKeepBlocks = 256;

// At least `bytes` of memory of the current device, or of pinned host memory.
hipError_t pool_alloc(void** p, size_t bytes, bool host);
// Back to the pool (null is allowed).  The block must be idle.
void pool_release(void* p);
// Freed, not kept: for memory that no later request will match.
void pool_free(void* p);
// Frees the kept blocks of the current device, or the pinned ones: for callers
// whose own allocation has failed.
void pool_trim(bool host);
// A handle has been closed: the pool's clock goes on by `ticks`, and kept blocks
// that have been unused for kKeepTicks are freed.
constexpr int kKeepTicks = 96;
constexpr int kTicksIndex = kKeepTicks / 3;
constexpr int kTicksState = 1;
void pool_age(int ticks);

}  // namespace eahr
