// The rules of the memory pool (dev_pool.h) on the CPU (hip_fake.h).
#include "hip_fake.h"

#include "dev_pool.h"

using namespace eahr;

namespace {

constexpr size_t kMiB = size_t(1) << 20;

void* take(size_t bytes, bool host = false) {
    void* p = nullptr;
    fake::expect(pool_alloc(&p, bytes, host) == hipSuccess && p, "an allocation fails");
    return p;
}

// A block above the limit is freed by itself; what was kept stays.
void oversized() {
    const bool host = true;   // the smaller limit: 256 MiB
    void* small[4];
    for (auto& p : small) p = take(kMiB, host);
    void* big = take(kKeepHost + kMiB, host);
    for (auto& p : small) pool_release(p);
    const long before = fake::frees[1];
    pool_release(big);
    fake::expect(fake::frees[1] == before + 1, "an oversized block takes kept blocks with it");
    fake::expect(fake::in_use[1] == 4 * kMiB, "an oversized block is kept");
    // at the limit the oldest go first
    void* fill = take(kKeepHost - 2 * kMiB, host);
    pool_release(fill);
    fake::expect(fake::in_use[1] == kKeepHost, "the pool is not filled to its limit");
}

}  // namespace

int main() {
    oversized();
    std::printf("ok\n");
    return 0;
}
