// The rules of the memory pool (dev_pool.h) on the CPU (hip_fake.h).
#include "hip_fake.h"

#include "dev_pool.h"
#include "eahr.h"

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

// A block nobody asks for again goes at the third index release counting its
// own owner's, or after kKeepTicks closed states; one in use in turn stays.
void ages() {
    pool_age(kKeepTicks);
    fake::expect(fake::in_use[0] == 0 && fake::in_use[1] == 0, "old blocks stay");
    pool_release(take(kMiB));
    for (int i = 0; i < 2; ++i) pool_age(kTicksIndex);
    fake::expect(fake::in_use[0] == kMiB, "a block goes at the second index release");
    pool_age(kTicksIndex);
    fake::expect(fake::in_use[0] == 0, "a block outlives the third index release");
    void* other = take(3 * kMiB);
    pool_release(take(kMiB));
    for (int i = 0; i < kKeepTicks - 1; ++i) pool_age(kTicksState);
    pool_release(other);
    fake::expect(fake::in_use[0] == 5 * kMiB, "a block goes early");   // 3 MiB round up to 4
    pool_age(kTicksState);
    fake::expect(fake::in_use[0] == 4 * kMiB, "not only the old block goes");
    for (int i = 0; i < 4 * kKeepTicks; ++i) {   // taken now and then
        if (i % 64 == 0) pool_release(take(3 * kMiB));
        pool_age(kTicksState);
        fake::expect(fake::frees[0] == 2 && fake::in_use[0] == 4 * kMiB, "a block in use in turn goes");
    }
}

// The public call frees what is kept and nothing that is in use.
void given_back() {
    void *p = take(kMiB), *h = take(kMiB, true);
    pool_release(take(2 * kMiB));
    pool_release(take(2 * kMiB, true));
    eahr_release_memory();
    fake::expect(fake::in_use[0] == kMiB && fake::in_use[1] == kMiB, "kept blocks stay, or one in use goes");
    pool_release(p);
    pool_release(h);
    eahr_release_memory();
    fake::expect(fake::in_use[0] == 0 && fake::in_use[1] == 0, "memory is held after the call");
}

}  // namespace

int main() {
    oversized();
    ages();
    given_back();
    std::printf("ok\n");
    return 0;
}
