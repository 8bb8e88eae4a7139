// The dense channel's handles when a HIP call fails, on the CPU (hip_fake.h;
// the kernels are stand-ins that check their buffers): whichever call of an
// entry point fails, no block goes back to the pool while the device may still
// use it, and the state can be used again or closed.
#include <vector>

#include "kernels_fake.h"

#include "dev_pool.h"
#include "eahr.h"
#include "pvs_internal.h"

namespace eahr {
hipError_t pool_alloc(void** p, size_t bytes, bool host) { return fake::alloc(p, bytes, host ? 1 : 0); }
void pool_release(void* p) {
    if (!p) return;
    fake::expect(!fake::busy, "a block was released while the device may use it");
    fake::release(p, fake::blocks.at(static_cast<char*>(p)).second);
}
void pool_free(void* p) { pool_release(p); }
void pool_age(int) {}
}  // namespace eahr

namespace {

constexpr int32_t kB = 3, kM = 5, kDim = 8;

// One program of a dense client; returns how many of its calls failed.  The
// call numbered `fail` of step `step` fails; `calls` is how many the step made.
int client(int32_t generator, int step, long fail, long* calls) {
    int at = 0, failed = 0;
    auto arm = [&]() {
        fake::step = at;
        fake::calls = 0;
        fake::fail_at = at == step ? fail : -1;
    };
    auto done = [&](int rc) {
        if (at == step) *calls = fake::calls;
        ++at;
        fake::fail_at = -1;
        failed += rc != EAHR_OK;
        return rc == EAHR_OK;
    };
    std::vector<float> rows(200 * kDim, 1.0f);
    pvs::g_rows = 100;
    pvs_index* ix = nullptr;
    arm();
    if (!done(pvs_build(rows.data(), 100, kDim, EAHR_PTR_HOST, nullptr, &ix))) return failed;
    std::vector<int64_t> ids(20 * kM);
    std::vector<float> scores(20 * kM);
    std::vector<int32_t> cnt(20), sts(20);
    pvs_state* st = nullptr;
    arm();
    if (done(pvs_open_gen(ix, 0, rows.data(), kB, EAHR_PTR_HOST, generator, &st))) {
        arm();
        done(pvs_next(st, kM, nullptr, ids.data(), scores.data(), cnt.data(), sts.data()));
        arm();   // again: after a failure from the same place, else from the cache
        if (done(pvs_next(st, kM, nullptr, ids.data(), scores.data(), cnt.data(), sts.data())))
            for (int32_t b = 0; b < kB; ++b) {
                fake::expect(cnt[b] == kM, "a later read is short");
                const int64_t first = failed ? 0 : kM;
                for (int32_t i = 0; i < kM; ++i)
                    fake::expect(ids[b * kM + i] == first + i, "a later read is not the next ranks");
            }
        pvs_close(st);
    } else {
        at += 2;
    }
    // a wider batch grows the buffers that the index keeps; after a growth that
    // failed, a batch of the old size must not find them missing
    for (int32_t wide : {20, kB}) {
        st = nullptr;
        arm();
        if (done(pvs_open_gen(ix, 0, rows.data(), wide, EAHR_PTR_HOST, generator, &st))) {
            arm();
            done(pvs_next(st, kM, nullptr, ids.data(), scores.data(), cnt.data(), sts.data()));
            pvs_close(st);
        } else {
            at += 1;
        }
    }
    arm();
    pvs::g_rows = 200;
    done(pvs_insert(ix, rows.data(), 100, EAHR_PTR_HOST, nullptr));
    int64_t epoch = 0;
    arm();
    done(pvs_snapshot(ix, &epoch));
    pvs_free(ix);
    return failed;
}

}  // namespace

int main() {
    long runs = 0;
    for (int32_t generator : {EAHR_GEN_INTERVALS, EAHR_GEN_FULL_SCAN}) {
        long n = 0;
        fake::expect(client(generator, -1, -1, &n) == 0, "the program fails by itself");
        for (int step = 0; step < 10; ++step)
            for (long fail = 0;; ++fail) {
                n = 0;
                const int failed = client(generator, step, fail, &n);
                ++runs;
                if (n <= fail) break;   // the step makes no such call
                fake::expect(failed >= 1, "a failed call was not reported");
            }
    }
    std::printf("ok %ld\n", runs);
    return 0;
}
