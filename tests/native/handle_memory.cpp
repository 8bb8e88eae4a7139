// Memory that one long-lived index of a program holds on to, on the CPU
// (hip_fake.h, the library's own pool).
#include <vector>

#include "kernels_fake.h"

#include "dev_pool.h"
#include "eahr.h"

namespace {

constexpr int32_t kDim = 64;
constexpr size_t kMiB = size_t(1) << 20;

size_t held() { return fake::in_use[0] + fake::in_use[1]; }

pvs_index* build(const std::vector<float>& rows, int64_t n) {
    pvs_index* ix = nullptr;
    pvs::g_rows = n;
    fake::expect(pvs_build(rows.data(), n, kDim, EAHR_PTR_HOST, nullptr, &ix) == EAHR_OK, "build");
    return ix;
}

void read(pvs_index* ix, const std::vector<float>& rows, int32_t B) {
    pvs_state* st = nullptr;
    std::vector<int64_t> ids(B);
    std::vector<float> sc(B);
    std::vector<int32_t> cnt(B), sts(B);
    fake::expect(pvs_open(ix, 0, rows.data(), B, EAHR_PTR_HOST, &st) == EAHR_OK, "open");
    fake::expect(pvs_next(st, 1, nullptr, ids.data(), sc.data(), cnt.data(), sts.data()) == EAHR_OK, "next");
    pvs_close(st);
}

// An index that grows by inserts keeps its arrays and nothing of the smaller ones.
void growth() {
    const int64_t step = 20000;
    const std::vector<float> rows(step * kDim, 1.0f);
    pvs_index* ix = build(rows, step);
    int64_t n = step;
    for (int i = 0; i < 8; ++i) {
        fake::expect(pvs_insert(ix, rows.data(), step, EAHR_PTR_HOST, nullptr) == EAHR_OK, "insert");
        n += step;
    }
    // codes, rows and three floats of at most 1.5 n rows, and the staging buffer
    const size_t most = static_cast<size_t>(n + n / 2) * (kDim + 4 * kDim + 13) + 65536 * kDim * 4;
    fake::expect(held() <= most + 8 * kMiB, "outgrown arrays are still held");
    pvs_free(ix);
}

// Reads that no longer need a large batch's buffers give them back in the end.
void closes() {
    const std::vector<float> rows(8192 * kDim, 1.0f);
    pvs_index* ix = build(rows, 100);
    read(ix, rows, 8);
    const size_t before = held();
    for (int wide = 0; wide < 2; ++wide) read(ix, rows, 8192);   // its query rows, codes and pinned copies
    const size_t spare = held();
    for (int i = 0; i < 200; ++i) read(ix, rows, 8);
    // what the index keeps for its next state stays, the closed states' own memory goes
    fake::expect(held() <= spare - 8192 * kDim * 4, "memory of closed states is held for ever");
    fake::expect(held() >= before, "a block in use was freed");
    pvs_free(ix);
}

}  // namespace

int main() {
    growth();
    closes();
    std::printf("ok\n");
    return 0;
}
