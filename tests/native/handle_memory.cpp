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

}  // namespace

int main() {
    growth();
    std::printf("ok\n");
    return 0;
}
