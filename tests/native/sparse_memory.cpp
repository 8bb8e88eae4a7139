// The sparse channel's device copies when the GPU's memory, or pinned memory,
// is taken by the dense channel's kept blocks, on the CPU (hip_fake.h).
#include <vector>

#include "hip_fake.h"

#include "dev_pool.h"
#include "eahr.h"
#include "pbm_kernels.h"

namespace pbmg {
void launch_bounds(const IndexView& ix, const QueryView& q, float* H, int32_t* post, int64_t*, hipStream_t) {
    for (int64_t i = 0; i < q.B * ix.n_ranges; ++i) {
        H[i] = 0.0f;
        post[i] = 0;
    }
}
int launch_expand(const IndexView&, const QueryView&, const Task*, int32_t, const int64_t*, const int64_t*, int32_t*, uint64_t*,
                  hipStream_t) {
    return 0;
}
}  // namespace pbmg

int main() {
    constexpr int64_t kDocs = 100000;
    constexpr size_t kMiB = size_t(1) << 20;
    const int64_t term_ptr[] = {0, kDocs};
    std::vector<int32_t> docs(kDocs);
    for (int64_t i = 0; i < kDocs; ++i) docs[i] = static_cast<int32_t>(i);
    const std::vector<float> imp(kDocs, 1.0f);
    pbm_index* ix = nullptr;
    fake::expect(pbm_build(term_ptr, 1, docs.data(), imp.data(), kDocs, 1024, &ix) == EAHR_OK, "build");
    for (size_t& b : fake::budget) b = 4 * kMiB;
    for (bool host : {false, true})
        for (int i = 0; i < 2; ++i) {   // all of it is kept by the pool
            void *p = nullptr, *q = nullptr;
            fake::expect(eahr::pool_alloc(&p, 2 * kMiB, host) == hipSuccess, "first block");
            fake::expect(eahr::pool_alloc(&q, 2 * kMiB, host) == hipSuccess, "second block");
            eahr::pool_release(p);
            eahr::pool_release(q);
        }
    fake::expect(pbm_upload(ix) == EAHR_OK, "the upload fails beside memory that is only kept");
    const int32_t term = 0;
    const float w = 1.0f;
    const eahr_sparse_query q{&term, &w, 1};
    pbm_gpu_state* st = nullptr;
    fake::expect(pbm_gpu_open(ix, &q, 1, &st) == EAHR_OK, "the state's buffers fail beside memory that is only kept");
    pbm_gpu_close(st);
    pbm_free(ix);
    std::printf("ok\n");
    return 0;
}
