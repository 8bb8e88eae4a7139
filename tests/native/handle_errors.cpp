// The dense channel's handles when a HIP call fails, on the CPU (hip_fake.h;
// the kernels are stand-ins that check their buffers): whichever call of an
// entry point fails, no block goes back to the pool while the device may still
// use it, and the state can be used again or closed.
#include <cstring>
#include <vector>

#include "hip_fake.h"

#include "dev_pool.h"
#include "eahr.h"
#include "pvs_internal.h"
#include "pvs_kernels.h"

namespace eahr {
hipError_t pool_alloc(void** p, size_t bytes, bool host) { return fake::alloc(p, bytes, host ? 1 : 0); }
void pool_release(void* p) {
    if (!p) return;
    fake::expect(!fake::busy, "a block was released while the device may use it");
    fake::release(p, fake::blocks.at(static_cast<char*>(p)).second);
}
void pool_age() {}
}  // namespace eahr

namespace pvs {
// every visible row scores 0: keys in id order
static uint64_t key_of(int64_t row) { return (static_cast<uint64_t>(~0x80000000u) << 32) | static_cast<uint64_t>(row); }
static int64_t g_rows = 0;
static void queued(std::initializer_list<std::pair<const void*, size_t>> bufs) {
    for (const auto& b : bufs) fake::expect(fake::inside(b.first, b.second), "a kernel was given a bad buffer");
    fake::busy = true;
}

void launch_quantize(const float* src, int64_t n, int32_t d, int64_t, int64_t row0, bool tiled, int8_t* codes, int32_t dp,
                     float* scale, float*, float*, QueryMeta* qm, float* rows, int32_t df, float, uint32_t*, hipStream_t) {
    queued({{src, n * d * 4}, {codes, (row0 + n) * dp}, {rows, (row0 + n) * df * 4}});
    if (tiled) queued({{scale, (row0 + n) * 4}});
    else {
        queued({{qm, n * sizeof(QueryMeta)}});
        for (int64_t i = 0; i < n; ++i) qm[i] = QueryMeta{1.0f, 1.0f, 0.0f, 1.0f, 0u};
    }
}
void launch_maxabs(const float*, int64_t, uint32_t* f, hipStream_t) { queued({{f, 16}}); }
void launch_set_bits(uint64_t* v, int64_t first, int64_t n, hipStream_t) { queued({{v, (first + n + 63) / 64 * 8}}); }
void launch_clear_ids(uint64_t*, const int64_t* ids, int64_t n, hipStream_t) { queued({{ids, n * 8}}); }
void launch_popcount(const uint64_t* v, int64_t words, unsigned long long* out, hipStream_t) {
    queued({{v, words * 8}, {out, 8}});
    *out = static_cast<unsigned long long>(g_rows);
}
static void scan(int64_t nblocks, const ScanQ* sq, int32_t nq, bool sample, const ScanOut& o) {
    queued({{sq, nq * sizeof(ScanQ)}});
    if (sample) queued({{o.sample, ((nq - 1) * o.sample_ld + (nblocks + o.sample_stride - 1) / o.sample_stride * 64) * 4}});
    else queued({{o.pairs, o.pair_sub * kSub * sizeof(uint4)}, {o.pair_cnt, kSub * kCntStride * 4}, {o.q_evals, kSub * nq * 4}});
}
void launch_scan(const IndexView&, const uint64_t*, int64_t nb, const int8_t*, const ScanQ* sq, int32_t nq, float, bool s,
                 const ScanOut& o, hipStream_t) {
    scan(nb, sq, nq, s, o);
}
void launch_scan_mfma(const IndexView&, const uint64_t*, int64_t nb, const int8_t*, const ScanQ* sq, int32_t nq, float, bool s,
                      const ScanOut& o, void* frag, bool, hipStream_t) {
    queued({{frag, 1}});
    scan(nb, sq, nq, s, o);
}
int mfma_tiles_for(const IndexView&, int32_t) { return 1; }
void launch_round_begin(const ScanQ* h, ScanQ* sq, int32_t nq, int32_t* counts, int64_t n, hipStream_t) {
    queued({{h, nq * sizeof(ScanQ)}, {sq, nq * sizeof(ScanQ)}, {counts, n * 4}});
    std::memcpy(sq, h, nq * sizeof(ScanQ));
}
void launch_regions(const ScanQ* h, ScanQ* sq, int32_t nq, hipStream_t) {
    queued({{h, nq * sizeof(ScanQ)}, {sq, nq * sizeof(ScanQ)}});
    std::memcpy(sq, h, nq * sizeof(ScanQ));
}
void launch_scan_report(const int32_t*, int64_t, int32_t*, const int32_t*, int32_t nq, int32_t* hp, int32_t* he, hipStream_t) {
    queued({{hp, kSub * 4}, {he, nq * 4}});
    std::memset(hp, 0, kSub * 4);
    std::memset(he, 0, nq * 4);
}
void launch_cert_report(int32_t*, const int32_t*, const ScanQ*, int32_t nq, int32_t* hc, int32_t* hf, hipStream_t) {
    queued({{hc, nq * 4}, {hf, nq * 4}});
    for (int32_t i = 0; i < nq; ++i) {
        hc[i] = static_cast<int32_t>(g_rows);
        hf[i] = 0;
    }
}
int64_t rescore_chunks(const int32_t*, int64_t) { return 0; }
void launch_rescore(const IndexView&, const float* q, const ScanQ* sq, int32_t nq, const int32_t*, const uint4* pairs, int64_t sub,
                    const int32_t*, int64_t, float, uint64_t* keys, int32_t*, int32_t*, int32_t*, int32_t, hipStream_t) {
    queued({{q, 1}, {sq, nq * sizeof(ScanQ)}, {pairs, sub * kSub * sizeof(uint4)}, {keys, sub * kSub * 8}});
}
void launch_full_keys(const IndexView&, const uint64_t*, int64_t n, const float*, const int32_t* qidx, int32_t ng, uint64_t* keys,
                      int64_t ld, hipStream_t) {
    queued({{qidx, ng * 4}, {keys, ng * ld * 8}});
    for (int32_t g = 0; g < ng; ++g)
        for (int64_t i = 0; i < n; ++i) keys[g * ld + i] = key_of(i);
}
void launch_select(const uint32_t* s, int64_t n, int64_t ld, float, ScanQ* sq, int32_t nq, int32_t* hits, hipStream_t) {
    queued({{s, ((nq - 1) * ld + n) * 4}, {sq, nq * sizeof(ScanQ)}, {hits, nq * 4}});
    for (int32_t i = 0; i < nq; ++i) hits[i] = static_cast<int32_t>(g_rows);
}
uint64_t* launch_segmented_sort(uint64_t* keys, uint64_t* tmp, const int32_t*, int32_t, const ScanQ* sq, int32_t nq, int64_t max,
                                uint64_t* packed, hipStream_t) {
    queued({{keys, max * 8}, {tmp, max * 8}, {sq, nq * sizeof(ScanQ)}});
    if (!packed) return keys;
    queued({{packed, nq * max * 8}});
    for (int32_t i = 0; i < nq; ++i)
        for (int64_t r = 0; r < max; ++r) packed[i * max + r] = key_of(r);
    return packed;
}
void launch_intervals(const IndexView&, const int8_t*, const ScanQ*, float, const int64_t* r, int64_t n, float* lo, float* hi,
                      hipStream_t) {
    queued({{r, n * 8}, {lo, n * 4}, {hi, n * 4}});
}
void launch_scores(const IndexView&, const float*, int32_t, const int64_t* r, int64_t n, float* out, hipStream_t) {
    queued({{r, n * 8}, {out, n * 4}});
}
}  // namespace pvs

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
