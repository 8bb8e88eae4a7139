// Stand-ins for the dense channel's kernels on the CPU: they check that their
// buffers are live and large enough, and rank the rows of an index by id.  A
// scan certifies every row, or with g_by_k the next k rows of each query (with
// g_spread a percentage fewer for each query after the first).
#pragma once
#include <cstring>
#include <initializer_list>
#include <utility>

#include "hip_fake.h"

#include "pvs_kernels.h"

namespace pvs {
// every visible row scores 0: keys in id order
static uint64_t key_of(int64_t row) { return (static_cast<uint64_t>(~0x80000000u) << 32) | static_cast<uint64_t>(row); }
static int64_t g_rows = 0;
static bool g_by_k = false;
static int64_t g_spread = 0;
static int64_t first_of(const ScanQ& q) { return g_by_k && q.has_cert ? q.id_cert + 1 : 0; }
static int64_t count_of(const ScanQ& q) {
    const int64_t left = g_rows - first_of(q);
    const int64_t k = q.k - q.k * q.qi * g_spread / 100;
    return g_by_k && k < left ? k : left;
}
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
    if (sample) queued({{o.sample, ((nq - 1) * o.sample_ld + sample_blocks(nblocks, o.sample_stride) * 64) * 4}});
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
void launch_cert_report(int32_t*, const int32_t*, const ScanQ* sq, int32_t nq, int32_t* hc, int32_t* hf, hipStream_t) {
    queued({{sq, nq * sizeof(ScanQ)}, {hc, nq * 4}, {hf, nq * 4}});
    for (int32_t i = 0; i < nq; ++i) {
        hc[i] = static_cast<int32_t>(count_of(sq[i]));
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
    int64_t n = 0;
    for (int32_t i = 0; i < nq; ++i) n += count_of(sq[i]);
    queued({{packed, n * 8}});
    for (int32_t i = 0; i < nq; ++i)
        for (int64_t r = 0; r < count_of(sq[i]); ++r) *packed++ = key_of(first_of(sq[i]) + r);
    return packed - n;
}
void launch_intervals(const IndexView&, const int8_t*, const ScanQ*, float, const int64_t* r, int64_t n, float* lo, float* hi,
                      hipStream_t) {
    queued({{r, n * 8}, {lo, n * 4}, {hi, n * 4}});
}
void launch_scores(const IndexView&, const float*, int32_t, const int64_t* r, int64_t n, float* out, hipStream_t) {
    queued({{r, n * 8}, {out, n * 4}});
}
}  // namespace pvs
