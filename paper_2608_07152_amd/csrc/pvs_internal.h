// Host-side structures of the PVS runtime (index in HBM, per-query state).
#pragma once
#include <hip/hip_runtime.h>

#include <atomic>
#include <cstdint>
#include <mutex>
#include <vector>

#include "eahr.h"
#include "host_parallel.h"
#include "pvs_kernels.h"

// A query's certified ranks as sort keys; grown without zero-filling (the
// keys are copied in right after).
using KeyCache = std::vector<uint64_t, ::eahr::NoInit<uint64_t>>;

namespace pvs {
// Threshold estimation samples one in stride runs of kSampleRun rows, with the
// largest stride that keeps at least this many blocks' worth of rows sampled.
// With stride 1 tau is the target-th largest lower bound, so at least the
// target is certified.  With a larger stride tau is taken from the sampled
// interval midpoints (close to the scores, so the rows certified, s >= tau,
// number about the target scaled by the stride) with this relative margin.
constexpr int64_t kSampleBlocks = 2048;
// The request itself is certified with a margin on its count in the sample,
// because falling short costs another scan.  Its rows may lie side by side, so
// they are taken to fall into the sample by whole runs: three standard
// deviations of a Poisson count of runs and one and a half runs more.  At worst,
// with every run full, about one query in 1,000 exceeds that and is scanned
// again; with four, every call of 256 queries for 1,000 ranks on 1M x 384 took
// 1,005 us instead of 973.
constexpr double kSampleMargin = 1.25;
constexpr double kSampleSigmas = 3.0;
// Smallest candidate pool allocated for a scan, and the largest pool one scan
// round may use (queries beyond it wait for the next round).
constexpr int64_t kMinCap = 4096;
constexpr int64_t kPoolMax = int64_t(1) << 28;
// Candidate regions are sized from the sample: hits / sampled fraction times
// kCapSlack plus kCapPad slots.
constexpr double kCapSlack = 1.5;
constexpr int64_t kCapPad = 2048;
// Ranks a scan aims to certify per query beyond the request: about
// kTargetBudget / (queries in the scan), clamped to [kTargetMin, kTargetMax].
// A single-query scan streams the whole code array, so certifying a deep
// prefix at once is cheap; a large batch shares one scan among many queries
// and pays float32 rescoring per candidate instead.
constexpr int64_t kTargetMin = 64;
constexpr int64_t kTargetMax = 2048;
constexpr int64_t kTargetBudget = 8192;
// Callers extend prefixes geometrically, so a scan also certifies ahead:
// up to kSpecFactor times the depth reached after the request, within
// kSpecBudget ranks per scan shared by its queries.  Rescoring a row costs
// about 1/1000 of streaming the codes once, so over-certifying is cheap next
// to an extra scan.  Measured on 8.8M x 768 (queries/s at batch 256 / 1 / 64):
// factor 8 and 2^20 ranks 1,860 / 90 / 1,085; 8 and 2^22 2,355 / 106 / 1,128;
// 16 and 2^22 2,338 / 117 / 1,241; 2^23 and 2^24 are slower again.
// A scan certifies at least max(kSpecFloor, min(kSpecFloorBudget, rows / 4) / queries)
// ranks per query (within the same budget): a round of a batch scan costs
// about as much as rescoring a few thousand ranks per query, and a round of
// a single-query scan (the whole code array streamed once) as much as
// rescoring about 10^5, so shallow requests are served ahead.  Measured on
// 8.8M x 768, single requests: floor budget 2^16 179 queries/s, 2^17 252,
// 2^18 247 (4096 alone: 182; batches of 64 and 256 unchanged).  Re-measured
// after the other changes (ms per batch-256 / batch-64 step): floor 4096 and
// 2^22 ranks 94.8 / 43.3; 8192 99.9 / 49.0; 2048 100.5 / 46.1; 2^23 94.4 / 44.0.
//
// A caller that asks once pays for ranks nobody reads, one that reads on for
// another scan.  So the first scan of a state certifies the request and about
// min(2^17, rows / 16) ranks ahead over its queries, unless its caller always
// reads on (eahr_topk, merges: pvs_expect_depth) or one of the last two states
// closed on the index read past what such a scan certifies (by ranks, not by
// calls: short pages served by one scan do not count).  Their rescoring is not
// free: it takes as long as the scan for 16 queries on 1M x 384 (72 and 78 us)
// and 100 on 2M x 1,024 (370 and 375), and a fifth of it on 8.8M x 768 (283 and
// 1,210 for one query, 365 and 2,095 for 256).  Certified 16 requests ahead at
// once, 256 queries for 1,000 ranks on 1M x 384 took 3,010 us and 256 for 100 on
// 8.8M x 768 4,950; as now 973 and 2,940.
//
// A state that reads on unpredicted takes a second scan, for all of its queries
// together (they would need one at this request or the next), which certifies
// up to what a deep first scan would have, or kSpecSecond times the depth
// reached: so it pays for one shallow scan more than with a deep first scan.
// Doubling pages, us in the first such state on an index / in later ones / with
// every first scan deep, before these rules: 4M x 768, 64 queries, seven pages
// from 640 12,940 / 12,110 / 13,530, four pages 3,750 / 2,780 / 3,130; 256
// queries, four pages from 100 6,090 / 4,110 / 5,190; 1M x 384, 64 queries, five
// from 640 5,060 / 4,640 / 7,950; 50K x 128, 32 queries, five from 50 626 / 475 /
// 674.  A second scan for each query as it ran out, four times the depth
// reached, took up to 14,260 us where a deep first scan took 5,000 (256 queries,
// five pages from 100 on 4M x 768; now 6,500).
constexpr int64_t kSpecSecond = 2;
constexpr int64_t kSpecFactor = 16;
constexpr int64_t kSpecBudget = int64_t(1) << 22;
constexpr int64_t kSpecFloor = 4096;
constexpr int64_t kSpecFloorBudget = int64_t(1) << 17;
// Scans of at least this many queries use the Int8 MFMA kernel; smaller ones
// the dot4 GEMV kernel, which streams the codes at the HBM rate for up to 8
// queries in one pass.  EAHR_SCAN_PATH=gemv|mfma forces one path (testing).
constexpr int32_t kMfmaMinQueries = 9;
enum class ScanPath { Auto, Gemv, Mfma };
// Candidate pools of at most this many slots are rescored without waiting for
// the scan's counters: the grid is sized for a full pool, and its empty
// workgroups cost less than the wait (about 15 us of an idle GPU).
constexpr int64_t kOneWaitSlots = int64_t(1) << 20;
}  // namespace pvs

// Whether pvs_next(m) on the active queries would be served from certified
// ranks alone (no scan).
bool pvs_covered(const pvs_state* st, int32_t m, const uint8_t* active);
// pvs_next without scores: only the ids of the emitted ranks are written.
int pvs_next_ids(pvs_state* st, int32_t m, const uint8_t* active, int64_t* ids, int32_t* count,
                 int32_t* status);
// Deepen the certified caches of the active queries of a state to `depth`
// ranks each (or to exhaustion) without emitting anything; a later pvs_next
// is then served from the caches.  The host fusion calls it while the CPU
// sparse channel of a round is still running, so the GPU works ahead.
// `added` (optional) receives the number of ranks certified by the call.
int pvs_fill(pvs_state* st, int64_t depth, const uint8_t* active, int64_t* added);
// pvs_fill whose scans certify about `depth` ranks per query and nothing
// further ahead (the caller sized the depth itself).
int pvs_fill_exact(pvs_state* st, int64_t depth, const uint8_t* active, int64_t* added);
// The caller reads no further ranks of query b (its request is settled): the
// query's certified keys that are still in a scan's pinned copy are not
// moved to its cache any more, and pvs_next / pvs_fill skip the query.
void pvs_retire(pvs_state* st, int32_t b);
// The caller will read on, deeper with each call: the state's first scan
// certifies as far ahead as later ones.
void pvs_expect_depth(pvs_state* st);
// Whether query b of a state has failed (a rescored score outside its
// interval), also in work-ahead that pvs_next has not reported yet.
bool pvs_query_failed(const pvs_state* st, int32_t b);
// (query, row) pairs of query b scored in float32 so far.
int64_t pvs_query_evals(const pvs_state* st, int32_t b);
// Batch size a merged ranking was opened for (pvs_merge.cpp).
int32_t eahr_merge_batch(const pvs_merge* mg);
// No rank of the merge has been returned yet (and no query failed).
bool eahr_merge_unread(const pvs_merge* mg);

// Process-wide profile hooks used by the host fusion (pvs_profile_enable).
bool pvs_profile_on();
void pvs_profile_add_host(double dense_ms, double sparse_ms, double fuse_ms);

// Scan buffers of a state (device, plus pinned host mirrors).  A closing
// state hands them to its index, and the next state opened on that index
// adopts them, so repeated requests do not re-allocate them.
struct ScanBuffers {
    int32_t buf_nq = 0;
    int64_t buf_sample = 0;
    pvs::ScanQ* scanq = nullptr;
    int32_t* counts = nullptr;
    uint32_t* sample = nullptr;
    void* qfrag = nullptr;
    int64_t pool_cap = 0;
    uint4* pairs = nullptr;         // candidate pair records of a scan (pool)
    uint64_t* keys = nullptr;
    uint64_t* keys_tmp = nullptr;
    pvs::ScanQ* h_scanq = nullptr;
    int32_t* h_counts = nullptr;
    uint64_t* h_packed = nullptr;
    int64_t h_packed_cap = 0;
    // certified-rank caches of the closed state (emptied, capacity kept)
    std::vector<KeyCache> caches;
};

struct pvs_index {
    struct Snapshot {
        int64_t rows = 0;      // physical rows visible to the epoch (prefix)
        int64_t visible = 0;   // set bits of vis
        uint64_t* vis = nullptr;  // device bitmap, one word per 64-row block
    };
    int device = 0;
    hipStream_t stream = nullptr;
    int32_t d = 0, dp = 0, df = 0, nchunk = 0;
    int64_t rows = 0, cap = 0;
    int8_t* codes = nullptr;   // cap x dp, chunk-major 64-row blocks
    float* scale = nullptr;    // s_v
    float* vnorm = nullptr;    // ||v||_2 rounded up
    float* enorm = nullptr;    // ||e_v||_2 rounded up
    float* frows = nullptr;    // cap x df float32 rows
    uint64_t* live = nullptr;  // live visibility bitmap
    uint32_t* flags = nullptr;
    float* staging = nullptr;  // host->device staging for quantisation
    float nv_max = 0.0f, nev_max = 0.0f;
    float gamma = 0.0f;
    int32_t quant = EAHR_QUANT_PER_VECTOR;   // per-vector scales, or one shared scale
    float global_s = 0.0f;                   // the shared scale once fixed (global mode)
    std::vector<Snapshot> snaps;
    mutable ScanBuffers spare;   // buffers of the last closed state
    mutable bool has_spare = false;
    // whether the states closed last read past what a shallow first scan
    // certifies: 2 after one that did, one less after each that did not
    mutable std::atomic<int> read_on{0};
    // states opened on the index and not closed yet; pvs_free while some are
    // open only marks the index, and the last pvs_close releases it
    mutable std::mutex life_mu;
    mutable int64_t open_states = 0;
    mutable bool release_requested = false;
    ~pvs_index();
};

struct pvs_state {
    struct Query {
        float sq = 0, nq = 0, nqh = 0, neq = 0, wmax = 0;
        bool has_cert = false;          // a rank has been certified
        float s_cert = 0.0f;            // key (s_cert, id_cert) of the last certified rank
        int32_t id_cert = -1;
        // certified ranks in order, as their sort keys (~mono(s32) << 32 | id);
        // ids and scores are decoded only when emitted
        KeyCache cache;
        // the keys of its last scan that follow the cache, still in that
        // scan's pinned copy (h_packed[pend_off .. pend_off + pend_n))
        int64_t pend_off = 0, pend_n = 0;
        bool retired = false;           // no further ranks will be read (pvs_retire)
        int64_t emitted = 0;            // ranks returned by pvs_next
        bool failed = false;
        bool cert_exhausted = false;    // every visible row certified
        int retries = 0;                // consecutive scans that certified too few
        int scans = 0;                  // scans that served a request of it
        int64_t first = 0;              // its first request
        int64_t shallow = 0;            // ranks that a shallow first scan aims at
        int64_t cap_hint = 0;           // candidate capacity needed by the last overflow
        int64_t evals = 0;              // (query, row) pairs rescored in float32
    };
    const pvs_index* ix = nullptr;
    int64_t epoch = 0;
    int32_t B = 0;
    int32_t generator = EAHR_GEN_INTERVALS;   // interval scans, or one exhaustive float32 scan
    int64_t n_rows = 0, n_vis = 0;
    const uint64_t* vis = nullptr;
    int8_t* qcodes = nullptr;   // B x dp row-major
    float* qrows = nullptr;     // B x df
    std::vector<Query> q;
    std::vector<KeyCache> recycled;   // caches adopted from the index
    pvs_counters stats{};
    // per-query scan buffers, sized for buf_nq queries and buf_sample rows
    int32_t buf_nq = 0;
    int64_t buf_sample = 0;
    pvs::ScanQ* scanq = nullptr;
    int32_t* counts = nullptr;
    uint32_t* sample = nullptr;
    void* qfrag = nullptr;             // query codes in MFMA operand order
    // candidate pool (pool_cap slots) split into per-query regions per scan
    int64_t pool_cap = 0;
    uint4* pairs = nullptr;
    uint64_t* keys = nullptr;
    uint64_t* keys_tmp = nullptr;
    pvs::ScanPath path = pvs::ScanPath::Auto;
    bool spec_off = false;             // scans certify no further ahead than asked
    bool reads_on = false;             // the first scan certifies as far ahead as later ones
    bool expected = false;             // its caller said so (pvs_expect_depth)
    bool read_past = false;            // was asked for more than a shallow first scan certifies
    // test knob: first-attempt key regions and pool divided by this, so that
    // the overflow and rescan paths run (results do not change)
    int64_t cap_shrink = 1;
    // test knob (EAHR_TEST_FAIL_QUERY): this query's rescoring judges its
    // scores against a zero-width interval, so its list fails through the
    // normal containment check (App. A.1); -1: off
    int32_t test_fail_qi = -1;
    hipEvent_t ev[7] = {};             // profiling events (created on first use)
    pvs::ScanQ* h_scanq = nullptr;     // pinned host mirrors
    int32_t* h_counts = nullptr;
    uint64_t* h_packed = nullptr;
    int64_t h_packed_cap = 0;
    void release_scan_buffers();
    ~pvs_state();
};
