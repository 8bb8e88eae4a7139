// Internal interface between the PVS host runtime and its gfx950 kernels.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace pvs {

constexpr int kBlockRows = 64;     // rows per code block (one wavefront lane per row)
constexpr int kChunk = 16;         // bytes of one code chunk (one 16-byte load per lane)
constexpr int kMaxDim = 4096;      // 127^2 * 4096 < 2^31 and a_m < 1
constexpr int kSortTile = 2048;    // keys merged per workgroup
constexpr int kMaxGemvQueries = 8; // queries per GEMV scan pass
constexpr int kMaxMfmaQueries = 256;  // queries per MFMA scan pass (8 tiles of 32)
// The sample is drawn in runs of kSampleRun consecutive rows, one from every
// `stride` runs: position i of it is row sample_row(i, stride), and there are
// sample_blocks(...) * 64 positions, those at the end possibly past the last row.
// Which run of each `stride` follows the multiples of the golden section, so
// that rows stored in turn from several sources, whatever their number, are
// sampled alike.  Rows stored by topic or with near-duplicates side by side fall
// into the sample by whole runs, and the margin that covers this (kSampleSigmas)
// grows with the run's length: with whole blocks as runs and a margin for
// independent rows, a request for neighbours stored side by side took up to
// three scans.  Eight rows of one 16-byte chunk are a cache line, so the sample
// is read about as fast as whole blocks are (the pass of 100 queries of
// 2M x 1,024 with its selection 106 us and 105, the pass of 256 of 8.8M x 768
// 136 and 117); runs of four read half lines (128 us instead of 106).
constexpr int kSampleRun = 8;
inline int64_t sample_runs(int64_t nblocks, int64_t stride) {
    return (nblocks * (kBlockRows / kSampleRun) + stride - 1) / stride;
}
inline int64_t sample_blocks(int64_t nblocks, int64_t stride) {
    return (sample_runs(nblocks, stride) + kBlockRows / kSampleRun - 1) / (kBlockRows / kSampleRun);
}
__host__ __device__ inline int64_t sample_row(int64_t i, int64_t stride) {
    const uint64_t s = static_cast<uint64_t>(i) / kSampleRun;
    const uint64_t r = static_cast<uint64_t>(static_cast<uint32_t>(s) * 0x9e3779b9u) * static_cast<uint64_t>(stride) >> 32;
    return static_cast<int64_t>((s * stride + r) * kSampleRun) + i % kSampleRun;
}
// The candidate pool of a scan is split into kSub sub-regions, each with its
// own append counter; the code block (or workgroup) picks the sub-region
// from its index, so concurrent appends hit kSub different counters instead
// of one.  Counters sit kCntStride ints (64 bytes) apart.
constexpr int kSub = 64;
constexpr int kCntStride = 16;
// The counters of certified keys, one per query of a scan, sit kCertStride
// ints (a cache line) apart: concurrent additions to one line are applied one
// after another (next to each other, 256 counters held the rescoring of 9.8M
// pairs at d = 384 to 2.59 ms; apart it takes 1.20 ms).
constexpr int kCertStride = 32;

// Per scanning query, uploaded before every scan.  All fields are read
// uniformly by a wavefront (scalar loads).
struct ScanQ {
    int32_t qi;        // query index inside its state
    float tau;         // interval threshold: candidates have hi >= tau,
                       // certified ranks have s32 >= tau
    float s_cert;      // score of the last certified rank (valid if has_cert)
    int32_t id_cert;   // its row id
    int32_t has_cert;
    int32_t k;         // rank of tau among the sampled values (select pass)
    float sq;          // s_q
    float nq;          // ||q||_2 rounded up
    float nqh;         // ||q_hat||_2 rounded up
    float neq;         // ||e_q||_2 rounded up
    float wmax;        // upper bound of E + G over every row of the index
    int32_t pad;
    int64_t cand_off;  // first slot of this query's key region
    int64_t cand_cap;  // its key region holds kSub * cand_cap keys
};
static_assert(sizeof(ScanQ) == 64, "ScanQ layout");

// Row storage of an index.  Codes of 64 consecutive rows form one block laid
// out chunk-major: byte j of row r lives at
//   ((r / 64) * nchunk + j / 16) * 1024 + (r % 64) * 16 + j % 16,
// so one 16-byte load per lane streams a whole 1 KiB chunk of a block.
struct IndexView {
    const uint4* codes;
    const float* scale;
    const float* vnorm;
    const float* enorm;
    const float* rows;     // float32 rows, stride df floats
    int32_t d, dp, df, nchunk;
};

// An encoded query: s_q, ||q||, ||e_q||, ||q_hat|| (rounded up), and whether it
// holds a non-finite value.
struct QueryMeta {
    float s, norm, enorm, hnorm;
    uint32_t bad;
};

// Launchers (all asynchronous on `stream`).  Kernels that hand a few numbers
// to the host write them into pinned host memory themselves: a copy costs a
// launch of its own and more host time than one.
void launch_quantize(const float* src, int64_t nrows, int32_t d, int64_t src_stride,
                     int64_t row0, bool tiled, int8_t* codes, int32_t dp, float* scale,
                     float* vnorm, float* enorm, QueryMeta* qmeta, float* rows, int32_t df,
                     float fixed_s, uint32_t* flags, hipStream_t stream);
// Largest |x| of count floats into flags[3] (float bits), non-finite into flags[0].
void launch_maxabs(const float* src, int64_t count, uint32_t* flags, hipStream_t stream);

// Outputs of a scan pass.  Sample pass: two 16-bit codes (sample_pack) of every
// (query, position) pair of the sample, row-major [query][sample_ld].
// Main pass: every candidate pair (hi >= tau)
// becomes one record (row, index of the query in the scan, exact integer dot
// product, 0).  A wavefront reserves all records of its block (or of its
// block and half of the query tiles, in the wide MFMA kernel) with one atomic
// on the counter of sub-region s = block or workgroup index % kSub,
// pair_cnt[s * kCntStride], and writes them at pairs[s * pair_sub + j] for
// j < pair_sub; the counter counts every record handed out, also past the
// sub-region's end (the pool overflowed).  A wavefront writes the records of
// one row next to each other, so rescoring reads the row once for all of
// them.
struct ScanOut {
    uint32_t* sample = nullptr;
    int64_t sample_ld = 0;
    int64_t sample_stride = 1;   // sampled runs of rows are multiples of this
    int32_t sample_mid = 0;      // tau is selected from midpoints, not lower bounds
    float norm_sum = 0.0f;       // largest ||v|| plus largest ||e_v|| of the index
    uint4* pairs = nullptr;
    int64_t pair_sub = 0;        // records per sub-region
    int32_t* pair_cnt = nullptr;
    // main pass: q_evals[s * q_ld + i] (zeroed by the caller), summed over
    // the kSub copies s, counts the records of the query with scan index i,
    // i.e. the float32 evaluations its rescoring will make when the pool did
    // not overflow (a block or workgroup adds to copy s = its index % kSub,
    // so the atomics of concurrent blocks spread over kSub addresses)
    int32_t* q_evals = nullptr;
    int32_t q_ld = 0;
    int32_t qbase = 0;           // scan index of the pass's first query
};

void launch_scan(const IndexView& ix, const uint64_t* vis, int64_t nblocks, const int8_t* qcodes,
                 const ScanQ* sq, int32_t nq, float gamma, bool sample, const ScanOut& o,
                 hipStream_t stream);

// Int8 MFMA variant (same outputs as launch_scan).  `frag` is device scratch
// of (dp / 32) * 8 KiB for the query codes in MFMA operand order; have_frag: it
// still holds those of the same nq <= kMaxMfmaQueries queries.
void launch_scan_mfma(const IndexView& ix, const uint64_t* vis, int64_t nblocks,
                      const int8_t* qcodes, const ScanQ* sq, int32_t nq, float gamma, bool sample,
                      const ScanOut& o, void* frag, bool have_frag, hipStream_t stream);
int mfma_tiles_for(const IndexView& ix, int32_t nq);

// tau = the k-th largest selection value of each query's sample, rounded down
// to a sample code's value (-inf when fewer than k pairs are eligible), into sq; the
// number of sampled pairs of query b with hi >= tau to h_hits[b] (pinned).
void launch_select(const uint32_t* sample, int64_t n, int64_t ld, float norm_sum, ScanQ* sq, int32_t nq,
                   int32_t* h_hits, hipStream_t stream);

// Start of a scan round: sq = the host's h_sq, and ncounts (a multiple of 4)
// counters cleared.
void launch_round_begin(const ScanQ* h_sq, ScanQ* sq, int32_t nq, int32_t* counts, int64_t ncounts,
                        hipStream_t stream);
// The key regions (cand_off, cand_cap) of the host's h_sq into sq.
void launch_regions(const ScanQ* h_sq, ScanQ* sq, int32_t nq, hipStream_t stream);
// After a main pass: the chunk bases of rescoring (cbase, kSub + 1 ints), and
// to the host each sub-region's counter (h_pcnt) and each query's records
// (h_evals, the sum of the kSub copies).
void launch_scan_report(const int32_t* pair_cnt, int64_t pair_sub, int32_t* cbase, const int32_t* q_evals,
                        int32_t nq, int32_t* h_pcnt, int32_t* h_evals, hipStream_t stream);
// After rescoring: to the host each query's count of certified keys and its
// failure; the device's count is cut to the query's key region, and where the
// query's keys start when they are packed goes into the count's line.
void launch_cert_report(int32_t* cert_cnt, const int32_t* fail, const ScanQ* sq, int32_t nq,
                        int32_t* h_cert, int32_t* h_fail, hipStream_t stream);

// Rescoring reads the kept records of every sub-region of the pool (at most
// pair_sub each, in chunks of kRescoreChunk; chunks = rescore_chunks of the
// host copy of the counters), computes each pair's float32 score and checks
// it against its interval, and appends the keys of the certified pairs of
// query b at keys[cand_off + j], j < min(cert_cnt[b * kCertStride], kSub * cand_cap)
// (cert_cnt zeroed by the caller counts them all; order of appends
// unspecified).  cbase: the chunk bases of launch_scan_report; chunks: their
// number, or any larger one (workgroups past it end at once); the kSub counters
// row_reads[s * kCntStride] (zeroed by the caller) sum to the number of row
// loads, one per run of records of one row inside a wavefront's share.
// fail_qi (tests only, -1 otherwise): the state query whose rescored scores
// are judged against a zero-width interval, so that its list fails.  nq: the
// scan's queries (records refer to sq[0, nq)); when their float32 query rows
// fit in LDS, workgroups copy them there once instead of reloading them.
constexpr int kRescoreChunk = 256;
int64_t rescore_chunks(const int32_t* pair_cnt, int64_t pair_sub);
void launch_rescore(const IndexView& ix, const float* qrows, const ScanQ* sq, int32_t nq,
                    const int32_t* pair_cnt, const uint4* pairs, int64_t pair_sub,
                    const int32_t* cbase, int64_t chunks, float gamma, uint64_t* keys,
                    int32_t* cert_cnt, int32_t* fail, int32_t* row_reads, int32_t fail_qi,
                    hipStream_t stream);

// Exhaustive float32 keys of every row of [0, n_rows) for ng queries (state
// query indices qidx, device), query g's keys at keys + g * ld; invisible rows
// get ~0.
void launch_full_keys(const IndexView& ix, const uint64_t* vis, int64_t n_rows, const float* qrows,
                      const int32_t* qidx, int32_t ng, uint64_t* keys, int64_t ld,
                      hipStream_t stream);
// Sorts every query's candidate keys (cnt[b * cnt_ld] keys from cand_off) ascending;
// returns the buffer holding the result: keys or tmp (each query's keys from
// its cand_off), or, when given, packed, with the queries' keys one after
// another (cnt as launch_cert_report leaves it, cnt_ld = kCertStride).  packed
// may be pinned host memory: only the last kernel writes it, and nothing reads
// it.
uint64_t* launch_segmented_sort(uint64_t* keys, uint64_t* tmp, const int32_t* cnt, int32_t cnt_ld,
                                const ScanQ* sq, int32_t nq, int64_t max_cnt, uint64_t* packed,
                                hipStream_t stream);

void launch_intervals(const IndexView& ix, const int8_t* qcodes, const ScanQ* sq, float gamma,
                      const int64_t* rows, int64_t n, float* lo, float* hi, hipStream_t stream);

void launch_scores(const IndexView& ix, const float* qrows, int32_t qi, const int64_t* rows,
                   int64_t n, float* out, hipStream_t stream);

void launch_set_bits(uint64_t* vis, int64_t first, int64_t n, hipStream_t stream);
void launch_clear_ids(uint64_t* vis, const int64_t* ids, int64_t n, hipStream_t stream);
void launch_popcount(const uint64_t* vis, int64_t nwords, unsigned long long* out,
                     hipStream_t stream);

}  // namespace pvs
