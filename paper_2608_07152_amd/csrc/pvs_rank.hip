// Candidate rescoring, ordering and packing of the PVS dense channel.
//
// Every candidate pair gets its authoritative float32 score (the fixed
// order of group_dot) and is checked against its interval (App. A.1: a score
// outside it fails the request), recomputed from the integer dot product the
// scan recorded with the scan's own arithmetic, so identical to it.  A scan
// with threshold tau certifies exactly the candidates with s32 >= tau whose
// key follows the last certified key; their keys (~mono(s32) << 32 | row) are
// appended to the query's key region, so ascending keys are (score
// descending, id ascending).  Keys are unique inside a query; the segmented
// sort orders each query's certified keys.
#include <algorithm>
#include <atomic>

#include "pvs_device.h"

namespace pvs {

// ------------------------------------------------------------ bookkeeping
// Bound by launch latency, all of them: each stands for the copies and clears
// of its place in a round (13 of the 20 launches of a one-query call were
// copies and clears; on 20K x 128 the call took 181 us, now 107).
__global__ __launch_bounds__(256) void k_round_begin(const uint4* __restrict__ h_sq, uint4* __restrict__ sq,
                                                     int32_t n_sq, uint4* __restrict__ counts, int64_t n_counts) {
    const int64_t i0 = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x;
    const int64_t step = static_cast<int64_t>(gridDim.x) * 256;
    for (int64_t i = i0; i < n_sq; i += step) sq[i] = h_sq[i];
    for (int64_t i = i0; i < n_counts; i += step) counts[i] = make_uint4(0u, 0u, 0u, 0u);
}

void launch_round_begin(const ScanQ* h_sq, ScanQ* sq, int32_t nq, int32_t* counts, int64_t ncounts,
                        hipStream_t stream) {
    const int32_t n_sq = nq * static_cast<int32_t>(sizeof(ScanQ) / sizeof(uint4));
    const int64_t blocks = std::min<int64_t>(64, (std::max<int64_t>(n_sq, ncounts / 4) + 255) / 256);
    hipLaunchKernelGGL(k_round_begin, dim3(static_cast<uint32_t>(std::max<int64_t>(1, blocks))), dim3(256), 0, stream,
                       reinterpret_cast<const uint4*>(h_sq), reinterpret_cast<uint4*>(sq), n_sq,
                       reinterpret_cast<uint4*>(counts), ncounts / 4);
}

__global__ __launch_bounds__(256) void k_regions(const ScanQ* __restrict__ h_sq, ScanQ* __restrict__ sq, int32_t nq) {
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i >= nq) return;
    sq[i].cand_off = h_sq[i].cand_off;
    sq[i].cand_cap = h_sq[i].cand_cap;
}

void launch_regions(const ScanQ* h_sq, ScanQ* sq, int32_t nq, hipStream_t stream) {
    if (nq > 0) hipLaunchKernelGGL(k_regions, dim3((nq + 255) / 256), dim3(256), 0, stream, h_sq, sq, nq);
}

// The records of a scan round are cut into chunks of kRescoreChunk per pool
// sub-region; cbase[s] is the first chunk of sub-region s (exclusive prefix).
__global__ __launch_bounds__(256) void k_scan_report(const int32_t* __restrict__ pair_cnt, int64_t pair_sub,
                                                     int32_t* __restrict__ cbase, const int32_t* __restrict__ q_evals,
                                                     int32_t nq, int32_t* __restrict__ h_pcnt,
                                                     int32_t* __restrict__ h_evals) {
    static_assert(kSub == 64, "one sub-region per lane");
    if (blockIdx.x == 0 && threadIdx.x < kSub) {
        const int s = threadIdx.x;
        const int32_t c = pair_cnt[s * kCntStride];
        h_pcnt[s] = c;
        const int64_t n = c < pair_sub ? c : pair_sub;
        const int32_t own = static_cast<int32_t>((n + kRescoreChunk - 1) / kRescoreChunk);
        int32_t x = own;
        for (int off = 1; off < 64; off <<= 1) {
            const int32_t y = __shfl_up(x, off, 64);
            if (s >= off) x += y;
        }
        cbase[s] = x - own;
        if (s == kSub - 1) cbase[kSub] = x;
    }
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i < nq) {
        int32_t e = 0;
        for (int c = 0; c < kSub; ++c) e += q_evals[c * nq + i];
        h_evals[i] = e;
    }
}

void launch_scan_report(const int32_t* pair_cnt, int64_t pair_sub, int32_t* cbase, const int32_t* q_evals,
                        int32_t nq, int32_t* h_pcnt, int32_t* h_evals, hipStream_t stream) {
    hipLaunchKernelGGL(k_scan_report, dim3(std::max(1, (nq + 255) / 256)), dim3(256), 0, stream, pair_cnt, pair_sub,
                       cbase, q_evals, nq, h_pcnt, h_evals);
}

// Where the keys of query i start when the queries' keys lie one after another.
__device__ __forceinline__ int64_t* packed_offset(int32_t* cnt, int i) {
    return reinterpret_cast<int64_t*>(cnt + static_cast<int64_t>(i) * kCertStride + 2);
}
__device__ __forceinline__ int64_t packed_offset(const int32_t* cnt, int i) {
    return *reinterpret_cast<const int64_t*>(cnt + static_cast<int64_t>(i) * kCertStride + 2);
}

// One thread per query; a workgroup adds up the counts of the queries before
// its own for the offsets, once: each workgroup of the sort did it for itself
// before, which grows with the square of the batch.
__global__ __launch_bounds__(256) void k_cert_report(int32_t* __restrict__ cert_cnt, const int32_t* __restrict__ fail,
                                                     const ScanQ* __restrict__ sq, int32_t nq,
                                                     int32_t* __restrict__ h_cert, int32_t* __restrict__ h_fail) {
    __shared__ int64_t s_before[4], s_own[4];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int first = blockIdx.x * 256, i = first + tid;
    // (another workgroup may have cut a count already: the same value again)
    auto kept = [&](int j, int32_t c) { return min(static_cast<int64_t>(c), kSub * sq[j].cand_cap); };
    int64_t before = 0;
    for (int j = tid; j < first; j += 256) before += kept(j, cert_cnt[j * kCertStride]);
    for (int off = 32; off > 0; off >>= 1) before += __shfl_xor(before, off, 64);
    const int32_t c = i < nq ? cert_cnt[i * kCertStride] : 0;
    const int64_t own = i < nq ? kept(i, c) : 0;
    int64_t upto = own;
    for (int off = 1; off < 64; off <<= 1) {
        const int64_t y = __shfl_up(upto, off, 64);
        if (lane >= off) upto += y;
    }
    if (lane == 63) {
        s_before[wave] = before;
        s_own[wave] = upto;
    }
    __syncthreads();
    if (i >= nq) return;
    int64_t at = upto - own;
    for (int w = 0; w < 4; ++w) at += s_before[w] + (w < wave ? s_own[w] : 0);
    h_cert[i] = c;
    h_fail[i] = fail[i];
    if (c > own) cert_cnt[i * kCertStride] = static_cast<int32_t>(own);
    *packed_offset(cert_cnt, i) = at;
}

void launch_cert_report(int32_t* cert_cnt, const int32_t* fail, const ScanQ* sq, int32_t nq,
                        int32_t* h_cert, int32_t* h_fail, hipStream_t stream) {
    if (nq > 0)
        hipLaunchKernelGGL(k_cert_report, dim3((nq + 255) / 256), dim3(256), 0, stream, cert_cnt, fail, sq, nq, h_cert,
                           h_fail);
}

// --------------------------------------------------------------- rescoring
// The records of quarter `wave` of chunk x (one wavefront, 64 records).
// Lane j first prepares record j (its interval from the recorded dot with
// the scan's arithmetic, its query's tau and last certified key); each
// 16-lane group g then scores records 16 g .. 16 g + 15 one after another
// (the group's lanes hold the record's row and query row in the fixed order
// of the authoritative score, so four records are scored at once), and the
// record's own lane judges its score.  Records of one row are adjacent, so a
// group loads the row once for them; likewise the query row, which comes
// from LDS (slot = the record's query in the scan) when LDSQ.  At the end
// the keys of each query are appended to its region with one atomic.
// J: chunks per lane (0: rows scored in segments); FULL: df / 4 == 16 J.
template <int J, bool FULL, bool LDSQ>
__device__ __forceinline__ void rescore_quarter(
    int x, int wave, const float4* __restrict__ rows, int32_t df4, const float4* __restrict__ qsrc,
    const ScanQ* __restrict__ sq, const int32_t* __restrict__ cbase,
    const int32_t* __restrict__ pair_cnt, const uint4* __restrict__ pairs, int64_t pair_sub,
    const float* __restrict__ scale, const float* __restrict__ vnorm,
    const float* __restrict__ enorm, float gamma, uint64_t* __restrict__ keys,
    int32_t* __restrict__ cert_cnt, int32_t* __restrict__ fail, int32_t* __restrict__ row_reads,
    int32_t fail_qi) {
    constexpr int PER_WAVE = kRescoreChunk / 4;
    static_assert(PER_WAVE == 64, "one record per lane");
    const int lane = threadIdx.x & 63;
    // the sub-region of this chunk: the last s with cbase[s] <= chunk
    int slo = 0, shi = kSub;
    while (shi - slo > 1) {
        const int mid = (slo + shi) >> 1;
        if (cbase[mid] <= x) slo = mid;
        else shi = mid;
    }
    const int s = slo;
    const int64_t cnt = pair_cnt[s * kCntStride];
    const int64_t n_s = cnt < pair_sub ? cnt : pair_sub;
    const int64_t i0 = static_cast<int64_t>(x - cbase[s]) * kRescoreChunk + wave * PER_WAVE;
    const int n = static_cast<int>(n_s - i0 < PER_WAVE ? n_s - i0 : PER_WAVE);
    if (n <= 0) return;
    // this lane's record
    const bool mine = lane < n;
    const uint4 rec = mine ? pairs[s * pair_sub + i0 + lane] : make_uint4(0u, 0u, 0u, 0u);
    const int32_t my_row = static_cast<int32_t>(rec.x);
    const int32_t my_b = static_cast<int32_t>(rec.y);
    const ScanQ& MQ = sq[my_b];
    const int32_t my_qi = MQ.qi;
    float my_lo, my_hi;
    pair_interval(MQ, scale[my_row], vnorm[my_row], enorm[my_row], static_cast<int32_t>(rec.z), gamma,
                  my_lo, my_hi);
    if (my_qi == fail_qi) {
        // failure injection (tests only): the judged interval of this query
        // shrinks to the ulps around c, so its scores fall outside it
        const float c = (MQ.sq * scale[my_row]) * static_cast<float>(static_cast<int32_t>(rec.z));
        my_lo = next_down(c);
        my_hi = next_up(c);
    }
    const float my_tau = MQ.tau, my_scert = MQ.s_cert;
    const int32_t my_idcert = MQ.id_cert;
    const bool my_hascert = MQ.has_cert != 0;
    uint64_t mykey = 0;
    bool cert = false, bad = false;
    const int g = lane >> 4, j = lane & 15;
    float4 v[J > 0 ? J : 1], q[J > 0 ? J : 1];
    int32_t prow = -1, pqi = -1;
    int reads = 0;   // row loads of this lane's group
    static_for(
        [&](auto I_) {
            constexpr int i = decltype(I_)::value;
            // the group's record i, held by lane 16 g + i
            const int32_t row = bcast16<i>(my_row);
            const int32_t qi = bcast16<i>(LDSQ ? my_b : my_qi);   // LDSQ: the LDS slot
            if (16 * g + i < n) {   // the same in every lane of the group
                float sc;
                if constexpr (J > 0) {
                    if (row != prow) {
                        load_chunks<J, FULL>(rows + static_cast<int64_t>(row) * df4, j, df4, v);
                        prow = row;
                        ++reads;
                    }
                    if (qi != pqi) {   // from LDS when LDSQ
                        load_chunks<J, FULL>(qsrc + static_cast<int64_t>(qi) * df4, j, df4, q);
                        pqi = qi;
                    }
                    sc = group_dot<J, FULL>(v, q, j, df4);
                } else {
                    sc = group_score_seg(rows + static_cast<int64_t>(row) * df4,
                                         qsrc + static_cast<int64_t>(qi) * df4, j, df4);
                    ++reads;
                }
                if (j == i) {
                    bad = !(my_lo <= sc && sc <= my_hi);
                    const bool dropped = my_hascert && (sc > my_scert || (sc == my_scert && row <= my_idcert));
                    if (!dropped && sc >= my_tau) {
                        mykey = (static_cast<uint64_t>(~mono32(sc)) << 32) | static_cast<uint32_t>(row);
                        cert = true;
                    }
                }
            }
        },
        std::make_integer_sequence<int, 16>{});
    reads = __builtin_amdgcn_readlane(reads, 0) + __builtin_amdgcn_readlane(reads, 16) +
            __builtin_amdgcn_readlane(reads, 32) + __builtin_amdgcn_readlane(reads, 48);
    // one of kSub counters (one address for every wavefront would serialise)
    if (lane == 0) atomicAdd(&row_reads[(blockIdx.x & (kSub - 1)) * kCntStride], reads);
    if (bad) fail[my_b] = 1;
    // group the certified lanes by query (one pass per distinct query, ALU
    // only), then the first lane of each group appends the group with one
    // atomic, all groups in the same instruction
    const int myb = cert ? my_b : -1;
    uint64_t todo = __ballot(cert);
    if (!todo) return;
    int leader = 0, rank = 0, size = 0;
    while (todo) {
        const int l0 = __ffsll(static_cast<unsigned long long>(todo)) - 1;
        const int b0 = __builtin_amdgcn_readlane(myb, l0);
        const uint64_t grp = __ballot(myb == b0);
        if (myb == b0) {
            leader = l0;
            rank = __popcll(grp & ((1ull << lane) - 1ull));
            size = __popcll(grp);
        }
        todo &= ~grp;
    }
    int base = 0;
    if (cert && lane == leader) base = atomicAdd(&cert_cnt[myb * kCertStride], size);
    base = __shfl(base, leader, 64);
    if (!cert) return;
    const int64_t pos = static_cast<int64_t>(base) + rank;
    if (pos < kSub * MQ.cand_cap) keys[MQ.cand_off + pos] = mykey;
}

// One wavefront per quarter of a chunk of kRescoreChunk records.  LDSQ: a
// workgroup of sixteen wavefronts takes four chunks and first copies the
// scan's nq float32 query rows to LDS, and the groups read their query rows
// from there instead of reloading them from L2 per record (the loads that
// bound the kernel when records of one row belong to different queries).
// Workgroups that each loop over many chunks after one copy measured slower
// (on a three-query scan, 9.3 against 3.8 ms).
template <int J, bool FULL, bool LDSQ>
__global__ __launch_bounds__(LDSQ ? 1024 : 256) void k_rescore(
    const float4* __restrict__ rows, int32_t df4, const float4* __restrict__ qrows,
    const ScanQ* __restrict__ sq, int32_t nq, const int32_t* __restrict__ cbase,
    const int32_t* __restrict__ pair_cnt, const uint4* __restrict__ pairs, int64_t pair_sub,
    const float* __restrict__ scale, const float* __restrict__ vnorm,
    const float* __restrict__ enorm, float gamma, uint64_t* __restrict__ keys,
    int32_t* __restrict__ cert_cnt, int32_t* __restrict__ fail, int32_t* __restrict__ row_reads,
    int32_t fail_qi) {
    if constexpr (LDSQ) {
        extern __shared__ float4 s_q[];   // query row b at s_q[b * df4]
        if (static_cast<int>(blockIdx.x) * 4 >= cbase[kSub]) return;   // the same in every thread
        for (int k = threadIdx.x; k < nq * df4; k += blockDim.x) {
            const int b = k / df4;
            s_q[k] = qrows[static_cast<int64_t>(sq[b].qi) * df4 + (k - b * df4)];
        }
        __syncthreads();
        const int x = static_cast<int>(blockIdx.x) * 4 + static_cast<int>(threadIdx.x >> 8);
        if (x < cbase[kSub])
            rescore_quarter<J, FULL, true>(x, (threadIdx.x >> 6) & 3, rows, df4, s_q, sq, cbase, pair_cnt, pairs,
                                           pair_sub, scale, vnorm, enorm, gamma, keys, cert_cnt, fail, row_reads,
                                           fail_qi);
    } else {
        if (static_cast<int>(blockIdx.x) >= cbase[kSub]) return;
        rescore_quarter<J, FULL, false>(blockIdx.x, threadIdx.x >> 6, rows, df4, qrows, sq, cbase, pair_cnt, pairs,
                                        pair_sub, scale, vnorm, enorm, gamma, keys, cert_cnt, fail, row_reads,
                                        fail_qi);
    }
}

// LDS of the query-row variant: at most a gfx950 CU's 160 KiB.
constexpr size_t kRescoreLdsMax = 160 * 1024;

template <int J, bool FULL>
static void rescore_j(const IndexView& ix, const float* qrows, const ScanQ* sq, int32_t nq,
                      const int32_t* cbase, int64_t chunks, const int32_t* pair_cnt,
                      const uint4* pairs, int64_t pair_sub, float gamma, uint64_t* keys,
                      int32_t* cert_cnt, int32_t* fail, int32_t* row_reads, int32_t fail_qi,
                      hipStream_t stream) {
    const int32_t df4 = ix.df / 4;
    const size_t lds = static_cast<size_t>(nq) * df4 * sizeof(float4);
    // one query: its row stays in the groups' registers anyway
    if constexpr (J > 0) {
        static std::atomic<int> ready{0};   // 1: LDS attribute set, -1: refused
        if (nq > 1 && lds <= kRescoreLdsMax && ready.load() == 0) {
            const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(&k_rescore<J, FULL, true>),
                                                     hipFuncAttributeMaxDynamicSharedMemorySize,
                                                     static_cast<int>(kRescoreLdsMax));
            ready.store(e == hipSuccess ? 1 : -1);
            if (e != hipSuccess) (void)hipGetLastError();
        }
        if (nq > 1 && lds <= kRescoreLdsMax && ready.load() > 0) {
            const uint32_t groups = static_cast<uint32_t>((chunks + 3) / 4);
            hipLaunchKernelGGL((k_rescore<J, FULL, true>), dim3(groups), dim3(1024), lds, stream,
                               reinterpret_cast<const float4*>(ix.rows), df4,
                               reinterpret_cast<const float4*>(qrows), sq, nq, cbase, pair_cnt, pairs, pair_sub,
                               ix.scale, ix.vnorm, ix.enorm, gamma, keys, cert_cnt, fail, row_reads, fail_qi);
            return;
        }
    }
    hipLaunchKernelGGL((k_rescore<J, FULL, false>), dim3(static_cast<uint32_t>(chunks)), dim3(256), 0, stream,
                       reinterpret_cast<const float4*>(ix.rows), df4, reinterpret_cast<const float4*>(qrows), sq,
                       nq, cbase, pair_cnt, pairs, pair_sub, ix.scale, ix.vnorm, ix.enorm, gamma, keys, cert_cnt,
                       fail, row_reads, fail_qi);
}

int64_t rescore_chunks(const int32_t* pair_cnt, int64_t pair_sub) {
    int64_t c = 0;
    for (int s = 0; s < kSub; ++s) {
        const int64_t n = std::min<int64_t>(pair_cnt[s], pair_sub);
        c += (n + kRescoreChunk - 1) / kRescoreChunk;
    }
    return c;
}

void launch_rescore(const IndexView& ix, const float* qrows, const ScanQ* sq, int32_t nq,
                    const int32_t* pair_cnt, const uint4* pairs, int64_t pair_sub,
                    const int32_t* cbase, int64_t chunks, float gamma, uint64_t* keys,
                    int32_t* cert_cnt, int32_t* fail, int32_t* row_reads, int32_t fail_qi,
                    hipStream_t stream) {
    if (chunks <= 0) return;
    const int J = group_chunks(ix.df);
    const bool full = J > 0 && ix.df / 4 == 16 * J;
#define PVS_RS(N)                                                                                      \
    case N:                                                                                            \
        if (full)                                                                                      \
            rescore_j<N, true>(ix, qrows, sq, nq, cbase, chunks, pair_cnt, pairs, pair_sub, gamma, keys, \
                               cert_cnt, fail, row_reads, fail_qi, stream);                            \
        else                                                                                           \
            rescore_j<N, false>(ix, qrows, sq, nq, cbase, chunks, pair_cnt, pairs, pair_sub, gamma,     \
                                keys, cert_cnt, fail, row_reads, fail_qi, stream);                     \
        break;
    switch (J) {
        PVS_RS(1)
        PVS_RS(2)
        PVS_RS(3)
        PVS_RS(4)
        PVS_RS(6)
        PVS_RS(8)
        PVS_RS(12)
        PVS_RS(16)
        default:
            rescore_j<0, false>(ix, qrows, sq, nq, cbase, chunks, pair_cnt, pairs, pair_sub, gamma, keys,
                                cert_cnt, fail, row_reads, fail_qi, stream);
            break;
    }
#undef PVS_RS
}

// ------------------------------------------------------------------ sorting
// Ascending sort of every tile of 512 WAVES keys of every query's region.
// Keys past the region's count are padded with ~0 (no real key: a row id is
// below 2^31) and not written back.
//
// A bitonic network over registers: thread t holds keys [8 t, 8 t + 8), so a
// step of stride below 8 stays inside a thread, below 512 inside a wavefront
// (lane exchanges), and only the strides between wavefronts go through LDS:
// 3 such steps for four wavefronts and 6 for eight.  Every step runs
// ascending: the first step of a merge compares mirrored positions.  Bound by
// the vector instructions of one tile's chain of steps when there are few
// tiles.  One tile of 2,048 keys takes 11.3 us; a network that kept every key
// in LDS, with a barrier after each of its 66 steps, took 64 us.
__device__ __forceinline__ void key_order(uint64_t& a, uint64_t& b) {
    const bool sw = b < a;
    const uint64_t x = sw ? b : a, y = sw ? a : b;
    a = x;
    b = y;
}

// The key of lane l ^ X of a wavefront.  X is a single bit below 64 or a full
// mask 2^k - 1 (a mirrored step).  Inside 16 lanes these are data-parallel
// moves (quad permutations, mirrored lanes, a rotation by 8); across rows of
// 16 and halves of 32 the swap instructions give both sides' values.  The
// LDS lane permutation in their place took 45 us instead of 37 for a tile of 8,192 keys
// and sixteen wavefronts.
template <int CTRL>
__device__ __forceinline__ uint64_t dpp64(uint64_t x) {
    const int lo = __builtin_amdgcn_update_dpp(0, static_cast<int>(x), CTRL, 0xF, 0xF, false);
    const int hi = __builtin_amdgcn_update_dpp(0, static_cast<int>(x >> 32), CTRL, 0xF, 0xF, false);
    return (static_cast<uint64_t>(static_cast<uint32_t>(hi)) << 32) | static_cast<uint32_t>(lo);
}

template <int X>
__device__ __forceinline__ uint64_t lane_xor(uint64_t x) {
    static_assert(X == 1 || X == 2 || X == 3 || X == 4 || X == 7 || X == 8 || X == 15 || X == 16 || X == 31 ||
                      X == 32 || X == 63, "a single bit or a full mask");
    if constexpr (X == 1) return dpp64<0xB1>(x);
    else if constexpr (X == 2) return dpp64<0x4E>(x);
    else if constexpr (X == 3) return dpp64<0x1B>(x);
    else if constexpr (X == 4) return dpp64<0x141>(dpp64<0x1B>(x));   // 7 ^ 3
    else if constexpr (X == 7) return dpp64<0x141>(x);
    else if constexpr (X == 8) return dpp64<0x128>(x);
    else if constexpr (X == 15) return dpp64<0x140>(x);
    else if constexpr (X == 31) return lane_xor<16>(lane_xor<15>(x));
    else if constexpr (X == 63) return lane_xor<32>(lane_xor<31>(x));
    else {
        const uint32_t lo = static_cast<uint32_t>(x), hi = static_cast<uint32_t>(x >> 32);
        const bool upper = (threadIdx.x & X) != 0;
        uint32_t l, h;
        if constexpr (X == 16) {
            const auto a = __builtin_amdgcn_permlane16_swap(lo, lo, false, false);
            const auto c = __builtin_amdgcn_permlane16_swap(hi, hi, false, false);
            l = upper ? a[0] : a[1];
            h = upper ? c[0] : c[1];
        } else {
            const auto a = __builtin_amdgcn_permlane32_swap(lo, lo, false, false);
            const auto c = __builtin_amdgcn_permlane32_swap(hi, hi, false, false);
            l = upper ? a[0] : a[1];
            h = upper ? c[0] : c[1];
        }
        return (static_cast<uint64_t>(h) << 32) | l;
    }
}

template <int WAVES>
__global__ __launch_bounds__(64 * WAVES) void k_sort_tiles(const uint64_t* __restrict__ keys,
                                                           uint64_t* __restrict__ dst, int packed,
                                                           const int32_t* __restrict__ cnt, int cnt_ld,
                                                           const ScanQ* __restrict__ sq) {
    constexpr int PER = 8;
    constexpr int T = 64 * WAVES * PER;
    __shared__ uint64_t s[T];
    const int tid = threadIdx.x;
    const int b = blockIdx.y;
    const int64_t n = cnt[b * cnt_ld];
    const int64_t base = static_cast<int64_t>(blockIdx.x) * T;
    if (base >= n) return;
    const int m = static_cast<int>(min(static_cast<int64_t>(T), n - base));
    const uint64_t* k = keys + sq[b].cand_off + base;
    uint64_t* d = dst + (packed ? packed_offset(cnt, b) : sq[b].cand_off) + base;
    uint64_t v[PER];
    // any assignment of the unsorted keys to threads will do: the coalesced one
#pragma unroll
    for (int i = 0; i < PER; ++i) {
        const int at = i * 64 * WAVES + tid;
        v[i] = at < m ? k[at] : ~0ull;
    }
    // sizes 2, 4, 8: inside the thread
    key_order(v[0], v[1]); key_order(v[2], v[3]); key_order(v[4], v[5]); key_order(v[6], v[7]);
    key_order(v[0], v[3]); key_order(v[1], v[2]); key_order(v[4], v[7]); key_order(v[5], v[6]);
    key_order(v[0], v[1]); key_order(v[2], v[3]); key_order(v[4], v[5]); key_order(v[6], v[7]);
    auto half_clean = [&]() {   // strides 4, 2, 1
        key_order(v[0], v[4]); key_order(v[1], v[5]); key_order(v[2], v[6]); key_order(v[3], v[7]);
        key_order(v[0], v[2]); key_order(v[1], v[3]); key_order(v[4], v[6]); key_order(v[5], v[7]);
        key_order(v[0], v[1]); key_order(v[2], v[3]); key_order(v[4], v[5]); key_order(v[6], v[7]);
    };
    key_order(v[0], v[7]); key_order(v[1], v[6]); key_order(v[2], v[5]); key_order(v[3], v[4]);
    key_order(v[0], v[2]); key_order(v[1], v[3]); key_order(v[4], v[6]); key_order(v[5], v[7]);
    key_order(v[0], v[1]); key_order(v[2], v[3]); key_order(v[4], v[5]); key_order(v[6], v[7]);
    // this thread keeps the smaller keys of each pair when `low`
    auto keep = [&](const uint64_t (&p)[PER], bool low) {
#pragma unroll
        for (int i = 0; i < PER; ++i) v[i] = ((p[i] < v[i]) == low) ? p[i] : v[i];
    };
    auto exchange = [&](uint64_t (&p)[PER], int x, bool mirror) {   // p[i] = thread t ^ x's key
        __syncthreads();
#pragma unroll
        for (int i = 0; i < PER; ++i) s[i * 64 * WAVES + tid] = v[i];
        __syncthreads();
#pragma unroll
        for (int i = 0; i < PER; ++i) p[i] = s[(mirror ? PER - 1 - i : i) * 64 * WAVES + (tid ^ x)];
    };
    // the merge of 2^LEVEL threads' keys: a mirrored step (thread
    // t ^ (2^LEVEL - 1), register 7 - i), then strides 8 x: thread t ^ x
    static_for(
        [&](auto L_) {
            constexpr int LEVEL = decltype(L_)::value + 1;
            uint64_t p[PER];
            if constexpr (LEVEL <= 6) {
#pragma unroll
                for (int i = 0; i < PER; ++i) p[i] = lane_xor<(1 << LEVEL) - 1>(v[PER - 1 - i]);
            } else {
                exchange(p, (1 << LEVEL) - 1, true);
            }
            keep(p, (tid & (1 << (LEVEL - 1))) == 0);
            static_for(
                [&](auto J_) {
                    constexpr int X = 1 << (LEVEL - 2 - decltype(J_)::value);
                    uint64_t r[PER];
                    if constexpr (X < 64) {
#pragma unroll
                        for (int i = 0; i < PER; ++i) r[i] = lane_xor<X>(v[i]);
                    } else {
                        exchange(r, X, false);
                    }
                    keep(r, (tid & X) == 0);
                },
                std::make_integer_sequence<int, LEVEL - 1>{});
            half_clean();
        },
        std::make_integer_sequence<int, WAVES == 1 ? 6 : WAVES == 4 ? 8 : 9>{});
    // through LDS once more, so that neighbouring lanes write neighbouring keys
    __syncthreads();
#pragma unroll
    for (int i = 0; i < PER; ++i) s[tid * PER + i] = v[i];
    __syncthreads();
    for (int i = tid; i < m; i += 64 * WAVES) d[i] = s[i];
}

// One merge level: runs of length `run` (a multiple of kSortTile) are merged
// pairwise, by merge path.  Workgroup (x, b) writes outputs
// [x kSortTile, (x + 1) kSortTile) of query b, which lie in one pair of runs:
// searches on the pair's cross diagonals give the parts of the left and
// right runs that fill them (the left run first among equal keys; keys are
// unique inside a query), those are staged in LDS, and each thread merges
// eight consecutive outputs after a search of its own diagonal there.
__global__ __launch_bounds__(256) void k_merge(const uint64_t* __restrict__ src,
                                               uint64_t* __restrict__ dst, int packed,
                                               const int32_t* __restrict__ cnt, int cnt_ld,
                                               const ScanQ* __restrict__ sq, int64_t run) {
    constexpr int T = kSortTile;
    constexpr int PER = T / 256;
    static_assert(T % 256 == 0, "eight outputs per thread");
    __shared__ uint64_t seg[T];   // the left part, then the right part
    __shared__ uint64_t out[T];
    __shared__ int64_t s_split[2];
    const int b = blockIdx.y;
    const int64_t n = cnt[b * cnt_ld];
    const int64_t o0 = static_cast<int64_t>(blockIdx.x) * T;
    if (o0 >= n) return;
    const int64_t o1 = min(o0 + T, n);
    const uint64_t* s = src + sq[b].cand_off;
    uint64_t* d = dst + (packed ? packed_offset(cnt, b) : sq[b].cand_off);
    const int64_t start = (o0 / (2 * run)) * (2 * run);
    const int64_t mid = min(start + run, n);
    const int64_t end = min(start + 2 * run, n);
    const int64_t la = mid - start, lb = end - mid;
    const uint64_t* A = s + start;
    const uint64_t* B = s + mid;
    // Left-run elements among the first `diag` outputs of the pair: the
    // first m with A[m] > B[diag - 1 - m], searched by a wavefront 64 ways at
    // a time (four dependent loads for runs of millions, not twenty).
    const int lane = threadIdx.x & 63;
    const int wave = threadIdx.x >> 6;
    if (wave < 2) {
        const int64_t diag = (wave == 0 ? o0 : o1) - start;
        int64_t lo = diag > lb ? diag - lb : 0, hi = diag < la ? diag : la;
        while (lo < hi) {   // the same in every lane
            const int64_t m = lo + ((hi - lo) * lane) / 64;   // in [lo, hi), ascending with the lane
            const bool p = A[m] <= B[diag - 1 - m];           // true exactly below the answer
            const int c = __popcll(__ballot(p));              // lanes below the answer
            const int64_t m_below = __shfl(m, c > 0 ? c - 1 : 0, 64);
            const int64_t m_at = __shfl(m, c < 64 ? c : 63, 64);
            const int64_t nlo = c > 0 ? m_below + 1 : lo;
            hi = c < 64 ? m_at : hi;
            lo = nlo;
        }
        if (lane == 0) s_split[wave] = lo;
    }
    __syncthreads();
    const int64_t a0 = s_split[0], a1 = s_split[1];
    const int64_t b0 = (o0 - start) - a0, b1 = (o1 - start) - a1;
    const int na = static_cast<int>(a1 - a0), nb = static_cast<int>(b1 - b0);
    for (int i = threadIdx.x; i < na + nb; i += 256) seg[i] = i < na ? A[a0 + i] : B[b0 + i - na];
    __syncthreads();
    // this thread's outputs [t0, t0 + PER) of the tile
    const int t0 = threadIdx.x * PER;
    if (t0 < na + nb) {
        const uint64_t* sa = seg;
        const uint64_t* sb = seg + na;
        int lo = t0 > nb ? t0 - nb : 0, hi = t0 < na ? t0 : na;
        while (lo < hi) {
            const int m = (lo + hi) >> 1;
            if (sa[m] <= sb[t0 - 1 - m]) lo = m + 1;
            else hi = m;
        }
        int ia = lo, ib = t0 - lo;
        const int t1 = min(t0 + PER, na + nb);
        for (int t = t0; t < t1; ++t) {
            const bool takea = ib >= nb || (ia < na && sa[ia] <= sb[ib]);
            out[t] = takea ? sa[ia++] : sb[ib++];
        }
    }
    __syncthreads();
    for (int i = threadIdx.x; i < na + nb; i += 256) d[o0 + i] = out[i];
}

// Tiles of 512 keys by one wavefront, 2,048 by four, 4,096 by eight: the
// smallest that holds the longest list, so that short lists need no merge
// (one tile of 512 takes 7.3 us, of 2,048 11.3 us; a merge level of a few
// thousand keys takes 8 us and its launch).  Longer lists start from 4,096:
// a tile of 8,192 keys took 37 us, more than two of its halves and a merge.
uint64_t* launch_segmented_sort(uint64_t* keys, uint64_t* tmp, const int32_t* cnt, int32_t cnt_ld,
                                const ScanQ* sq, int32_t nq, int64_t max_cnt, uint64_t* packed,
                                hipStream_t stream) {
    if (nq <= 0 || max_cnt <= 0) return packed ? packed : keys;
    const int64_t tile = max_cnt <= 512 ? 512 : max_cnt <= 2048 ? 2048 : 4096;
    const dim3 grid(static_cast<uint32_t>((max_cnt + tile - 1) / tile), nq);
    uint64_t* a = (packed && tile >= max_cnt) ? packed : keys;
    const int direct = a == packed;
    if (tile == 512)
        hipLaunchKernelGGL(k_sort_tiles<1>, grid, dim3(64), 0, stream, keys, a, direct, cnt, cnt_ld, sq);
    else if (tile == 2048)
        hipLaunchKernelGGL(k_sort_tiles<4>, grid, dim3(256), 0, stream, keys, a, direct, cnt, cnt_ld, sq);
    else
        hipLaunchKernelGGL(k_sort_tiles<8>, grid, dim3(512), 0, stream, keys, a, direct, cnt, cnt_ld, sq);
    uint64_t* b = tmp;
    for (int64_t run = tile; run < max_cnt; run *= 2) {
        const int64_t g = (max_cnt + kSortTile - 1) / kSortTile;
        const bool last = 2 * run >= max_cnt;
        if (last && packed) b = packed;
        hipLaunchKernelGGL(k_merge, dim3(static_cast<uint32_t>(g), nq), dim3(256), 0, stream, a, b,
                           last && packed ? 1 : 0, cnt, cnt_ld, sq, run);
        uint64_t* t = a;
        a = b;
        b = t;
    }
    return a;
}

}  // namespace pvs
