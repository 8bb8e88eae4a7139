#include "dev_pool.h"

#include "eahr.h"

#include <algorithm>
#include <cstdint>
#include <list>
#include <mutex>
#include <new>
#include <unordered_map>
#include <vector>

namespace eahr {
namespace {

constexpr int kHostSlot = -1;   // "device" of pinned host memory

struct Block {
    void* p;
    size_t bytes;
    int where;          // device, or kHostSlot
    uint64_t since = 0;   // the clock when it was released
};

struct Pool {
    std::mutex mu;
    std::unordered_map<void*, Block> live;   // handed out
    std::list<Block> kept;                   // oldest first
    uint64_t clock = 0;
};

// Never destroyed: handles may be closed while the process ends, after the
// destructors of static objects.
Pool& pool() {
    static Pool* p = new Pool();
    return *p;
}

void free_block(const Block& b) {
    if (b.where == kHostSlot) (void)hipHostFree(b.p);
    else (void)hipFree(b.p);
}

size_t keep_limit(int where) { return where == kHostSlot ? kKeepHost : kKeepDevice; }

size_t kept_bytes(const Pool& P, int where, size_t* blocks) {
    size_t n = 0;
    *blocks = 0;
    for (const auto& b : P.kept)
        if (b.where == where) {
            n += b.bytes;
            ++*blocks;
        }
    return n;
}

hipError_t raw_alloc(void** p, size_t bytes, bool host) {
    // pinned memory that kernels of every GPU may write
    return host ? hipHostMalloc(p, bytes, hipHostMallocPortable | hipHostMallocMapped) : hipMalloc(p, bytes);
}

}  // namespace

hipError_t pool_alloc(void** p, size_t bytes, bool host) {
    *p = nullptr;
    // whole pages of 4 KiB, or of 2 MiB for large blocks, so that blocks fit
    // requests of about their size again
    const size_t unit = bytes >= (size_t(2) << 20) ? size_t(2) << 20 : size_t(4) << 10;
    bytes = std::max<size_t>(1, (bytes + unit - 1) / unit) * unit;
    int where = kHostSlot;
    if (!host) {
        const hipError_t e = hipGetDevice(&where);
        if (e != hipSuccess) return e;
    }
    Pool& P = pool();
    try {
        {
            std::lock_guard<std::mutex> lk(P.mu);
            // the smallest kept block that fits and is not much larger
            auto best = P.kept.end();
            for (auto it = P.kept.begin(); it != P.kept.end(); ++it)
                if (it->where == where && it->bytes >= bytes && it->bytes <= bytes + bytes / 4 &&
                    (best == P.kept.end() || it->bytes < best->bytes))
                    best = it;
            if (best != P.kept.end()) {
                const Block b = *best;
                P.live.emplace(b.p, b);
                P.kept.erase(best);
                *p = b.p;
                return hipSuccess;
            }
        }
        void* q = nullptr;
        hipError_t e = raw_alloc(&q, bytes, host);
        if (e == hipErrorOutOfMemory) {
            (void)hipGetLastError();
            pool_trim(host);
            e = raw_alloc(&q, bytes, host);
        }
        if (e != hipSuccess) return e;
        try {
            std::lock_guard<std::mutex> lk(P.mu);
            P.live.emplace(q, Block{q, bytes, where});
        } catch (...) {
            free_block(Block{q, bytes, where});
            return hipErrorOutOfMemory;
        }
        *p = q;
        return hipSuccess;
    } catch (const std::bad_alloc&) {
        return hipErrorOutOfMemory;
    }
}

static void release(void* p, bool keep) {
    if (!p) return;
    Pool& P = pool();
    std::list<Block> drop;
    {
        std::lock_guard<std::mutex> lk(P.mu);
        const auto it = P.live.find(p);
        if (it == P.live.end()) return;
        Block b = it->second;
        b.since = P.clock;
        P.live.erase(it);
        try {
            // a block above the limit goes by itself and takes no other with it
            (keep && b.bytes <= keep_limit(b.where) ? P.kept : drop).push_back(b);
        } catch (...) {
            free_block(b);
            return;
        }
        size_t blocks = 0, n = kept_bytes(P, b.where, &blocks);
        for (auto k = P.kept.begin(); k != P.kept.end() && (n > keep_limit(b.where) || blocks > kKeepBlocks);) {
            const auto at = k++;
            if (at->where != b.where) continue;
            n -= at->bytes;
            --blocks;
            drop.splice(drop.end(), P.kept, at);
        }
    }
    for (const auto& b : drop) free_block(b);
}

void pool_release(void* p) { release(p, true); }
void pool_free(void* p) { release(p, false); }

void pool_trim(bool host) {
    int where = kHostSlot;
    if (!host && hipGetDevice(&where) != hipSuccess) return;
    Pool& P = pool();
    std::list<Block> drop;
    {
        std::lock_guard<std::mutex> lk(P.mu);
        for (auto it = P.kept.begin(); it != P.kept.end();) {
            const auto at = it++;
            if (at->where == where) drop.splice(drop.end(), P.kept, at);
        }
    }
    for (const auto& b : drop) free_block(b);
}

void pool_age(int ticks) {
    Pool& P = pool();
    std::list<Block> drop;
    {
        std::lock_guard<std::mutex> lk(P.mu);
        P.clock += static_cast<uint64_t>(ticks);
        while (!P.kept.empty() && P.clock - P.kept.front().since >= kKeepTicks)
            drop.splice(drop.end(), P.kept, P.kept.begin());
    }
    for (const auto& b : drop) free_block(b);
}

}  // namespace eahr

extern "C" void eahr_release_memory(void) {
    eahr::Pool& P = eahr::pool();
    std::list<eahr::Block> drop;
    {
        std::lock_guard<std::mutex> lk(P.mu);
        drop.swap(P.kept);
    }
    for (const auto& b : drop) eahr::free_block(b);
}
