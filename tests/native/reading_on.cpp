// How far ahead scans certify, on the CPU (kernels_fake.h: a scan certifies
// the k ranks it is asked for): a caller that asks once is not made to pay for
// ranks nobody reads by callers that do not need another scan either, and one
// that reads on is served by two scans, and by one from its second state on.
#include <vector>

#include "kernels_fake.h"

#include "eahr.h"

namespace {

constexpr int32_t kDim = 8, kB = 4;
constexpr int64_t kRows = 100000;

struct Read {
    int64_t scans, certified;
};

// One state: a call for each of `pages`, of all queries or of each in turn.
Read read(pvs_index* ix, const std::vector<int32_t>& pages, bool in_turn = false) {
    const std::vector<float> q(kB * kDim, 1.0f);
    pvs_state* st = nullptr;
    fake::expect(pvs_open(ix, 0, q.data(), kB, EAHR_PTR_HOST, &st) == EAHR_OK, "open");
    int64_t at = 0;
    for (const int32_t m : pages) {
        std::vector<int64_t> ids(static_cast<size_t>(kB) * m, -1);
        std::vector<float> sc(ids.size());
        std::vector<int32_t> cnt(kB), sts(kB);
        for (int32_t turn = 0; turn < (in_turn ? kB : 1); ++turn) {
            uint8_t active[kB] = {};
            active[turn] = 1;
            fake::expect(pvs_next(st, m, in_turn ? active : nullptr, ids.data(), sc.data(), cnt.data(), sts.data()) ==
                             EAHR_OK, "next");
        }
        for (int32_t b = 0; b < kB; ++b)
            for (int32_t i = 0; i < m && at + i < pvs::g_rows; ++i)
                fake::expect(ids[static_cast<size_t>(b) * m + i] == at + i, "a rank is wrong");
        at += m;
    }
    pvs_counters c{};
    fake::expect(pvs_stats(st, &c) == EAHR_OK, "stats");
    pvs_close(st);
    return {c.scans, c.certified};
}

}  // namespace

int main() {
    pvs::g_by_k = true;
    pvs::g_rows = kRows;
    const std::vector<float> rows(kRows * kDim, 1.0f);
    pvs_index* ix = nullptr;
    fake::expect(pvs_build(rows.data(), kRows, kDim, EAHR_PTR_HOST, nullptr, &ix) == EAHR_OK, "build");
    const Read once = read(ix, {20});
    fake::expect(once.scans == 1, "one request takes one scan");
    auto shallow = [&](const char* what) {
        const Read r = read(ix, {20});
        fake::expect(r.scans == 1 && r.certified == once.certified, what);
    };
    fake::expect(read(ix, {20, 20}).scans == 1, "two short pages take one scan");
    shallow("two pages from one scan made the next state's deeper");
    fake::expect(read(ix, {20}, true).scans == kB, "queries in turn take a scan each");
    shallow("queries read in turn made the next state's scan deeper");
    const std::vector<int32_t> deep = {640, 1280, 2560, 5120};
    fake::expect(read(ix, deep).scans <= 3, "a first state that reads on");
    for (int i = 0; i < 5; ++i) fake::expect(read(ix, deep).scans == 1, "a later state that reads on takes one scan");
    fake::expect(read(ix, {20}).certified > once.certified, "the rule is not tested");
    fake::expect(read(ix, {20}).certified > once.certified, "the rule is not tested");
    shallow("states that asked once did not end the deep scans");
    // past the end of the list, from one scan
    fake::expect(read(ix, {static_cast<int32_t>(kRows) - 1, 5, 5}).scans <= 2, "a whole list");
    // the queries of a first state that reads on run out of certified ranks at
    // different requests, and share their second scan
    for (int i = 0; i < 3; ++i) read(ix, {20});
    pvs::g_spread = 15;
    const Read pages = read(ix, {400, 400, 400, 400, 400, 400});
    fake::expect(pages.scans == 2, "queries that run out one after another take a scan each");
    pvs::g_spread = 0;
    pvs_free(ix);
    // a collection that one shallow scan certifies whole
    pvs::g_rows = 200;
    fake::expect(pvs_build(rows.data(), 200, kDim, EAHR_PTR_HOST, nullptr, &ix) == EAHR_OK, "build");
    const Read all = read(ix, {150});
    fake::expect(read(ix, {150, 150, 150}).scans <= 2, "a short list");
    pvs_free(ix);
    std::printf("ok %ld %ld\n", static_cast<long>(once.certified), static_cast<long>(all.certified));
    return 0;
}
