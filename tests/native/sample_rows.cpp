// The rows of the threshold sample (sample_row of pvs_kernels.h): in order, one
// run of every `stride`, all there but for the end, near enough to each other for
// the scans' 32-bit offsets, and spread evenly over rows stored in turn from any
// number of sources.
#include <algorithm>
#include <cstdio>
#include <cstdlib>
#include <vector>

#include "pvs_kernels.h"

static void expect(bool ok, const char* what, long nblocks, long stride, long at) {
    if (ok) return;
    std::printf("FAILED: %s (%ld blocks, stride %ld, at %ld)\n", what, nblocks, stride, at);
    std::exit(1);
}

int main() {
    using namespace pvs;
    const long sizes[] = {1, 2, 63, 2048, 4095, 4096, 4097, 6145, 15625, 16384, 31250, 131072, 137500, 1000003};
    for (const long nb : sizes) {
        const long stride = std::max(1L, nb / 2048);
        const long runs = sample_runs(nb, stride), pos = sample_blocks(nb, stride) * 64, rows = nb * 64;
        expect(runs * stride >= rows / kSampleRun && (runs - 1) * stride < rows / kSampleRun, "runs", nb, stride, runs);
        expect(pos >= runs * kSampleRun && pos < runs * kSampleRun + 64, "positions", nb, stride, pos);
        long there = 0;
        for (long i = 0; i < pos; ++i) {
            const long r = sample_row(i, stride), run = r / kSampleRun;
            expect(r % kSampleRun == i % kSampleRun, "row of a run", nb, stride, i);
            expect(run >= i / kSampleRun * stride && run < (i / kSampleRun + 1) * stride, "run of its stride", nb, stride, i);
            if (stride == 1) expect(r == i, "every row", nb, stride, i);
            if (i % 32 == 31) {
                const long first = sample_row(i - 31, stride);
                expect(r > first && r - first <= 32 * stride + kSampleRun * stride, "span of 32 positions", nb, stride, i);
            }
            there += r < rows;
        }
        expect(there >= (runs - 1) * kSampleRun, "rows past the end", nb, stride, there);
        if (stride == 1) continue;
        std::vector<long> ways = {2, 3, 5, 8, 16, 24, 32, 64, 100, 128, 256, 8 * stride, 16 * stride, 64 * stride};
        for (const long w : ways) {
            if (w > 256 && w > rows / 256) continue;
            const long classes = std::min(w, 64L);   // w sources in turn, in groups of neighbours
            std::vector<long> n(classes, 0);
            for (long i = 0; i < pos; ++i) {
                const long r = sample_row(i, stride);
                if (r < rows) ++n[r % w * classes / w];
            }
            for (long c = 0; c < classes; ++c) {
                long size = 0;
                for (long x = 0; x < w; ++x) size += x * classes / w == c;
                const double share = static_cast<double>(n[c]) / there * w / size;
                expect(share > 0.7 && share < 1.3, "a source's share of the sample", nb, stride, w);
            }
        }
    }
    std::printf("ok\n");
    return 0;
}
