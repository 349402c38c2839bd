// Host-side check of how the bit-reproducible form walks a row's run of sorted
// pairs (the same functions the kernel calls), up to the largest call of
// 2^32 - 1 pairs: a run's slices follow each other, cover it and hold whole
// batches; batches follow each other and end with the run; no lane reads
// past the run, and those of a batch read its pairs in order.  Exit status
// 0 = every check passed.
#include "../../paper_2605_20353_amd/csrc/det_runs.hpp"

#include <cstdio>

using namespace gcp;

static long g_checks = 0, g_bad = 0;

static void expect(bool ok, const char* what, uint32_t b, uint32_t e, uint32_t slices, uint32_t batch)
{
    ++g_checks;
    if (ok) return;
    if (g_bad < 10) std::printf("%s: run [%u, %u), %u slices, batches of %u\n", what, b, e, slices, batch);
    ++g_bad;
}

static void check_run(uint32_t b, uint32_t e, uint32_t slices, uint32_t batch)
{
    uint32_t at = b;
    for (uint32_t i = 0; i < slices; ++i) {
        uint32_t lo = 0, hi = 0;
        det_slice(b, e, slices, i, batch, lo, hi);
        expect(lo == at && hi >= lo && hi <= e, "slices follow each other", b, e, slices, batch);
        expect(hi == e || (hi - lo) % batch == 0, "whole batches", b, e, slices, batch);
        at = hi;
        // the slice's last two batches (all of a short one)
        uint32_t p = hi - lo > 3 * batch ? hi - 2 * batch : lo, n = 0;
        for (int steps = 0; p < hi && steps < 9; ++steps, p += n) {
            n = det_batch(p, hi, batch);
            expect(n >= 1 && n <= batch && n <= hi - p && (n == batch || n == hi - p), "batches", b, e, slices, batch);
            for (uint32_t lane = 0; lane < batch; ++lane) {
                const uint32_t x = det_lane(p, hi, lane);
                expect(lane < n ? x - p == lane : x < hi, "lanes", b, e, slices, batch);
            }
        }
        expect(p == hi, "batches end with the slice", b, e, slices, batch);
        if (hi > lo) expect(det_lane(hi, hi, batch - 1) < hi, "read-ahead", b, e, slices, batch);
    }
    expect(at == e, "slices cover the run", b, e, slices, batch);
}

int main()
{
    const uint32_t top = 0xffffffffu;
    const uint32_t lens[] = {1, 2, 7, 8, 9, 63, 64, 65, 511, 512, 513, 2047, 2049, 10007, 1u << 20, (1u << 31) - 5,
                             top - 4096, top - 63, top - 7, top - 1, top};
    for (uint32_t batch : {8u, 16u, 32u, 64u})
        for (uint32_t slices : {4u * (64u / batch), 4u})
            for (uint32_t len : lens)
                for (uint32_t b : {0u, 5u, top / 2, top - len})
                    if ((uint64_t)b + len <= top) check_run(b, b + len, slices, batch);
    std::printf("%ld checks, %ld wrong\n", g_checks, g_bad);
    return g_bad != 0;
}
