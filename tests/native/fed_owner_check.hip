// Host-side check of the rule for the threads of the batched owner workgroups:
// fewer than 1024 only where all workgroups then start at once, and never where
// the fullest row block would hold the launch up.  Exit status 0 = every check
// passed.
#include "../../paper_2605_20353_amd/csrc/fed_owner.hpp"

#include <cstdio>

using namespace gcp;

static long g_checks = 0, g_bad = 0;

static void expect(int want, int64_t blocks, double total, double largest, int64_t p0, int64_t p1, int64_t p2)
{
    const int64_t places[3] = {p0, p1, p2};
    const int got = fed_owner_threads(blocks, total, largest, places);
    ++g_checks;
    if (got == want) return;
    std::printf("%lld row blocks, %g entries, %g in the fullest, places %lld %lld %lld: %d threads\n", (long long)blocks,
                total, largest, (long long)p0, (long long)p1, (long long)p2, got);
    ++g_bad;
}

int main()
{
    expect(512, 640, 16 * 2 * 65536.0, 65536 * 256 / 5000.0, 512, 1024, 2048);   // equal blocks, two rounds else
    expect(1024, 312, 8 * 2 * 30000.0, 30000 * 128 / 350.0, 256, 768, 1792);      // three full blocks a client
    expect(1024, 648, 8 * 3 * 30000.0, 30000 * 64 / 200.0, 512, 1280, 2560);      // the same, narrower row blocks
    expect(1024, 256, 16 * 65536.0, 65536.0 / 16, 256, 512, 1024);                // all start anyway
    expect(1024, 5000, 5000 * 1000.0, 1000.0, 256, 512, 1024);                    // too many for any size
    expect(256, 1000, 1000 * 1000.0, 1000.0, 250, 500, 1000);                     // equal blocks, four rounds else
    expect(1024, 0, 0.0, 0.0, 256, 512, 1024);
    expect(1024, 10, 100.0, 50.0, 0, 0, 0);
    std::printf("%ld checks, %ld wrong\n", g_checks, g_bad);
    return g_bad != 0;
}
