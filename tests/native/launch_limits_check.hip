// Host-side check of the grid sizes of the library's streaming launches (the
// gradient's zeroing and Adam's update): a launch may not have 2^32 threads or
// more in a dimension, whatever the arrays' size, and gives every 16 bytes a
// thread as long as that allows.  Exit status 0 = every check passed.
#include "../../paper_2605_20353_amd/csrc/lg_kernels.hpp"

#include <cstdio>

namespace gcp {
int64_t ceil_div(int64_t a, int64_t b) { return (a + b - 1) / b; }
}  // namespace gcp

static long g_checks = 0, g_bad = 0;

static void check(const char* what, int64_t n, unsigned blocks, int64_t items)
{
    ++g_checks;
    const uint64_t threads = (uint64_t)blocks * 256;
    if (blocks >= 1 && threads <= 0xffffffffull && (threads >= (uint64_t)items || threads > 0xffffffffull - 256)) return;
    if (g_bad < 10) std::printf("%s of %lld: %u workgroups\n", what, (long long)n, blocks);
    ++g_bad;
}

int main()
{
    for (int b = 0; b <= 40; ++b)
        for (int64_t n : {(int64_t(1) << b) - 1, int64_t(1) << b, (int64_t(1) << b) + 1, 3 * (int64_t(1) << b) / 2})
            for (int bytes : {4, 8}) check("zeroing", n, gcp::zero_blocks(n, bytes), (n * bytes + 15) / 16);
    for (int64_t items : {int64_t(0), int64_t(1), int64_t(256), int64_t(257), (int64_t(1) << 32) - 257, (int64_t(1) << 32) - 256,
                          (int64_t(1) << 32) - 255, int64_t(1) << 32, int64_t(1) << 38})
        check("streaming", items, gcp::stream_blocks(items), items);
    std::printf("%ld checks, %ld wrong\n", g_checks, g_bad);
    return g_bad != 0;
}
