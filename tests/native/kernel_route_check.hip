// Host-side check of which kernels a call runs: those of its order for 3-, 4-
// and 5-way tensors, the wide ones (64-bit row products) exactly from the model
// size on that 32-bit byte offsets do not reach, the general-order ones for
// other orders, bucketed mixed-radix keys and 5-way models of 4 GiB and more.
// Every row that the narrow kernels address has its last byte below 2^32.  Exit
// status 0 = every check passed.
#include "../../paper_2605_20353_amd/csrc/gcp_internal.hpp"

#include <cstdio>

using namespace gcp;

static long g_checks = 0, g_bad = 0;

static void check(int d, int64_t rows, int R, gcp_dtype dt, bool radix, bool bucketed)
{
    gcp_tensor_s t;
    t.d = d;
    t.dt = dt;
    t.layout.radix = radix;
    t.rowoff[d] = rows;
    const KernelOrder o = kernel_order(&t, R, bucketed);
    const bool big = (unsigned __int128)rows * (unsigned)R * (dt == GCP_F32 ? 4 : 8) > 0xffffffffull;
    const bool general = d < 3 || d > 5 || (bucketed && radix) || (d == 5 && big);
    ++g_checks;
    if (o.order == (general ? 0 : d) && o.wide == (!general && big)) return;
    if (g_bad < 10)
        std::printf("order %d, %lld rows, rank %d, %s, radix %d, bucketed %d: kernels of order %d, wide %d\n", d,
                    (long long)rows, R, dt == GCP_F32 ? "float" : "double", radix, bucketed, o.order, o.wide);
    ++g_bad;
}

int main()
{
    for (int d = 1; d <= 8; ++d)
        for (int R : {1, 3, 5, 32, 100, 128, 256})
            for (gcp_dtype dt : {GCP_F32, GCP_F64})
                for (int radix = 0; radix < 2; ++radix)
                    for (int bucketed = 0; bucketed < 2; ++bucketed) {
                        const int64_t edge = (int64_t)(0x100000000ull / ((uint64_t)R * (dt == GCP_F32 ? 4 : 8)));
                        for (int64_t rows : {int64_t(10), edge - 1, edge, edge + 1, 2 * edge, (int64_t(1) << 32) - 1})
                            if (rows >= 1 && rows < (int64_t(1) << 32)) check(d, rows, R, dt, radix, bucketed);
                    }
    std::printf("%ld checks, %ld wrong\n", g_checks, g_bad);
    return g_bad != 0;
}
