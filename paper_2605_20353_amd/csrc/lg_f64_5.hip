// The sampled loss/gradient kernels in double, order 5: a translation unit of their
// own, so that they build in parallel.
#include "lg_kernels.hpp"

namespace gcp {
GCP_LG_INSTANTIATE(double, 5, false)
}
