// The sampled loss/gradient kernels in float, order 3: a translation unit of their
// own, so that they build in parallel.
#include "lg_kernels.hpp"

namespace gcp {
GCP_LG_INSTANTIATE(float, 3, false)
}
