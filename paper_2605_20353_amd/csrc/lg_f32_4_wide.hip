// The sampled loss/gradient kernels in float, order 4, for models of 4 GiB and
// more: a translation unit of their own, so that they build in parallel.
#include "lg_kernels.hpp"

namespace gcp {
GCP_LG_INSTANTIATE(float, 4, true)
}
