// Field passes of batches with many small instances (lbm_batch.hpp).
#include <hip/hip_runtime.h>

#include "lbm_batch.hpp"

namespace lbmb {

ManyKernels many_kernels() {
  return ManyKernels{{&k_batch_init<float, false, true>, &k_batch_init<float, true, true>},
                     {&k_batch_init<double, false, true>, &k_batch_init<double, true, true>},
                     &k_batch_moments<true>};
}

}  // namespace lbmb
