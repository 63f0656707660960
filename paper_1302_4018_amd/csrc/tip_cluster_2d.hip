// The cluster solver on 2-dimensional lattices.
#include "tip_cluster_kernel.h"

namespace tip {

hipError_t launch_cluster_2d(const ClArgs& a, uint32_t rows, bool weighted, hipStream_t st) {
  return launch_cluster_dim<2>(a, rows, weighted, st);
}

}  // namespace tip
