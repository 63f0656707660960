// The cluster solver on 3-dimensional lattices.
#include "tip_cluster_kernel.h"

namespace tip {

hipError_t launch_cluster_3d(const ClArgs& a, uint32_t rows, bool weighted, hipStream_t st) {
  return launch_cluster_dim<3>(a, rows, weighted, st);
}

}  // namespace tip
