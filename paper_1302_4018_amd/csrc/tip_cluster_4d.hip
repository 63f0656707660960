// The cluster solver on 4-dimensional lattices.
#include "tip_cluster_kernel.h"

namespace tip {

hipError_t launch_cluster_4d(const ClArgs& a, uint32_t rows, bool weighted, hipStream_t st) {
  return launch_cluster_dim<4>(a, rows, weighted, st);
}

}  // namespace tip
