// The resident solver on 3-dimensional lattices.
#include "tip_resident_kernel.h"

namespace tip {

hipError_t launch_resident_3d(const ResArgs& a, unsigned grid, hipStream_t st) {
  return launch_resident_dim<3>(a, grid, st);
}

}  // namespace tip
