// The resident solver on 2-dimensional lattices.
#include "tip_resident_kernel.h"

namespace tip {

hipError_t launch_resident_2d(const ResArgs& a, unsigned grid, hipStream_t st) {
  return launch_resident_dim<2>(a, grid, st);
}

}  // namespace tip
