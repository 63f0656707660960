// The resident solver on 2-dimensional lattices.
#include "tip_resident_kernel.h"

namespace tip {

hipError_t launch_resident_2d(const ResArgs& a, bool eo, unsigned grid, hipStream_t st) {
  return launch_resident_dim<2>(a, eo, grid, st);
}

}  // namespace tip
