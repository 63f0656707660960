// The resident solver on 4-dimensional lattices.
#include "tip_resident_kernel.h"

namespace tip {

hipError_t launch_resident_4d(const ResArgs& a, unsigned grid, hipStream_t st) {
  return launch_resident_dim<4>(a, grid, st);
}

}  // namespace tip
