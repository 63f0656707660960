// Tables of the resident solver.
#include "tip_kernel_common.h"
#include "tip_resident.h"

namespace tip {

// Row e of parity P of the even-odd system is the half-lattice index of
// k_eo_hop: x + V3 (t >> 1), x the index of all coordinates but the last.
__global__ __launch_bounds__(kBlock) void k_res_tables(Geom g, const double* __restrict__ diag,
                                                       const double* __restrict__ w, uint32_t n, uint32_t npad,
                                                       double2* __restrict__ wgt, double* __restrict__ D,
                                                       double* __restrict__ Dinv, uint32_t* __restrict__ site) {
  const uint32_t e = blockIdx.x * kBlock + threadIdx.x;
  const uint32_t P = blockIdx.y;
  if (e >= npad) return;
  const size_t V = g.V, nd = (size_t)g.ndim;
  const bool pad = e >= n;
  const uint32_t V3 = g.stride[g.ndim - 1];
  const uint32_t x3 = e % V3, tau = e / V3;
  uint32_t sum = P;
  for (int mu = 0; mu + 1 < g.ndim; ++mu) sum += coord(x3, g, mu);
  const uint32_t s = pad ? 0u : x3 + V3 * (2u * tau + (sum & 1u));
  site[P * npad + e] = s;
  D[P * npad + e] = pad ? 0.0 : diag[s];
  Dinv[P * npad + e] = pad ? 0.0 : diag[V + s];
  if (w)
    for (size_t mu = 0; mu < nd; ++mu)
      wgt[(P * nd + mu) * npad + e] =
          pad ? make_double2(0.0, 0.0) : make_double2(w[mu * V + s], w[mu * V + nbr_bwd(s, g, (int)mu)]);
}

hipError_t launch_res_tables(const Geom& g, const double* diag, const double* coupling, uint32_t n, uint32_t npad,
                             double2* wgt, double* D, double* Dinv, uint32_t* site, hipStream_t st) {
  const dim3 grid((npad + kBlock - 1) / kBlock, 2);
  k_res_tables<<<grid, kBlock, 0, st>>>(g, diag, coupling, n, npad, wgt, D, Dinv, site);
  return hipGetLastError();
}

__global__ void k_res_reset(int* first_failed) { *first_failed = 0x7fffffff; }
hipError_t launch_res_reset(int* first_failed, hipStream_t st) {
  k_res_reset<<<1, 1, 0, st>>>(first_failed);
  return hipGetLastError();
}

int res_wgs_per_cu(uint32_t n) {
  if (n > 4096) return 1;                            // two waves per SIMD by their registers
  const int by_lds = (int)(kLdsPerCu / (((size_t)n + 1) * 8 + 256));
  const int by_waves = n <= 256 ? 16 : (n <= 2048 ? 4 : 2);
  return by_lds < by_waves ? by_lds : by_waves;
}

}  // namespace tip
