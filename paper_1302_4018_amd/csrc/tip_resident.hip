// Tables of the resident solver.
#include "tip_kernel_common.h"
#include "tip_resident.h"

namespace tip {

// Row e of parity P of the even-odd system is the half-lattice index of
// k_eo_hop: x + V3 (t >> 1), x the index of all coordinates but the last.
__global__ __launch_bounds__(kBlock) void k_res_tables(Geom g, int eo, const double* __restrict__ diag,
                                                       const double* __restrict__ w, uint32_t n, uint32_t npad,
                                                       uint32_t* __restrict__ nbr, double2* __restrict__ wgt,
                                                       double* __restrict__ D, double* __restrict__ Dinv,
                                                       uint32_t* __restrict__ site) {
  const uint32_t e = blockIdx.x * kBlock + threadIdx.x;
  const uint32_t P = blockIdx.y;
  if (e >= npad) return;
  const size_t V = g.V, nd = (size_t)g.ndim;
  const uint32_t V3 = g.stride[g.ndim - 1];
  if (e >= n) {
    site[P * npad + e] = 0u;
    D[P * npad + e] = 0.0;
    Dinv[P * npad + e] = 0.0;
    for (size_t mu = 0; mu < nd; ++mu) {
      if (!eo) nbr[(P * nd + mu) * npad + e] = n | (n << 16);
      if (w) wgt[(P * nd + mu) * npad + e] = make_double2(0.0, 0.0);
    }
    return;
  }
  uint32_t s = e;
  if (eo) {
    const uint32_t x3 = e % V3, tau = e / V3;
    uint32_t sum = P;
    for (int mu = 0; mu + 1 < g.ndim; ++mu) sum += coord(x3, g, mu);
    s = x3 + V3 * (2u * tau + (sum & 1u));
  }
  site[P * npad + e] = s;
  D[P * npad + e] = diag[s];
  Dinv[P * npad + e] = diag[V + s];
  for (size_t mu = 0; mu < nd; ++mu) {
    const uint32_t f = nbr_fwd(s, g, (int)mu), b = nbr_bwd(s, g, (int)mu);
    if (!eo) nbr[(P * nd + mu) * npad + e] = f | (b << 16);
    if (w) wgt[(P * nd + mu) * npad + e] = make_double2(w[mu * V + s], w[mu * V + b]);
  }
}

hipError_t launch_res_tables(const Geom& g, bool eo, const double* diag, const double* coupling, uint32_t n,
                             uint32_t npad, uint32_t* nbr, double2* wgt, double* D, double* Dinv, uint32_t* site,
                             hipStream_t st) {
  const dim3 grid((npad + kBlock - 1) / kBlock, eo ? 2 : 1);
  k_res_tables<<<grid, kBlock, 0, st>>>(g, eo ? 1 : 0, diag, coupling, n, npad, nbr, wgt, D, Dinv, site);
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
