// Tables and exchange words of the cluster solver.
#include "tip_cluster.h"
#include "tip_kernel_common.h"

namespace tip {

__global__ __launch_bounds__(kBlock) void k_cl_tables(Geom g, int cut, const double* __restrict__ diag,
                                                      const double* __restrict__ w, size_t npad,
                                                      uint32_t* __restrict__ nbr, double2* __restrict__ wgt,
                                                      double* __restrict__ D, uint32_t* __restrict__ site) {
  const size_t e = (size_t)blockIdx.x * kBlock + threadIdx.x;
  if (e >= npad) return;
  const bool pad = e >= g.V;
  // the row's site, and the row of a site: the sides in their order but for
  // `cut`, which comes last
  auto walk = [&](uint32_t in, bool to_site) {
    uint32_t rest = in, step = 1, out = 0;
    for (int o = 0; o < g.ndim; ++o) {
      const int mu = o + 1 == g.ndim ? cut : (o < cut ? o : o + 1);
      if (to_site) {
        out += (rest % g.n[mu]) * g.stride[mu];
        rest /= g.n[mu];
      } else {
        out += coord(in, g, mu) * step;
        step *= g.n[mu];
      }
    }
    return out;
  };
  const uint32_t s = pad ? 0u : walk((uint32_t)e, true);
  D[e] = pad ? 0.0 : diag[s];
  site[e] = s;
  for (int o = 0; o < g.ndim; ++o) {
    const int mu = o + 1 == g.ndim ? cut : (o < cut ? o : o + 1);
    const uint32_t f = nbr_fwd(s, g, mu), b = nbr_bwd(s, g, mu);
    if (o + 1 < g.ndim)
      nbr[o * npad + e] =
          pad ? 0u : (((walk(f, false) - (uint32_t)e) & 0xffffu) | ((walk(b, false) - (uint32_t)e) << 16));
    if (w)
      wgt[o * npad + e] = pad ? make_double2(0.0, 0.0) : make_double2(w[mu * (size_t)g.V + s], w[mu * (size_t)g.V + b]);
  }
}

hipError_t launch_cl_tables(const Geom& g, int cut, const double* diag, const double* coupling, size_t npad,
                            uint32_t* nbr, double2* wgt, double* D, uint32_t* site, hipStream_t st) {
  k_cl_tables<<<(unsigned)((npad + kBlock - 1) / kBlock), kBlock, 0, st>>>(g, cut, diag, coupling, npad, nbr, wgt, D,
                                                                          site);
  return hipGetLastError();
}

__global__ __launch_bounds__(kBlock) void k_cl_reset(unsigned long long* words, size_t n, int* queue) {
  const size_t i = (size_t)blockIdx.x * kBlock + threadIdx.x;
  if (i < n) words[i] = 0;
  if (i == 0) queue[0] = 0, queue[1] = 0x7fffffff;
}

hipError_t launch_cl_reset(unsigned long long* words, size_t n, int* queue, hipStream_t st) {
  k_cl_reset<<<(unsigned)((n + kBlock) / kBlock), kBlock, 0, st>>>(words, n, queue);
  return hipGetLastError();
}

int cl_threads(uint32_t rows) { return rows <= 2048 ? 256 : 512; }

}  // namespace tip
