// CG on the even-odd system of the covariant operator with one workgroup per
// right-hand side: the resident solver of tip_resident_kernel.h for three
// complex components.  p (48 bytes per row) lies in LDS, r, p and A p in
// registers, x in the workgroup's memory.
//
// Bound by the links, which every workgroup reads from L2: 2 ndim matrices of
// 144 bytes per row and hop.  Up to 2048 rows (8^4): 512 threads with four rows
// each, two waves per SIMD at 256 registers; the loop over dimensions is not
// unrolled, so that two links are in registers at a time, one on its way.  8^4
// with couplings, 64 probes (192 systems, one per CU): 0.82 ms in the kernel, 8.8
// of the 16 lines an XCD's L2 delivers per cycle; estimate and gradient, operator
// set-up included, 3.35 -> 1.64 ms.
#include <algorithm>
#include <type_traits>

#include "tip_lds_common.h"
#include "tip_resident.h"

namespace tip {

template <int ND, bool W, int NT, int K, bool FULL>
__global__ __launch_bounds__(NT) void k_resident_cov(const ResArgs a) {
  using C = double2;
  constexpr bool XREG = K == 1;                       // x in registers, else in the workgroup's memory
  constexpr int RL = K == 4 ? 2 : 0;                  // rows of r in the LDS that p leaves free (48 KB)
  C* const S = reinterpret_cast<C*>(tip_dyn_lds);     // [3][n]
  __shared__ double red[2][NT / 64];
  __shared__ int s_failed;
  const uint32_t tid = threadIdx.x;
  const uint32_t n = FULL ? (uint32_t)(NT * K) : a.t.n;
  const uint32_t npad = a.t.npad;
  C* const be = reinterpret_cast<C*>(a.ws) + (size_t)blockIdx.x * a.ws_stride;   // b on its component, by parity
  C* const bo = be + npad;
  C* const xe = be + 2 * (size_t)npad;                // [3][npad]
  C* const xo = xe + 3 * (size_t)npad;                // [3][npad]
  const double* const D0 = a.t.D;
  const double* const D1 = a.t.D + npad;
  const double* const I1 = a.t.Dinv + npad;
  static_assert(FULL || K == 1, "a system of 64 rows or more is a power of two: FULL");
  auto in = [&](uint32_t e) { return FULL || e < n; };

  // out(k, row, sum_mu [w U x(s + mu) + w' U^H x(s - mu)], d[row]) for the
  // thread's rows of parity P, from the other parity's vector in S
  auto hop = [&](int P, const double* d_, auto&& out) {
    const GlobalPtr<Double2> up = opaque(reinterpret_cast<const Double2*>(a.links) + (size_t)P * ND * 9 * n);
    const GlobalPtr<Double2> un = opaque(reinterpret_cast<const Double2*>(a.links) + (size_t)(1 - P) * ND * 9 * n);
    const GlobalPtr<Double2> wg = opaque(reinterpret_cast<const Double2*>(a.t.wgt) + (size_t)P * ND * npad);
    const GlobalPtr<double> d = opaque(d_);
    uint32_t at = tid;
    asm volatile("" : "+v"(at));
    auto row = [&](int k) { return FULL ? at + (uint32_t)(k * NT) : at & (n - 1u); };
    auto load = [&](GlobalPtr<Double2> u, int mu, uint32_t e, Double2 (&v)[9]) {
#pragma unroll
      for (int q = 0; q < 9; ++q) v[q] = load_row(u, (uint32_t)(mu * 9 + q) * n, e);
    };
    // one link applied to the neighbour in row o
    auto term = [&](const Double2 (&v)[9], bool fwd, uint32_t o, double wgt, C (&h)[3]) {
      C u[9], xn[3];
#pragma unroll
      for (int q = 0; q < 9; ++q) u[q] = make_double2(v[q].x, v[q].y);
#pragma unroll
      for (int c = 0; c < 3; ++c) xn[c] = S[(uint32_t)c * n + o];
      if constexpr (W) {
        C y[3];
        if (fwd) mul_u(u, xn, y);
        else mul_uh(u, xn, y);
        add_weighted<C, 3>(wgt, y, h);
      } else if (fwd) {
        mul_u_acc(u, xn, h);
      } else {
        mul_uh_acc(u, xn, h);
      }
    };
    // two links in registers: one on its way from L2 while the other is applied
    Double2 uf[9], ub[9];
    load(up, 0, row(0), uf);
#pragma unroll
    for (int k = 0; k < K; ++k) {
      const uint32_t e = row(k);
      const double dv = load_row(d, (uint32_t)(k * NT), at);
      C h[3] = {make_double2(0.0, 0.0), make_double2(0.0, 0.0), make_double2(0.0, 0.0)};
#pragma unroll 1
      for (int mu = 0; mu < ND; ++mu) {
        const EoNeighbours nb = eo_neighbours<ND>(a.g, P, e, n, mu);
        Double2 wt = {1.0, 1.0};
        if constexpr (W) wt = load_row(wg, (uint32_t)mu * npad, e);
        load(un, mu, nb.bwd, ub);
        asm volatile("" ::: "memory");
        term(uf, true, nb.fwd, wt.x, h);
        asm volatile("" ::: "memory");
        // the next forward link: the next dimension's, or the next row's first
        const bool more = mu + 1 < ND;
        load(up, more ? mu + 1 : 0, more ? e : row(k + 1 < K ? k + 1 : 0), uf);
        asm volatile("" ::: "memory");
        term(ub, false, nb.bwd, wt.y, h);
        asm volatile("" ::: "memory");
      }
      out(k, at + (uint32_t)(k * NT), h, dv);
    }
  };
  auto rows = [&](auto&& f) {
    uint32_t at = tid;
    asm volatile("" : "+v"(at));
#pragma unroll
    for (int k = 0; k < K; ++k) f(k, at + (uint32_t)(k * NT));
  };
  auto row_of = [&](auto* v, int k, uint32_t e) -> auto& { return (v + k * NT)[e - (uint32_t)(k * NT)]; };
  auto put = [&](uint32_t e, const C (&v)[3]) {
    if (!in(e)) return;
#pragma unroll
    for (int c = 0; c < 3; ++c) S[(uint32_t)c * n + e] = v[c];
  };

  for (int sys = blockIdx.x; sys < a.nsys; sys += gridDim.x) {
    double* const oo = a.out + 4 * (size_t)sys;
    int* const oi = a.outi + 3 * (size_t)sys;
    if (wg_failed_before<NT>(a.first_failed, sys, &s_failed)) {
      if (tid == 0) oi[0] = kPadding, oi[1] = 0, oi[2] = 0;
      continue;
    }
    const int64_t rhs = a.rhs0 + sys;
    const int comp = (int)(rhs % 3);
    double bn = 0.0;
    for (uint32_t e = tid; e < n; e += NT)
      for (int P = 0; P < 2; ++P) {
        const C v = probe_entry(a.t.site[(size_t)P * npad + e], (uint64_t)(rhs / 3), comp, a.g, a.seed, a.mask);
        be[(size_t)P * npad + e] = v;
        bn += norm2(v);
      }
    const double bnorm2 = wg_total<NT>(bn, red[0]);
    // b of a row: its value on the right-hand side's component
    auto rhs_row = [&](const C* b, int k, uint32_t e, C (&v)[3]) {
      const C y = in(e) ? row_of(b, k, e) : make_double2(0.0, 0.0);
#pragma unroll
      for (int c = 0; c < 3; ++c) v[c] = c == comp ? y : make_double2(0.0, 0.0);
    };
    C rr[K - RL][3], p[K][3], t[K][3], x[XREG ? K : 1][3];
    C* const R = S + 3 * n;
    auto get_r = [&](int k, int c) { return k < RL ? R[(k * 3 + c) * NT + (int)tid] : rr[k < RL ? 0 : k - RL][c]; };
    auto set_r = [&](int k, int c, C v) {
      if (k < RL) R[(k * 3 + c) * NT + (int)tid] = v;
      else rr[k < RL ? 0 : k - RL][c] = v;
    };
    double acc = 0.0;
    // reduced right-hand side b_e + H_eo D_o^-1 b_o
    rows([&](int k, uint32_t e) {
      C v[3];
      rhs_row(bo, k, e, v);
      const double f = row_of(I1, k, e);
      for (int c = 0; c < 3; ++c) v[c] = cscale(f, v[c]);
      put(e, v);
    });
    __syncthreads();
    hop(0, D0, [&](int k, uint32_t e, const C (&h)[3], double) {
      C b[3];
      rhs_row(be, k, e, b);
#pragma unroll
      for (int c = 0; c < 3; ++c) {
        p[k][c] = in(e) ? cadd(b[c], h[c]) : make_double2(0.0, 0.0);
        set_r(k, c, p[k][c]);
        acc += norm2(p[k][c]);
        if constexpr (XREG) x[k][c] = make_double2(0.0, 0.0);
        else row_of(xe + c * npad, k, e) = make_double2(0.0, 0.0);
      }
    });
    double rho = wg_total<NT>(acc, red[1]);
    rows([&](int k, uint32_t e) { put(e, p[k]); });
    __syncthreads();
    int it = 0, restarts = 0;
    int state = (a.start_frozen || rho <= a.tol2 * bnorm2) ? kFrozen : kActive;
    double qre = 0.0, qim = 0.0, rt2 = 0.0;
    for (;;) {
      while (state == kActive) {
        hop(1, I1, [&](int k, uint32_t, const C (&h)[3], double d) {
#pragma unroll
          for (int c = 0; c < 3; ++c) t[k][c] = cscale(d, h[c]);
        });
        __syncthreads();
        rows([&](int k, uint32_t e) { put(e, t[k]); });
        __syncthreads();
        acc = 0.0;
        hop(0, D0, [&](int k, uint32_t e, const C (&h)[3], double d) {
#pragma unroll
          for (int c = 0; c < 3; ++c) {
            t[k][c] = in(e) ? csub(cscale(d, p[k][c]), h[c]) : make_double2(0.0, 0.0);
            acc += redot(p[k][c], t[k][c]);
          }
        });
        const double pAp = wg_total<NT>(acc, red[0]);
        if (!(pAp > 0.0) || !isfinite(pAp) || (a.force_iter > 0 && restarts == 0 && it + 1 == a.force_iter)) {
          state = kBreakdown;
          break;
        }
        const double alpha = rho / pAp;
        acc = 0.0;
        rows([&](int k, uint32_t e) {
#pragma unroll
          for (int c = 0; c < 3; ++c) {
            const C v = axpy(-alpha, t[k][c], get_r(k, c));
            set_r(k, c, v);
            acc += norm2(v);
            // x on its way while the sum is formed
            if constexpr (!XREG) t[k][c] = row_of(xe + c * npad, k, e);
          }
        });
        const double rho_new = wg_total<NT>(acc, red[1]);
        ++it;
        if (!isfinite(rho_new)) state = kBreakdown;
        else if (rho_new <= (restarts == 0 ? a.freeze2 : a.tol2) * bnorm2) state = kFrozen;
        else if (it >= a.max_iter) state = kNoConv;
        const double beta = rho_new / rho;
        rho = rho_new;
        rows([&](int k, uint32_t e) {
#pragma unroll
          for (int c = 0; c < 3; ++c) {
            if constexpr (XREG) x[k][c] = axpy(alpha, p[k][c], x[k][c]);
            else row_of(xe + c * npad, k, e) = axpy(alpha, p[k][c], t[k][c]);
            p[k][c] = axpy(beta, p[k][c], get_r(k, c));
          }
          put(e, p[k]);
        });
        __syncthreads();
      }
      if (state != kFrozen) break;
      // the FP64 true residual b - A x and b^H x: x_o = D_o^-1 (b_o + H_oe x_e)
      // with the odd sites' part, then the even sites' part
      rows([&](int k, uint32_t e) {
#pragma unroll
        for (int c = 0; c < 3; ++c) {
          if constexpr (XREG) p[k][c] = x[k][c];
          else p[k][c] = row_of(xe + c * npad, k, e);
        }
        put(e, p[k]);
      });
      __syncthreads();
      double a0 = 0.0, a1 = 0.0, a2 = 0.0;
      hop(1, I1, [&](int k, uint32_t e, const C (&h)[3], double d) {
        C b[3];
        rhs_row(bo, k, e, b);
        const double dd = row_of(D1, k, e);
#pragma unroll
        for (int c = 0; c < 3; ++c) {
          t[k][c] = make_double2(0.0, 0.0);
          if (!in(e)) continue;
          const C y = cadd(b[c], h[c]);
          t[k][c] = cscale(d, y);
          a0 += norm2(axpy(-dd, t[k][c], y));
          a1 += redot(b[c], t[k][c]);
          a2 += imdot(b[c], t[k][c]);
          if (a.xout) row_of(xo + c * npad, k, e) = t[k][c];
        }
      });
      __syncthreads();
      rows([&](int k, uint32_t e) { put(e, t[k]); });
      __syncthreads();
      hop(0, D0, [&](int k, uint32_t e, const C (&h)[3], double d) {
        C b[3];
        rhs_row(be, k, e, b);
#pragma unroll
        for (int c = 0; c < 3; ++c) {
          const C v = in(e) ? csub(b[c], csub(cscale(d, p[k][c]), h[c])) : make_double2(0.0, 0.0);
          set_r(k, c, v);
          a0 += norm2(v);
          a1 += redot(b[c], p[k][c]);
          a2 += imdot(b[c], p[k][c]);
        }
      });
      rt2 = wg_total<NT>(a0, red[0]);
      qre = wg_total<NT>(a1, red[1]);
      __syncthreads();
      qim = wg_total<NT>(a2, red[0]);
      if (rt2 <= a.tol2 * bnorm2) {
        state = kAccepted;
        break;
      }
      if (restarts >= a.max_restarts || it >= a.max_iter || !isfinite(rt2)) {
        state = kNoConv;
        break;
      }
      // restart CG from x: r = p = b - A x
      state = kActive;
      ++restarts;
      rho = rt2;
      rows([&](int k, uint32_t e) {
#pragma unroll
        for (int c = 0; c < 3; ++c) p[k][c] = get_r(k, c);
        put(e, p[k]);
      });
      __syncthreads();
    }
    if (state == kAccepted && a.xout) {
      if constexpr (XREG)
        rows([&](int k, uint32_t e) {
          for (int c = 0; c < 3; ++c)
            if (in(e)) row_of(xe + c * npad, k, e) = x[k][c];
        });
      const size_t block = ((size_t)(sys >> a.logB) * 3 * a.g.V) << a.logB;
      const size_t lane = (size_t)(sys & ((1 << a.logB) - 1));
      C* const xout = reinterpret_cast<C*>(a.xout);
      for (uint32_t e = tid; e < n; e += NT)
        for (int P = 0; P < 2; ++P) {
          const size_t s = a.t.site[(size_t)P * npad + e];
          for (int c = 0; c < 3; ++c)
            xout[block + (((size_t)c * a.g.V + s) << a.logB) + lane] = (P ? xo : xe)[(size_t)c * npad + e];
        }
    }
    if (tid == 0) {
      if (state != kAccepted) atomicMin(a.first_failed, sys);
      oo[0] = qre;
      oo[1] = rt2;
      oo[2] = bnorm2;
      oo[3] = qim;
      oi[0] = state;
      oi[1] = it;
      oi[2] = restarts;
    }
    __syncthreads();                                  // red and S are free for the next system
  }
}

template <int ND, bool W>
hipError_t launch_cov_nd(const ResArgs& a, unsigned grid, hipStream_t st) {
  const uint32_t n = a.t.n;
  size_t lds = (size_t)n * 3 * sizeof(double2);
  if (n == 2048) lds += 2 * 512 * 3 * sizeof(double2);       // rows of r
  auto go = [&](auto kernel, int nt) {
    // a kernel's need is the same in every launch, but for systems of less than 64
    // rows, which need no allowance
    if (const hipError_t e = n < 64 ? hipSuccess : allow_lds(kernel, lds); e != hipSuccess) return e;
    kernel<<<grid, nt, lds, st>>>(a);
    return hipGetLastError();
  };
  if (n < 64) return go(k_resident_cov<ND, W, 64, 1, false>, 64);
  if (n == 64) return go(k_resident_cov<ND, W, 64, 1, true>, 64);
  if (n == 128) return go(k_resident_cov<ND, W, 128, 1, true>, 128);
  if (n == 256) return go(k_resident_cov<ND, W, 256, 1, true>, 256);
  if (n == 512) return go(k_resident_cov<ND, W, 512, 1, true>, 512);
  if (n == 1024) return go(k_resident_cov<ND, W, 512, 2, true>, 512);
  if (n == 2048) return go(k_resident_cov<ND, W, 512, 4, true>, 512);
  return hipErrorInvalidValue;
}

hipError_t launch_resident_cov(const ResArgs& a, unsigned grid, hipStream_t st) {
  auto dim = [&](auto nd) {
    constexpr int ND = decltype(nd)::value;
    return a.t.wgt ? launch_cov_nd<ND, true>(a, grid, st) : launch_cov_nd<ND, false>(a, grid, st);
  };
  return a.g.ndim == 2 ? dim(std::integral_constant<int, 2>{})
         : a.g.ndim == 3 ? dim(std::integral_constant<int, 3>{})
                         : dim(std::integral_constant<int, 4>{});
}

int res_cov_wgs_per_cu(uint32_t n) {
  const int by_lds = kLdsPerCu / (int)(n * 48 + 256);
  const int by_waves = n <= 64 ? 8 : (n <= 256 ? (int)(512 / n) : 1);      // two waves per SIMD
  return std::max(1, std::min(by_lds, by_waves));
}

}  // namespace tip
