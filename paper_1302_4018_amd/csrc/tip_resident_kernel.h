// CG on the even-odd system of the real scalar operator (power-of-two sides)
// with one workgroup per right-hand side.
//
// A lattice whose search direction fits in the LDS of one CU needs no launch,
// no reduction over workgroups and no vector traffic between the passes of an
// iteration: the workgroup keeps p in LDS, r, p and A p in registers, and
// runs the whole solve -- right-hand side, iterations, FP64 true residual,
// restarts -- in one launch, the scalars of CG held by every thread.  The
// block solver spends six launches of 3-6 us on an iteration of such a lattice.
//
// What bounds it is the operator's tables, read from L2 by every workgroup:
// 16 ndim + 8 bytes per row and hop.  At 32^3 with couplings an iteration moves
// 2.3 MB per CU in 25.6 us: over the whole kernel 8.7 of the 16 lines that an XCD's
// L2 delivers per cycle.
// Measured, one call with a prepared operator (block solver -> this): 16^2, 256
// probes 2.66 -> 0.051 ms; 32^3 with couplings, 512 probes 36.8 -> 3.5 ms.  On
// the way, 32^3: tables hoisted out of the iteration by the compiler and spilled
// 5.4 ms; their addresses formed from scalars where they are used, x fetched
// during the sum of ||r||^2 and seven rows of r in LDS 3.9 ms; neighbour rows
// computed instead of read 3.5 ms.
#pragma once

#include "tip_lds_common.h"
#include "tip_resident.h"

namespace tip {

// NT threads, K rows per thread: thread t owns rows t, t + NT, ...  FULL: the
// system has exactly NT K rows, so no row is tested.
template <int ND, bool W, int NT, int K, bool FULL>
__global__ __launch_bounds__(NT) void k_resident(const ResArgs a) {
  constexpr bool HOIST = K <= 4;                      // the thread's table rows stay in registers for the whole solve
  constexpr int PF = K >= 16 ? 2 : 3;                  // else rows whose table loads run ahead of the arithmetic
  constexpr bool XREG = K <= 8;                       // x in registers, else in the workgroup's memory
  constexpr int RL = K >= 32 ? 7 : 0;                 // rows of r in the LDS that p leaves free (28 KB)
  double* S = reinterpret_cast<double*>(tip_dyn_lds);
  __shared__ double red[2][NT / 64];
  __shared__ int s_failed;
  const uint32_t tid = threadIdx.x;
  const uint32_t n = FULL ? (uint32_t)(NT * K) : a.t.n;
  const uint32_t npad = FULL ? (uint32_t)((NT * K + 2047) & ~2047) : a.t.npad;
  double* const be = a.ws + (size_t)blockIdx.x * a.ws_stride;
  double* const bo = be + npad;
  double* const xe = be + 2 * (size_t)npad;
  double* const xo = xe + npad;

  static_assert(FULL || K == 1, "a system of 64 rows or more is a power of two: FULL");
  auto in = [&](uint32_t e) { return FULL || e < n; };
  // fin(k, row, sum_mu [w_mu(s) S(s + mu) + w_mu(s - mu) S(s - mu)], d[row])
  // for the thread's rows of parity P, from the other parity's vector in S
  auto hop = [&](int P, const double* d_, auto&& fin) {
    const Double2* const wg_ = reinterpret_cast<const Double2*>(a.t.wgt) + (size_t)P * ND * npad;
    const GlobalPtr<Double2> wg = HOIST ? (GlobalPtr<Double2>)wg_ : opaque(wg_);
    const GlobalPtr<double> d = HOIST ? (GlobalPtr<double>)d_ : opaque(d_);
    uint32_t at = tid;
    if constexpr (!HOIST) asm volatile("" : "+v"(at));
    constexpr int NB = HOIST ? K : PF + 1;
    Double2 wt[NB][ND];
    double dv[NB];
    auto load = [&](int k) {
      if (!FULL && (uint32_t)(k * NT) >= n) return;
#pragma unroll
      for (int mu = 0; mu < ND; ++mu)
        if constexpr (W) wt[k % NB][mu] = load_row(wg, (uint32_t)mu * npad + (uint32_t)(k * NT), at);
      dv[k % NB] = load_row(d, (uint32_t)(k * NT), at);
    };
#pragma unroll
    for (int k = 0; k < (HOIST ? K : PF); ++k) load(k);
#pragma unroll
    for (int k = 0; k < K; ++k) {
      if (!FULL && (uint32_t)(k * NT) >= n) break;
      if constexpr (!HOIST) {
        if (k + PF < K) load(k + PF);
        // the compiler would otherwise move every row's loads to the front,
        // out of the iteration even, and spill them
        asm volatile("" ::: "memory");
      }
      double f[ND], b[ND], h = 0.0;
#pragma unroll
      for (int mu = 0; mu < ND; ++mu) {
        // computed, not read: 12 of 68 bytes per row and hop in three dimensions, and
        // the LDS reads would wait for them; rows past the system read its own
        // words and are zeroed below
        const EoNeighbours q = eo_neighbours<ND>(a.g, P, FULL ? at + (uint32_t)(k * NT) : at & (n - 1u), n, mu);
        f[mu] = S[q.fwd], b[mu] = S[q.bwd];
      }
      __builtin_amdgcn_sched_barrier(0);              // all LDS reads of the row in flight together
#pragma unroll
      for (int mu = 0; mu < ND; ++mu) {
        if constexpr (W) {
          h = fma(wt[k % NB][mu].x, f[mu], h);
          h = fma(wt[k % NB][mu].y, b[mu], h);
        } else {
          h += f[mu];
          h += b[mu];
        }
      }
      if constexpr (!FULL) h = in(at) ? h : 0.0;   // K = 1 there
      fin(k, at + (uint32_t)(k * NT), h, dv[k % NB]);
    }
  };
  auto rows = [&](auto&& f) {
    uint32_t at = tid;
    if constexpr (!HOIST) asm volatile("" : "+v"(at));
#pragma unroll
    for (int k = 0; k < K; ++k) {
      if (!FULL && (uint32_t)(k * NT) >= n) break;
      if constexpr (!HOIST)
        if (k % 8 == 0) asm volatile("" ::: "memory");
      f(k, at + (uint32_t)(k * NT));
    }
  };
  // the thread's row k of a vector in memory: a uniform address plus the thread's offset
  auto row_of = [&](auto* v, int k, uint32_t e) -> auto& { return (v + k * NT)[e - (uint32_t)(k * NT)]; };
  double rr[K - RL];
  double* const R = S + n + 1;
  auto get_r = [&](int k) { return k < RL ? R[k * NT + (int)tid] : rr[k < RL ? 0 : k - RL]; };
  auto set_r = [&](int k, double v) {
    if (k < RL) R[k * NT + (int)tid] = v;
    else rr[k < RL ? 0 : k - RL] = v;
  };
  const double* const D0 = a.t.D;
  const double* const D1 = a.t.D + npad;
  const double* const I1 = a.t.Dinv + npad;

  for (int sys = blockIdx.x; sys < a.nsys; sys += gridDim.x) {
    double* const oo = a.out + 3 * (size_t)sys;
    int* const oi = a.outi + 3 * (size_t)sys;
    if (wg_failed_before<NT>(a.first_failed, sys, &s_failed)) {
      if (tid == 0) oi[0] = kPadding, oi[1] = 0, oi[2] = 0;
      continue;
    }
    const int parts = a.parts, part = sys % parts;
    const uint64_t m = (uint64_t)(a.rhs0 + sys / parts);
    auto entry = [&](uint32_t s) { return probe_entry(s, m, 0, a.g, a.seed, a.mask); };
    double bn = 0.0;
    for (uint32_t e = tid; e < n; e += NT)
      for (int P = 0; P < 2; ++P) {
        const double2 v = entry(a.t.site[(size_t)P * npad + e]);
        const double b = part ? v.y : v.x;
        be[(size_t)P * npad + e] = b;
        bn = fma(b, b, bn);
      }
    const double bnorm2 = wg_total<NT>(bn, red[0]);
    double p[K], t[K], x[XREG ? K : 1];
    double acc = 0.0;
    // reduced right-hand side b_e + H_eo D_o^-1 b_o
    rows([&](int k, uint32_t e) {
      if (in(e)) S[e] = row_of(I1, k, e) * row_of(bo, k, e);
    });
    __syncthreads();
    hop(0, D0, [&](int k, uint32_t e, double h, double) {
      p[k] = in(e) ? row_of(be, k, e) + h : 0.0;
      set_r(k, p[k]);
      acc = fma(p[k], p[k], acc);
    });
    rows([&](int k, uint32_t e) {
      if constexpr (XREG) x[k] = 0.0;
      else if (in(e)) st_nt(&row_of(xe, k, e), 0.0);
    });
    double rho = wg_total<NT>(acc, red[1]);
    rows([&](int k, uint32_t e) {
      if (in(e)) S[e] = get_r(k);
    });
    __syncthreads();
    int it = 0, restarts = 0;
    int state = (a.start_frozen || rho <= a.tol2 * bnorm2) ? kFrozen : kActive;
    double q = 0.0, rt2 = 0.0;
    for (;;) {
      while (state == kActive) {
        acc = 0.0;
        hop(1, I1, [&](int k, uint32_t, double h, double d) { t[k] = d * h; });
        __syncthreads();
        rows([&](int k, uint32_t e) {
          if (in(e)) S[e] = t[k];
        });
        __syncthreads();
        hop(0, D0, [&](int k, uint32_t, double h, double d) {
          t[k] = fma(d, p[k], -h);
          acc = fma(p[k], t[k], acc);
        });
        const double pAp = wg_total<NT>(acc, red[0]);
        if (!(pAp > 0.0) || !isfinite(pAp) || (a.force_iter > 0 && restarts == 0 && it + 1 == a.force_iter)) {
          state = kBreakdown;
          break;
        }
        const double alpha = rho / pAp;
        acc = 0.0;
        rows([&](int k, uint32_t e) {
          const double rk = fma(-alpha, t[k], get_r(k));
          set_r(k, rk);
          acc = fma(rk, rk, acc);
          // x on its way while the sum is formed
          if constexpr (!XREG) t[k] = in(e) ? ld_nt(&row_of(xe, k, e)) : 0.0;
        });
        const double rho_new = wg_total<NT>(acc, red[1]);
        ++it;
        if (!isfinite(rho_new)) state = kBreakdown;
        else if (rho_new <= (restarts == 0 ? a.freeze2 : a.tol2) * bnorm2) state = kFrozen;
        else if (it >= a.max_iter) state = kNoConv;
        const double beta = rho_new / rho;
        rho = rho_new;
        // x += alpha p; p = r + beta p (the last reads of S lie before the sums)
        rows([&](int k, uint32_t e) {
          if constexpr (XREG) x[k] = fma(alpha, p[k], x[k]);
          else if (in(e)) st_nt(&row_of(xe, k, e), fma(alpha, p[k], t[k]));
          p[k] = fma(beta, p[k], get_r(k));
          if (in(e)) S[e] = p[k];
        });
        __syncthreads();
      }
      if (state != kFrozen) break;
      // the FP64 true residual b - A x and b . x
      rows([&](int k, uint32_t e) {
        double v;
        if constexpr (XREG) v = x[k];
        else v = in(e) ? row_of(xe, k, e) : 0.0;
        if (in(e)) S[e] = v;
      });
      __syncthreads();
      double a0 = 0.0, a1 = 0.0;
      // x_o = D_o^-1 (b_o + H_oe x_e) and the odd sites' part, then the even sites' part
      hop(1, I1, [&](int k, uint32_t e, double h, double d) {
        t[k] = 0.0;
        if (!in(e)) return;
        const double b = row_of(bo, k, e), y = b + h;
        t[k] = d * y;
        const double ro = fma(-row_of(D1, k, e), t[k], y);
        a0 = fma(ro, ro, a0);
        a1 = fma(b, t[k], a1);
        if (a.xout) row_of(xo, k, e) = t[k];
      });
      __syncthreads();
      rows([&](int k, uint32_t e) {
        if constexpr (!XREG) p[k] = in(e) ? S[e] : 0.0;    // x_e
        if (in(e)) S[e] = t[k];
      });
      __syncthreads();
      hop(0, D0, [&](int k, uint32_t e, double h, double d) {
        double rk = 0.0;
        if (in(e)) {
          double xk;
          if constexpr (XREG) xk = x[k];
          else xk = p[k];
          const double b = row_of(be, k, e);
          rk = b - fma(d, xk, -h);
          a0 = fma(rk, rk, a0);
          a1 = fma(b, xk, a1);
        }
        set_r(k, rk);
      });
      rt2 = wg_total<NT>(a0, red[0]);
      q = wg_total<NT>(a1, red[1]);
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
        p[k] = get_r(k);
        if (in(e)) S[e] = p[k];
      });
      __syncthreads();
    }
    if (state == kAccepted && a.xout) {
      if constexpr (XREG)
        rows([&](int k, uint32_t e) {
          if (in(e)) xe[e] = x[k];
        });
      const int j = sys / parts;
      const size_t lane = (((size_t)(j >> a.logB) * a.g.V) << a.logB) + (size_t)(j & ((1 << a.logB) - 1));
      for (uint32_t e = tid; e < n; e += NT)
        for (int P = 0; P < 2; ++P) {
          const uint32_t s = a.t.site[(size_t)P * npad + e];
          a.xout[(lane + ((size_t)s << a.logB)) * (size_t)parts + (size_t)part] = xe[(size_t)P * npad + e];
        }
    }
    if (tid == 0) {
      if (state != kAccepted) atomicMin(a.first_failed, sys);
      oo[0] = q;
      oo[1] = rt2;
      oo[2] = bnorm2;
      oi[0] = state;
      oi[1] = it;
      oi[2] = restarts;
    }
    __syncthreads();                                  // red and S are free for the next system
  }
}

// Threads and rows per thread.  Up to 256 rows one wave: its sums need no
// barrier.  Up to 2048 rows 256 threads with 8 rows each, above that 512
// threads, two waves per SIMD, whose 256 registers hold the three vectors of
// 32 rows.
template <int ND, bool W>
hipError_t launch_resident_nd(const ResArgs& a, unsigned grid, hipStream_t st) {
  const uint32_t n = a.t.n;
  size_t lds = ((size_t)n + 1) * sizeof(double);
  if (n == 16384) lds += 7 * 512 * sizeof(double);           // rows of r
  auto go = [&](auto kernel, int nt) {
    // a kernel's need is the same in every launch, but for systems of less than 64
    // rows, which need no allowance
    if (const hipError_t e = n < 64 ? hipSuccess : allow_lds(kernel, lds); e != hipSuccess) return e;
    kernel<<<grid, nt, lds, st>>>(a);
    return hipGetLastError();
  };
  if (n < 64) return go(k_resident<ND, W, 64, 1, false>, 64);
  if (n == 64) return go(k_resident<ND, W, 64, 1, true>, 64);
  if (n == 128) return go(k_resident<ND, W, 64, 2, true>, 64);
  if (n == 256) return go(k_resident<ND, W, 64, 4, true>, 64);
  if (n == 512) return go(k_resident<ND, W, 256, 2, true>, 256);
  if (n == 1024) return go(k_resident<ND, W, 256, 4, true>, 256);
  if (n == 2048) return go(k_resident<ND, W, 256, 8, true>, 256);
  if (n == 4096) return go(k_resident<ND, W, 512, 8, true>, 512);
  if (n == 8192) return go(k_resident<ND, W, 512, 16, true>, 512);
  if (n == 16384) return go(k_resident<ND, W, 512, 32, true>, 512);
  return hipErrorInvalidValue;
}

template <int ND>
hipError_t launch_resident_dim(const ResArgs& a, unsigned grid, hipStream_t st) {
  return a.t.wgt ? launch_resident_nd<ND, true>(a, grid, st) : launch_resident_nd<ND, false>(a, grid, st);
}

}  // namespace tip
