// CG on the real scalar operator of a whole lattice, one system solved by G
// workgroups, each with a slab of planes of the longest dimension.
//
// A workgroup keeps its slab of p and the two planes beside it in LDS and r and
// A p in registers, and runs the whole solve in one launch.  With G > 1 an
// iteration exchanges two sums (p^H A p, ||r||^2) and, with the second, the
// boundary planes of r: a neighbour forms p = r + beta p on its halo planes by
// itself.  All exchanges go through self-validating words in memory, 3-4 us an
// iteration; the workgroups of a cluster are resident together by a cooperative
// launch, and every wait has a limit: for whole solves one that starts again while
// they make progress.  A launch that ran into it is left to the block solver.
//
// Bound, like the resident solver, by the tables each CU reads from L2: 20 ndim
// + 4 bytes per row and iteration with couplings.  The least G that holds a
// lattice is used; more only in probe classes, when CUs would idle.  Measured (block solver ->
// this): 16 uneven 3-D tori, sides 8..48, 1180 systems, 86.5 -> 21.9 ms in FP64
// and, in place of the single-precision passes, 76.9 -> 21.9 ms; 21x34x15, 50
// probes, set-up included, 8.4 -> 1.03 ms.  An iteration of one system alone
// takes 8.1 us with 7500 rows and 9.4 with 15000, on a loaded chip 10.5 and 21.4.
#pragma once

#include "tip_cluster.h"
#include "tip_lds_common.h"

namespace tip {

// A word that carries its own validity: 32 bits of payload under a 32-bit tag
// (the exchange's number).  A reader polls the word itself, so a value needs
// no flag and no order among stores; relaxed accesses of agent scope, which
// go past the XCDs' separate L2s, are enough.
__device__ __forceinline__ void put_word(unsigned long long* w, uint32_t v, uint32_t tag) {
  __hip_atomic_store(w, ((unsigned long long)tag << 32) | v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void put_double(unsigned long long* w, size_t hi, double v, uint32_t tag) {
  put_word(w, (uint32_t)__double2loint(v), tag);
  put_word(w + hi, (uint32_t)__double2hiint(v), tag);
}
// Waits for the word's tag, at most `polls` polls and not past another
// thread's stall.  A word whose writer may be in the middle of a solve comes with
// the writer's beat: the count starts again whenever that has changed.  A solve
// makes at most max_iter iterations, so every wait ends.
__device__ __forceinline__ bool get_word(const unsigned long long* w, uint32_t tag, int* stalled, int polls,
                                         const unsigned long long* beat, uint32_t& v) {
  unsigned long long seen = 0;
  for (int n = 0;;) {
    const unsigned long long x = __hip_atomic_load(w, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    v = (uint32_t)x;
    if ((uint32_t)(x >> 32) == tag) return true;
    const bool last = ++n >= polls;
    if (!last && (n & 1023) != 0) continue;
    if (__hip_atomic_load(stalled, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM)) return false;
    const unsigned long long b = beat ? __hip_atomic_load(beat, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : 0;
    if (b != seen) {
      seen = b;
      n = 0;
    } else if (last) {
      break;
    }
  }
  __hip_atomic_store(stalled, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
  return false;
}
constexpr int kClBeat = 64;                  // iterations between a workgroup's beats, 2 ms at the most
constexpr int kNotPositive = 64;             // a state besides those of the results: p^H A p <= 0
// M numbers at once, word i at w(i) and w(i) + hi where want(i): every word is
// asked for before any is waited for, so that M numbers cost one trip to
// memory, not 2 M.  NaN when the wait ran into its limit; the solve then ends as
// a breakdown.
template <int M, class Want, class At>
__device__ __forceinline__ void get_doubles(size_t hi, uint32_t tag, int* stalled, int polls, double (&out)[M],
                                            Want&& want, At&& w) {
  bool got[M];
#pragma unroll
  for (int i = 0; i < M; ++i) {
    got[i] = !want(i);
    out[i] = 0.0;
  }
  for (int n = 0;; ++n) {
    unsigned long long l[M], h[M];
#pragma unroll
    for (int i = 0; i < M; ++i)
      if (!got[i]) {
        l[i] = __hip_atomic_load(w(i), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        h[i] = __hip_atomic_load(w(i) + hi, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      }
    bool all = true;
#pragma unroll
    for (int i = 0; i < M; ++i)
      if (!got[i]) {
        got[i] = (uint32_t)(l[i] >> 32) == tag && (uint32_t)(h[i] >> 32) == tag;
        out[i] = __hiloint2double((int)(uint32_t)h[i], (int)(uint32_t)l[i]);
        all = all && got[i];
      }
    if (all) return;
    const bool last = n >= polls;
    if (last) __hip_atomic_store(stalled, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    if (last || ((n & 1023) == 1023 && __hip_atomic_load(stalled, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM))) {
#pragma unroll
      for (int i = 0; i < M; ++i)
        if (!got[i]) out[i] = __longlong_as_double(0x7ff8000000000000ll);
      return;
    }
  }
}

// NT threads, K rows per thread; cl_place gives a workgroup its place in a team.
// A team takes a packet of systems and splits into clusters of G workgroups, so
// that lattices of every size share one launch and keep all CUs busy.  S holds
// the plane below the slab, the slab, the plane above.
template <int ND, bool W, int NT, int K>
__global__ __launch_bounds__(NT) void k_cluster(const ClArgs a) {
  constexpr int PF = K >= 16 ? 2 : 3;                 // rows whose table loads run ahead of the arithmetic
  double* const S = reinterpret_cast<double*>(tip_dyn_lds);
  __shared__ double red[2][NT / 64];
  __shared__ uint32_t s_word[3];
  const uint32_t tid = threadIdx.x;
  const int T = a.T;
  int team, mate;
  cl_place(T, (int)blockIdx.x, team, mate);
  double* const bw = a.ws + (size_t)blockIdx.x * a.ws_rows;
  unsigned long long* const words = a.words + (size_t)team * cl_team_words(T);
  unsigned long long* const packet_word = words + 8 * T;
  unsigned long long* const beats = packet_word + 1;
  auto halo_of = [&](int m) { return a.halo + ((size_t)m * a.nteams + team) * 8 * (size_t)a.Amax; };
  uint32_t sum_tag = 0, halo_tag = 0, packet_tag = 0;

  for (;;) {
    // the next packet, taken by the team's first workgroup.  The clusters of the
    // packet before have made different numbers of exchanges: all go on from the
    // largest, so that no word in memory carries a number still to come.
    ++packet_tag;
    if (tid == 0) {
      uint32_t j = 0, hi = sum_tag, hh = halo_tag;
      if (T > 1) {
        // two buffers: nobody is more than one packet ahead of another
        unsigned long long* const counters = words + 4 * T + (packet_tag & 1) * 2 * T;
        put_word(counters + 2 * mate, sum_tag, packet_tag);
        put_word(counters + 2 * mate + 1, halo_tag, packet_tag);
        for (int m = 0; m < T; ++m) {
          uint32_t v = 0, u = 0;
          // workgroups without a system in a packet, or done with theirs, wait here
          // for whole solves
          if (!get_word(counters + 2 * m, packet_tag, a.stalled, a.polls, beats + m, v) ||
              !get_word(counters + 2 * m + 1, packet_tag, a.stalled, a.polls, beats + m, u))
            break;
          hi = v > hi ? v : hi;
          hh = u > hh ? u : hh;
        }
      }
      if (mate == 0) {
        for (;;) {
          j = (uint32_t)atomicAdd(&a.queue[0], 1);
          if ((int)j >= a.npackets || !a.skip ||
              __hip_atomic_load(&a.queue[1], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) > a.packets[j].job)
            break;
          for (int k = 0; k < a.packets[j].count; ++k) {
            int* const oi = a.outi + 3 * (size_t)a.jobs[a.packets[j].job + k].slot;
            oi[0] = kPadding, oi[1] = 0, oi[2] = 0;
          }
        }
        if (T > 1) put_word(packet_word, j, packet_tag);
      } else if (!get_word(packet_word, packet_tag, a.stalled, a.polls, nullptr, j)) {
        j = (uint32_t)a.npackets;
      }
      if (T > 1 && __hip_atomic_load(a.stalled, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM)) j = (uint32_t)a.npackets;
      s_word[0] = j;
      s_word[1] = hi;
      s_word[2] = hh;
    }
    __syncthreads();
    const int packet = (int)scalar(s_word[0]);
    sum_tag = scalar(s_word[1]);
    halo_tag = scalar(s_word[2]);
    if (packet >= a.npackets) return;
    const ClPacket pk = a.packets[packet];
    const int G = (int)scalar((uint32_t)pk.G), sub = mate / G, member = mate % G;
    if (sub >= (int)scalar((uint32_t)pk.count)) {
      __syncthreads();                                // s_word is read
      continue;
    }
    const int job = (int)scalar((uint32_t)pk.job) + sub;
    unsigned long long* const halo_me = halo_of(mate);
    const unsigned long long* const halo_dn = halo_of(sub * G + (member + G - 1) % G);
    const unsigned long long* const halo_up = halo_of(sub * G + (member + 1) % G);
    // Sum over the cluster, the same bits in every thread of every workgroup.
    // Two buffers: nobody is more than one sum ahead of another.
    auto total = [&](double v, double* buf) {
      const double mine = wg_total<NT>(v, buf);
      if (G == 1) return mine;
      ++sum_tag;
      unsigned long long* const w = words + (sum_tag & 1) * 2 * T + 2 * sub * G;
      if (tid == 0) put_double(w + 2 * member, 1, mine, sum_tag);
      const int l = (int)(tid & 63);
      double part[1];
      get_doubles<1>(1, sum_tag, a.stalled, a.polls, part, [&](int) { return l < G; }, [&](int) { return w + 2 * l; });
      return wave_total(part[0]);
    };
    const ClJob J = a.jobs[job];
    const ClProblem& pr = a.probs[__builtin_amdgcn_readfirstlane(J.prob)];
    const uint32_t A = scalar(pr.A);
    const uint32_t z0 = scalar((uint32_t)member * pr.nz / (uint32_t)G);
    const uint32_t z1 = scalar((uint32_t)(member + 1) * pr.nz / (uint32_t)G);
    const uint32_t n = (z1 - z0) * A, s0 = z0 * A;
    const uint32_t npad = scalar((uint32_t)pr.npad);
    // in scalar registers: read where they are used, each would cost a trip to
    // memory between the sums of every iteration
    const double tol2 = scalar(pr.tol2), freeze2 = scalar(pr.freeze2);
    const int max_iter = (int)scalar((uint32_t)pr.max_iter), force_iter = (int)scalar((uint32_t)pr.force_iter);
    const uint32_t* const t_nbr = scalar(pr.nbr) + s0;
    const Double2* const t_wgt = scalar(reinterpret_cast<const Double2*>(pr.wgt)) + s0;
    const double* const t_D = scalar(pr.D) + s0;
    double* const P = S + A;                          // the slab
    auto in = [&](uint32_t e) { return e < n; };

    // fin(k, row, hop sum, diagonal) for the thread's rows, from S.  Rows past
    // the slab read table rows and LDS words that exist; fin drops them.
    auto hop = [&](auto&& fin) {
      const GlobalPtr<uint32_t> nb = opaque(t_nbr);
      const GlobalPtr<Double2> wg = opaque(t_wgt);
      const GlobalPtr<double> d = opaque(t_D);
      uint32_t at = tid;
      asm volatile("" : "+v"(at));
      constexpr int NB = PF + 1;
      uint32_t ix[NB][ND - 1];
      Double2 wt[NB][ND];
      double dv[NB];
      auto load = [&](int k) {
        if ((uint32_t)(k * NT) >= n) return;
#pragma unroll
        for (int mu = 0; mu < ND; ++mu) {
          const uint32_t row = (uint32_t)mu * npad + (uint32_t)(k * NT);
          if (mu + 1 < ND) ix[k % NB][mu] = load_row(nb, row, at);
          if constexpr (W) wt[k % NB][mu] = load_row(wg, row, at);
        }
        dv[k % NB] = load_row(d, (uint32_t)(k * NT), at);
      };
#pragma unroll
      for (int k = 0; k < PF; ++k) load(k);
#pragma unroll
      for (int k = 0; k < K; ++k) {
        if ((uint32_t)(k * NT) >= n) break;
        if (k + PF < K) load(k + PF);
        asm volatile("" ::: "memory");                // keep the loads where they are
        double f[ND], b[ND], h = 0.0;
        const int l = (int)(at + (uint32_t)(k * NT));
#pragma unroll
        for (int mu = 0; mu < ND; ++mu) {
          if (mu + 1 < ND) {
            const int v = (int)ix[k % NB][mu];
            f[mu] = P[l + (int)(short)(v & 0xffff)];
            b[mu] = P[l + (v >> 16)];
          } else {
            f[mu] = P[l + (int)A];
            b[mu] = P[l - (int)A];
          }
        }
        __builtin_amdgcn_sched_barrier(0);            // all LDS reads of the row in flight together
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
        fin(k, at + (uint32_t)(k * NT), h, dv[k % NB]);
      }
    };
    auto rows = [&](auto&& f) {
      uint32_t at = tid;
      asm volatile("" : "+v"(at));
#pragma unroll
      for (int k = 0; k < K; ++k) {
        if ((uint32_t)(k * NT) >= n) break;
        if (k % 8 == 0) asm volatile("" ::: "memory");
        f(k, at + (uint32_t)(k * NT));
      }
    };
    auto row_of = [&](auto* v, int k, uint32_t e) -> auto& { return (v + k * NT)[e - (uint32_t)(k * NT)]; };

    // The boundary planes of a vector, one number per plane site and side
    // (0 the slab's first plane, 1 its last), in one of two buffers: between
    // two exchanges lies a sum.
    auto put_halo = [&](int side, uint32_t i, double v) {
      put_double(halo_me + ((size_t)(halo_tag & 1) * 2 + side) * 2 * a.Amax + i, a.Amax, v, halo_tag);
    };
    // f(word of S, neighbour's value) for the words of the two halo planes
    auto halo_words = [&](auto&& f) {
      constexpr int M = 4;
      for (uint32_t i0 = tid; i0 < 2 * A; i0 += M * NT) {
        double v[M];
        auto at = [&](int j) { return i0 + (uint32_t)(j * NT); };
        if (G == 1) {
#pragma unroll
          for (int j = 0; j < M; ++j)
            if (at(j) < 2 * A) v[j] = at(j) >= A ? P[at(j) - A] : P[n - A + at(j)];
        } else {
          get_doubles<M>(a.Amax, halo_tag, a.stalled, a.polls, v, [&](int j) { return at(j) < 2 * A; },
                         [&](int j) {
                           const bool up = at(j) >= A;
                           return (up ? halo_up : halo_dn) + ((size_t)(halo_tag & 1) * 2 + (up ? 0 : 1)) * 2 * a.Amax +
                                  (up ? at(j) - A : at(j));
                         });
        }
#pragma unroll
        for (int j = 0; j < M; ++j)
          if (at(j) < 2 * A) f(at(j) >= A ? P[n + at(j) - A] : S[at(j)], v[j]);
      }
    };
    // the halo planes of the vector whose slab is in P
    auto fill_halo = [&]() {
      __syncthreads();
      ++halo_tag;
      if (G > 1)
        for (uint32_t i = tid; i < A; i += NT) {
          put_halo(0, i, P[i]);
          put_halo(1, i, P[n - A + i]);
        }
      halo_words([](double& w, double v) { w = v; });
      __syncthreads();
    };

    // right-hand side
    double r[K], t[K], x[K];
    double acc = 0.0;
    for (uint32_t e = tid; e < n; e += NT) {
      const double2 v = probe_entry(pr.site[s0 + e], (uint64_t)J.m, 0, pr.g, pr.seed, pr.mask);
      const double b = J.part ? v.y : v.x;
      bw[e] = b;
      P[e] = b;
      acc = fma(b, b, acc);
    }
    const double bnorm2 = total(acc, red[0]);
    rows([&](int k, uint32_t e) {
      r[k] = in(e) ? row_of(bw, k, e) : 0.0;
      x[k] = 0.0;
    });
    fill_halo();
    double rho = bnorm2;
    int it = 0, restarts = 0;
    int state = (pr.start_frozen || bnorm2 == 0.0) ? kFrozen : kActive;
    double q = 0.0, rt2 = 0.0;
    for (;;) {
      while (state == kActive) {
        acc = 0.0;
        hop([&](int k, uint32_t e, double h, double d) {
          const double pk = in(e) ? row_of(P, k, e) : 0.0;
          t[k] = in(e) ? fma(d, pk, -h) : 0.0;
          acc = fma(pk, t[k], acc);
        });
        const double pAp = total(acc, red[0]);
        if (!(pAp > 0.0) || !isfinite(pAp) || (force_iter > 0 && restarts == 0 && it + 1 == force_iter)) {
          state = kNotPositive;
          break;
        }
        const double alpha = rho / pAp;
        acc = 0.0;
        ++halo_tag;
        rows([&](int k, uint32_t e) {
          r[k] = fma(-alpha, t[k], r[k]);
          acc = fma(r[k], r[k], acc);
          if (G > 1) {
            if ((uint32_t)(k * NT) < A && e < A) put_halo(0, e, r[k]);
            if ((uint32_t)(k * NT + NT) > n - A && in(e) && e >= n - A) put_halo(1, e - (n - A), r[k]);
          }
        });
        const double rho_new = total(acc, red[1]);
        ++it;
        if (tid == 0 && G < T && it % kClBeat == 0)
          put_word(beats + mate, (uint32_t)it, packet_tag);
        if (!isfinite(rho_new)) state = kBreakdown;
        else if (rho_new <= (restarts == 0 ? freeze2 : tol2) * bnorm2) state = kFrozen;
        else if (it >= max_iter) state = kNoConv;
        const double beta = rho_new / rho;
        rho = rho_new;
        // x += alpha p; p = r + beta p, on the halo planes from the neighbours' r
        rows([&](int k, uint32_t e) {
          const double pk = in(e) ? row_of(P, k, e) : 0.0;
          x[k] = fma(alpha, pk, x[k]);
          if (in(e)) row_of(P, k, e) = fma(beta, pk, r[k]);
        });
        if (G == 1) __syncthreads();
        if (state == kActive) {
          if (G == 1) halo_words([](double& w, double v) { w = v; });
          else halo_words([&](double& w, double v) { w = fma(beta, w, v); });
        }
        __syncthreads();
      }
      // asked for in mixed precision: no breakdown, but a restart from the FP64
      // residual, as the single-precision passes make of it.  (Out of the loop, where
      // its register cost 16 tori 22.5 ms in place of 21.9.)
      if (state == kNotPositive) state = pr.mixed ? kFrozen : kBreakdown;
      if (state != kFrozen) break;
      // the FP64 true residual b - A x
      rows([&](int k, uint32_t e) {
        if (in(e)) row_of(P, k, e) = x[k];
      });
      fill_halo();
      double a0 = 0.0, a1 = 0.0, a2 = 0.0;
      hop([&](int k, uint32_t e, double h, double d) {
        r[k] = 0.0;
        if (!in(e)) return;
        const double xk = row_of(P, k, e), b = row_of(bw, k, e);
        r[k] = b - fma(d, xk, -h);
        a0 = fma(r[k], r[k], a0);
        a1 = fma(b, xk, a1);
        a2 = fma(xk, r[k], a2);
      });
      rt2 = total(a0, red[0]);
      q = total(pr.mixed ? a1 + a2 : a1, red[1]);
      if (rt2 <= tol2 * bnorm2) {
        state = kAccepted;
        break;
      }
      if (restarts >= pr.max_restarts || it >= max_iter || !isfinite(rt2)) {
        state = kNoConv;
        break;
      }
      // restart CG from x: r = p = b - A x
      state = kActive;
      ++restarts;
      rho = rt2;
      rows([&](int k, uint32_t e) {
        if (in(e)) row_of(P, k, e) = r[k];
      });
      fill_halo();
    }
    if (state == kAccepted && a.xout)
      rows([&](int k, uint32_t e) {
        if (in(e)) a.xout[(size_t)J.x + ((size_t)pr.site[s0 + e] << a.logB) * (size_t)J.parts] = x[k];
      });
    if (tid == 0 && member == 0) {
      if (state != kAccepted) atomicMin(&a.queue[1], job);
      double* const oo = a.out + 3 * (size_t)J.slot;
      int* const oi = a.outi + 3 * (size_t)J.slot;
      oo[0] = q;
      oo[1] = rt2;
      oo[2] = bnorm2;
      oi[0] = state;
      oi[1] = it;
      oi[2] = restarts;
    }
    __syncthreads();                                  // S, red and s_word are free for the next system
  }
}

// Up to 1024 rows four per thread, up to 2048 eight, then 512 threads: two
// waves per SIMD, whose 256 registers hold three vectors of 30 rows, of which some
// spill (148 bytes a thread in three dimensions, 36 with 26 rows: 17.5 against
// 16.4 us an iteration at 13125 rows, but 26 rows send more lattices to a second
// workgroup).  Two vectors of 40 rows with x in memory took 23.0 ms on the 16
// tori where this took 22.4.
template <int ND, bool W>
hipError_t launch_cluster_nd(const ClArgs& a, uint32_t rows, hipStream_t st) {
  const size_t lds = (size_t)cl_lds_rows(rows, a.Amax) * sizeof(double);
  auto go = [&](auto kernel, int nt) {
    // the same for every launch: other threads launch the same kernel with other needs
    if (const hipError_t e = allow_lds(kernel, kClLdsRows * sizeof(double)); e != hipSuccess) return e;
    const unsigned grid = (unsigned)(a.nteams * a.T);
    if (a.T == 1) {
      kernel<<<grid, nt, lds, st>>>(a);
      return hipGetLastError();
    }
    // the workgroups of a team wait for one another: all must be resident
    void* args[] = {const_cast<ClArgs*>(&a)};
    return hipLaunchCooperativeKernel(reinterpret_cast<const void*>(kernel), dim3(grid), dim3((unsigned)nt), args,
                                      (unsigned)lds, st);
  };
  if (rows <= 1024) return go(k_cluster<ND, W, 256, 4>, 256);
  if (rows <= 2048) return go(k_cluster<ND, W, 256, 8>, 256);
  if (rows <= 4096) return go(k_cluster<ND, W, 512, 8>, 512);
  if (rows <= 8192) return go(k_cluster<ND, W, 512, 16>, 512);
  if (rows <= kClMaxRows) return go(k_cluster<ND, W, 512, kClRows>, 512);
  return hipErrorInvalidValue;
}

template <int ND>
hipError_t launch_cluster_dim(const ClArgs& a, uint32_t rows, bool weighted, hipStream_t st) {
  return weighted ? launch_cluster_nd<ND, true>(a, rows, st) : launch_cluster_nd<ND, false>(a, rows, st);
}

}  // namespace tip
