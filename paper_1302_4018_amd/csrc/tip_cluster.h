// Interface of the cluster solver (tip_cluster_kernel.h): CG on the real scalar
// operator of a whole lattice with any sides, each system solved by G
// workgroups that keep a slab of it each.  Not part of the public C ABI.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "tip_device.h"

namespace tip {

// One lattice.  Its rows are its sites with the longest dimension moved last;
// they are cut along it into planes (A sites, nz planes), and a slab is a run
// of planes.  The tables are indexed by row and padded by kClPad rows.  The
// longest dimension leaves the smallest planes, so the least halo.
struct ClProblem {
  Geom g;                        // with the probe kind of the call
  const uint32_t* nbr;           // [ndim - 1][npad] distances to the two neighbours along each dimension of the
                                 // plane: forward in the low half word, backward in the high one, both signed
  const double2* wgt;            // [ndim][npad] couplings to the two neighbours; null without couplings
  const double* D;               // [npad] diagonal
  const uint32_t* site;          // [npad] lattice site of the row
  size_t npad;
  double tol2, freeze2;
  uint64_t seed;
  int mask, start_frozen, max_iter, max_restarts, force_iter;
  int mixed;                     // what mixed precision promises: the quadrature b . x + x . r instead of b . x, and
                                 // restarts in place of breakdowns
  uint32_t A, nz;
};
constexpr uint32_t kClPad = 2048;

// One real system: part `part` (0 real, 1 imaginary) of right-hand side m.
struct ClJob {
  int prob, part, parts;
  int64_t m;                     // probe index
  int64_t x;                     // first element of its solution in xout (step parts << logB per site)
  int slot;                      // its place in out and outi
};

// Systems that a team of T workgroups solves at the same time, T / G of them at
// most: jobs job, job + 1, .. of one problem, G workgroups each.
struct ClPacket {
  int job, count, G;
};

// The packets of a launch are taken in order by its teams; every workgroup of
// the launch is resident from start to end.
struct ClArgs {
  const ClProblem* probs;
  const ClJob* jobs;
  const ClPacket* packets;
  int npackets, T, nteams, logB;
  uint32_t Amax;                 // widest plane of the launch
  double* ws;                    // per workgroup: b, ws_rows values
  size_t ws_rows;
  unsigned long long* words;     // per team: two buffers of T sums and of T pairs of counters, the packet, T beats
  unsigned long long* halo;      // per workgroup [2][2][2][Amax]
  double* xout;                  // or null
  double* out;                   // [jobs][3]: quadrature, ||b - A x||^2, ||b||^2
  int* outi;                     // [jobs][3]: state, iterations, restarts
  int* queue;                    // [0] next packet, [1] lowest failed job (packets above it may be skipped)
  int skip;                      // whether they are: jobs are in the order of their probes then
  int* stalled;                  // host memory: set when a wait ran into its limit
  int polls;                     // the limit
};
__host__ __device__ inline size_t cl_team_words(int T) { return (size_t)T * 9 + 1; }
constexpr int kClPolls = 1 << 22;            // some seconds

// Team and place in it of workgroup b.  Workgroups go round robin over the XCDs
// (b mod 8), each with its own L2: the workgroups in one place of their teams,
// which read the same slab of a lattice's tables, share 8 / T XCDs, so that an L2
// holds one slab and not the whole lattice.  (22x36x39 in clusters of two, 128
// systems: 33.5 us an iteration, 35.7 with every place on every XCD.)  nteams is a
// multiple of cl_team_step(T).
__host__ __device__ inline int cl_team_step(int T) { return T >= kNumXcd ? 1 : kNumXcd / T; }
__host__ __device__ inline void cl_place(int T, int b, int& team, int& mate) {
  const int xcd = b % kNumXcd, turn = b / kNumXcd;
  if (T >= kNumXcd) {
    const int turns = T / kNumXcd;
    mate = xcd + kNumXcd * (turn % turns);
    team = turn / turns;
  } else {
    const int per = kNumXcd / T;
    mate = xcd / per;
    team = turn * per + xcd % per;
  }
}

// p with its two halo planes, in 160 KB of LDS beside the sums
constexpr uint32_t kClLdsRows = 20440;
constexpr int kClMaxG = 32;
constexpr int kClRows = 30;                  // rows of r, A p and x in the registers of each of 512 threads
constexpr uint32_t kClMaxRows = kClRows * 512;

hipError_t launch_cl_tables(const Geom& g, int cut, const double* diag, const double* coupling, size_t npad,
                            uint32_t* nbr, double2* wgt, double* D, uint32_t* site, hipStream_t st);
// Clears the exchange words and the queue.
hipError_t launch_cl_reset(unsigned long long* words, size_t n, int* queue, hipStream_t st);
// Threads of the kernel that takes `rows` rows per workgroup, and the rows it
// keeps in LDS for them (whole rounds of its threads).
int cl_threads(uint32_t rows);
inline uint32_t cl_lds_rows(uint32_t rows, uint32_t A) {
  const uint32_t nt = (uint32_t)cl_threads(rows);
  return 2 * A + (rows + nt - 1) / nt * nt;
}
hipError_t launch_cluster_2d(const ClArgs& a, uint32_t rows, bool weighted, hipStream_t st);
hipError_t launch_cluster_3d(const ClArgs& a, uint32_t rows, bool weighted, hipStream_t st);
hipError_t launch_cluster_4d(const ClArgs& a, uint32_t rows, bool weighted, hipStream_t st);
inline hipError_t launch_cluster(int ndim, const ClArgs& a, uint32_t rows, bool weighted, hipStream_t st) {
  return ndim == 2 ? launch_cluster_2d(a, rows, weighted, st)
         : ndim == 3 ? launch_cluster_3d(a, rows, weighted, st)
                     : launch_cluster_4d(a, rows, weighted, st);
}

}  // namespace tip
