// Interface of the resident solver (tip_resident_kernel.h): CG on the even-odd
// system of the real scalar operator (power-of-two sides) with one workgroup
// per right-hand side and the search direction in LDS.  Not part of the public
// C ABI.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "tip_device.h"

namespace tip {

// Per-operator tables, one row per site of one parity P (row e of k_eo_hop's
// half-lattice numbering), padded to npad rows.
struct ResTables {
  const double2* wgt;        // [2][ndim][npad] w_mu(s), w_mu(s - mu); null without couplings
  const double* D;           // [2][npad] diagonal, 0 in padding rows
  const double* Dinv;        // [2][npad] its reciprocal
  const uint32_t* site;      // [2][npad] lattice site of the row
  uint32_t n, npad;
};

// One launch: systems 0 .. nsys-1, system i solving part i % parts (0
// real, 1 imaginary) of right-hand side rhs0 + i / parts.  A is real, so the
// two parts of a complex right-hand side are two real systems, and b^H A^-1 b,
// real for any b, is the sum of their quadratures.
struct ResArgs {
  Geom g;
  ResTables t;
  uint64_t seed;
  int mask;
  int parts;
  int64_t rhs0;
  int nsys;
  int start_frozen, max_iter, max_restarts, force_iter;
  double tol2, freeze2;
  const double* links;       // covariant: the even-odd link layout [2][ndim][9][n] double2
  double* ws;                // per workgroup: b (per parity), x (per parity), npad values each (covariant: npad
                             // and 3 npad complex ones)
  size_t ws_stride;          // values per workgroup
  double* xout;              // [blocks][V][2^logB][parts] solutions on the lattice, or null
  int logB;
  double* out;               // [nsys][3]: b . x, ||b - A x||^2, ||b||^2 (covariant: [nsys][4], Im b^H x last)
  int* outi;                 // [nsys][3]: state, iterations, restarts
  int* first_failed;         // lowest system that failed; systems above it may be skipped
};

constexpr uint32_t kResMaxRows = 16384;      // 8 bytes each in LDS

// Fills the tables on the device (diag: D(x) then 1 / D(x) on the lattice).
hipError_t launch_res_tables(const Geom& g, const double* diag, const double* coupling, uint32_t n, uint32_t npad,
                             double2* wgt, double* D, double* Dinv, uint32_t* site, hipStream_t st);
// Rows the tables are padded to, and workgroups that are resident on one CU.
inline uint32_t res_npad(uint32_t n) { return (n + 2047u) & ~2047u; }
int res_wgs_per_cu(uint32_t n);
int res_cov_wgs_per_cu(uint32_t n);
// first_failed = no system
hipError_t launch_res_reset(int* first_failed, hipStream_t st);
hipError_t launch_resident_2d(const ResArgs& a, unsigned grid, hipStream_t st);
hipError_t launch_resident_3d(const ResArgs& a, unsigned grid, hipStream_t st);
hipError_t launch_resident_4d(const ResArgs& a, unsigned grid, hipStream_t st);
constexpr uint32_t kResMaxRowsCov = 2048;    // 48 bytes each
hipError_t launch_resident_cov(const ResArgs& a, unsigned grid, hipStream_t st);
inline hipError_t launch_resident(const ResArgs& a, unsigned grid, hipStream_t st) {
  return a.g.ndim == 2 ? launch_resident_2d(a, grid, st)
         : a.g.ndim == 3 ? launch_resident_3d(a, grid, st)
                         : launch_resident_4d(a, grid, st);
}

}  // namespace tip
