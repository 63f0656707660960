// Device helpers of the solvers that keep a system in LDS (tip_resident_kernel.h,
// tip_cluster_kernel.h): sums every thread receives, and table rows loaded
// from scalar addresses.
#pragma once

#include "tip_kernel_common.h"

namespace tip {

// Lets a kernel be launched with up to `bytes` of dynamic LDS.
template <class K>
hipError_t allow_lds(K kernel, size_t bytes) {
  return hipFuncSetAttribute(reinterpret_cast<const void*>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize,
                             (int)bytes);
}

// Sum over a wave, in every lane: DPP adds inside rows of 16, across them,
// and the last lane's total read back.  The order is fixed.
template <int CTRL, int ROWS>
__device__ __forceinline__ double dpp_add(double v) {
  const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), CTRL, ROWS, 0xf, false);
  const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), CTRL, ROWS, 0xf, false);
  return v + __hiloint2double(hi, lo);
}
__device__ __forceinline__ double wave_total(double v) {
  v = dpp_add<0x111, 0xf>(v);      // row_shr:1
  v = dpp_add<0x112, 0xf>(v);      // row_shr:2
  v = dpp_add<0x114, 0xf>(v);      // row_shr:4
  v = dpp_add<0x118, 0xf>(v);      // row_shr:8
  v = dpp_add<0x142, 0xa>(v);      // row_bcast:15
  v = dpp_add<0x143, 0xc>(v);      // row_bcast:31
  return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(v), 63),
                          __builtin_amdgcn_readlane(__double2loint(v), 63));
}

// Sum over the workgroup, in every thread, with one barrier.  red is not
// written again before another barrier has passed (the callers alternate).
template <int NT>
__device__ __forceinline__ double wg_total(double v, double* red /* [NT / 64] */) {
  v = wave_total(v);
  if constexpr (NT == 64) return v;
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
  __syncthreads();
  double s = 0.0;
#pragma unroll
  for (int w = 0; w < NT / 64; ++w) s += red[w];
  return s;
}

// Whether a system below `sys` has failed: one load, the same answer in every
// thread, so that a workgroup skips a system as a whole while others fail.
// The word is free again after the next barrier of the workgroup.
template <int NT>
__device__ __forceinline__ bool wg_failed_before(const int* first_failed, int sys, int* word) {
  int f = 0;
  if (threadIdx.x == 0) f = __hip_atomic_load(first_failed, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  if constexpr (NT == 64) return __builtin_amdgcn_readfirstlane(f) < sys;
  __syncthreads();                                    // the word's last reads
  if (threadIdx.x == 0) *word = f;
  __syncthreads();
  return *word < sys;
}

// Neighbours along mu of row e of parity P of an even-odd system (n rows, sides
// powers of two, half-lattice numbering) in the other parity's: along the last
// dimension slices tau + delta and tau - 1 + delta, delta the parity of P and
// the other coordinates.
struct EoNeighbours {
  uint32_t fwd, bwd;
};
template <int ND>
__device__ __forceinline__ EoNeighbours eo_neighbours(const Geom& g, int P, uint32_t e, uint32_t n, int mu) {
  const uint32_t step = 1u << g.shift[mu];
  if (mu + 1 < ND) {
    const uint32_t m = ((1u << g.logn[mu]) - 1u) << g.shift[mu];
    return {(m & (e + step)) | (~m & e), (m & (e - step)) | (~m & e)};
  }
  uint32_t par = e ^ (uint32_t)P;
#pragma unroll
  for (int nu = 1; nu + 1 < ND; ++nu) par ^= e >> g.shift[nu];
  const uint32_t up = e + ((par & 1u) << g.shift[mu]);
  return {up & (n - 1u), (up - step) & (n - 1u)};
}

// A value that is the same in every lane, in scalar registers.
__device__ __forceinline__ uint32_t scalar(uint32_t v) { return (uint32_t)__builtin_amdgcn_readfirstlane((int)v); }
__device__ __forceinline__ double scalar(double v) {
  return __hiloint2double(__builtin_amdgcn_readfirstlane(__double2hiint(v)),
                          __builtin_amdgcn_readfirstlane(__double2loint(v)));
}
template <class T>
__device__ __forceinline__ const T* scalar(const T* p) {
  const uint64_t v = (uint64_t)p;
  return (const T*)((uint64_t)scalar((uint32_t)v) | ((uint64_t)scalar((uint32_t)(v >> 32)) << 32));
}

// A uniform pointer whose value the compiler cannot carry out of a loop: the
// addresses of a thread's rows are then formed where they are used, instead of
// being kept in registers for the whole solve.  It stays a pointer to global
// memory, so its loads count with the vector memory's own counter.
template <class T>
using GlobalPtr = const T __attribute__((address_space(1)))*;
typedef double Double2 __attribute__((ext_vector_type(2)));
template <class T>
__device__ __forceinline__ GlobalPtr<T> opaque(const T* p) {
  asm volatile("" : "+s"(p));
  return (GlobalPtr<T>)p;
}
// p[row + at] with row uniform: a scalar base and a 32-bit byte offset
template <class T>
__device__ __forceinline__ T load_row(GlobalPtr<T> p, uint32_t row, uint32_t at) {
  GlobalPtr<char> base = (GlobalPtr<char>)(p + row);
  asm("" : "+s"(base));                               // formed with scalar adds
  return *(GlobalPtr<T>)(base + at * (uint32_t)sizeof(T));
}

}  // namespace tip
