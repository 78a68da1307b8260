// Lane exchanges of a 64-lane wave seen as four rows of 16 lanes (lane
// l = c + 16 q), and the refined reciprocal and reciprocal square root, shared
// by the kernels that factorise 16x16 FP64 tiles in registers.
#pragma once

#include <hip/hip_runtime.h>

namespace ln {

using v4d = double __attribute__((ext_vector_type(4)));

__device__ inline void wave_sync() {   // LDS writes of the wave visible to its later reads
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

__device__ inline double join_d(unsigned lo, unsigned hi) {
  return __longlong_as_double(((long long)hi << 32) | lo);
}

__device__ inline double readlane_d(double v, int lane) {
  const long long b = __double_as_longlong(v);
  const int lo = __builtin_amdgcn_readlane((int)b, lane);
  const int hi = __builtin_amdgcn_readlane((int)(b >> 32), lane);
  return join_d(lo, hi);
}

// 1/sqrt(a): hardware estimate refined by two Newton steps
__device__ inline double rsqrt_nr(double a) {
  double y = __builtin_amdgcn_rsq(a);
  y = y * (1.5 - 0.5 * a * y * y);
  y = y * (1.5 - 0.5 * a * y * y);
  return y;
}

// 1/a: hardware estimate refined by two Newton steps on e = 1 - a y
__device__ inline double rcp_nr(double a) {
  double y = __builtin_amdgcn_rcp(a);
  y = fma(y, fma(-a, y, 1.0), y);
  y = fma(y, fma(-a, y, 1.0), y);
  return y;
}

template <int N>
__device__ inline int dpp_row_share(int v) {
  return __builtin_amdgcn_update_dpp(0, v, 0x150 + N, 0xF, 0xF, false);
}

// Lane n of every 16-lane row to all lanes of that row (DPP row broadcast);
// n is a constant once the caller's loop is unrolled.
__device__ inline double row_share_d(double v, int n) {
  const long long b = __double_as_longlong(v);
  int lo = (int)b, hi = (int)(b >> 32);
  switch (n) {
#define PT_ROW_SHARE(N)          \
  case N:                        \
    lo = dpp_row_share<N>(lo);   \
    hi = dpp_row_share<N>(hi);   \
    break;
    PT_ROW_SHARE(0) PT_ROW_SHARE(1) PT_ROW_SHARE(2) PT_ROW_SHARE(3)
    PT_ROW_SHARE(4) PT_ROW_SHARE(5) PT_ROW_SHARE(6) PT_ROW_SHARE(7)
    PT_ROW_SHARE(8) PT_ROW_SHARE(9) PT_ROW_SHARE(10) PT_ROW_SHARE(11)
    PT_ROW_SHARE(12) PT_ROW_SHARE(13) PT_ROW_SHARE(14) PT_ROW_SHARE(15)
#undef PT_ROW_SHARE
  }
  return join_d(lo, hi);
}

// Row g (lanes 16g .. 16g + 15) to all four rows, lane for lane: a permlane16
// swap gives rows (g mod 2) and 2 + (g mod 2) twice each, a permlane32 swap
// then the chosen one four times.
__device__ inline unsigned row_bcast_u(unsigned v, int g) {
  const auto p = __builtin_amdgcn_permlane16_swap(v, v, false, false);
  const unsigned y = (g & 1) ? p[1] : p[0];
  const auto r = __builtin_amdgcn_permlane32_swap(y, y, false, false);
  return (g & 2) ? r[1] : r[0];
}

__device__ inline double row_bcast_d(double v, int g) {
  const long long b = __double_as_longlong(v);
  return join_d(row_bcast_u((unsigned)b, g), row_bcast_u((unsigned)(b >> 32), g));
}

// v of the same lane in the partner row (row q ^ 1, by the permlane16 swap)
// and in the partner half (row q ^ 2, by the permlane32 swap), q the caller's
// row: the swaps give every lane the value of the lower and of the upper
// member of its pair.
__device__ inline double xor16_d(double v, int q) {
  const long long b = __double_as_longlong(v);
  const auto pl = __builtin_amdgcn_permlane16_swap((unsigned)b, (unsigned)b, false, false);
  const auto ph = __builtin_amdgcn_permlane16_swap((unsigned)(b >> 32), (unsigned)(b >> 32), false, false);
  return join_d((q & 1) ? pl[0] : pl[1], (q & 1) ? ph[0] : ph[1]);
}
__device__ inline double xor32_d(double v, int q) {
  const long long b = __double_as_longlong(v);
  const auto pl = __builtin_amdgcn_permlane32_swap((unsigned)b, (unsigned)b, false, false);
  const auto ph = __builtin_amdgcn_permlane32_swap((unsigned)(b >> 32), (unsigned)(b >> 32), false, false);
  return join_d((q & 2) ? pl[0] : pl[1], (q & 2) ? ph[0] : ph[1]);
}

// Sum over the four rows, lane for lane, in every row.
__device__ inline double row_sum_d(double v) {
  long long b = __double_as_longlong(v);
  auto pl = __builtin_amdgcn_permlane16_swap((unsigned)b, (unsigned)b, false, false);
  auto ph = __builtin_amdgcn_permlane16_swap((unsigned)(b >> 32), (unsigned)(b >> 32), false, false);
  v = join_d(pl[0], ph[0]) + join_d(pl[1], ph[1]);
  b = __double_as_longlong(v);
  pl = __builtin_amdgcn_permlane32_swap((unsigned)b, (unsigned)b, false, false);
  ph = __builtin_amdgcn_permlane32_swap((unsigned)(b >> 32), (unsigned)(b >> 32), false, false);
  return join_d(pl[0], ph[0]) + join_d(pl[1], ph[1]);
}

// The same through the LDS crossbar: every lane reads lane addr / 4 (addr =
// 4 (c + 16 g) for row g), two DS instructions instead of the VALU swaps.
__device__ inline double bperm_bcast_d(double v, int addr) {
  const long long b = __double_as_longlong(v);
  const int lo = __builtin_amdgcn_ds_bpermute(addr, (int)b);
  const int hi = __builtin_amdgcn_ds_bpermute(addr, (int)(b >> 32));
  return join_d(lo, hi);
}

// acc += X Y for one 16x16x16 product given the four k-slices of both operands
__device__ inline v4d mfma4(const v4d &a, const v4d &b, v4d acc) {
  acc = __builtin_amdgcn_mfma_f64_16x16x4f64(a[0], b[0], acc, 0, 0, 0);
  acc = __builtin_amdgcn_mfma_f64_16x16x4f64(a[1], b[1], acc, 0, 0, 0);
  acc = __builtin_amdgcn_mfma_f64_16x16x4f64(a[2], b[2], acc, 0, 0, 0);
  acc = __builtin_amdgcn_mfma_f64_16x16x4f64(a[3], b[3], acc, 0, 0, 0);
  return acc;
}

}  // namespace ln
