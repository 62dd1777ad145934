// The per-vector transform and split of the two-plane INT8 format (Section 4,
// "Cache format"), shared by the key writer, the query split and the fused
// front: a Sylvester Hadamard rotation in FP64 across one wave64 (lane l holds
// elements 64 i + hadamard_lane(l)), the wave's largest magnitude, and the split
// of one element into two INT8 planes under a scale.
#pragma once

#include "fold_device.h"

namespace fold {

constexpr double kLog2eF64 = 0x1.71547652b82fep+0;

template <int CTRL>
__device__ __forceinline__ double dpp_f64(double v) {
  const unsigned long long u = static_cast<unsigned long long>(__double_as_longlong(v));
  const uint32_t lo = static_cast<uint32_t>(__builtin_amdgcn_update_dpp(
      0, static_cast<int>(u), CTRL, 0xF, 0xF, false));
  const uint32_t hi = static_cast<uint32_t>(__builtin_amdgcn_update_dpp(
      0, static_cast<int>(u >> 32), CTRL, 0xF, 0xF, false));
  return __longlong_as_double(
      static_cast<long long>((static_cast<unsigned long long>(hi) << 32) | lo));
}

// v_permlane16_swap / v_permlane32_swap of a value with itself: *lo receives
// the value of the lane whose index bit 4 (ROW = 16) or 5 (32) is clear, *hi of
// the one where it is set.
template <int ROW>
__device__ __forceinline__ void swap_f64(double v, double* lo, double* hi) {
  const unsigned long long u = static_cast<unsigned long long>(__double_as_longlong(v));
  const uint32_t w[2] = {static_cast<uint32_t>(u), static_cast<uint32_t>(u >> 32)};
  unsigned long long l = 0, h = 0;
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const auto r = ROW == 16 ? __builtin_amdgcn_permlane16_swap(w[i], w[i], false, false)
                             : __builtin_amdgcn_permlane32_swap(w[i], w[i], false, false);
    l |= static_cast<unsigned long long>(r[0]) << (32 * i);
    h |= static_cast<unsigned long long>(r[1]) << (32 * i);
  }
  *lo = __longlong_as_double(static_cast<long long>(l));
  *hi = __longlong_as_double(static_cast<long long>(h));
}

// Which element of each 64 a lane of hadamard_wave holds.  The exchanges are
// the wave's register permutes, no LDS: quad swaps for index bits 0 and 1,
// the half-row mirror for bit 2 (it also flips bits 0 and 1), the row mirror
// for bit 3 (it flips 0 to 2 too), row and half swaps for bits 4 and 5; the
// element order makes each of them flip one index bit.
__device__ __forceinline__ int hadamard_lane(int lane) {
  return lane ^ ((lane & 4) ? 3 : 0) ^ ((lane & 8) ? 4 : 0);
}

// x[i] of lane l: element 64 i + hadamard_lane(l).  Strides 1, 2, 4, ... in
// that order.
template <int D>
__device__ __forceinline__ void hadamard_wave(double (&x)[D / 64], int lane) {
  const int e = hadamard_lane(lane);
#pragma unroll
  for (int i = 0; i < D / 64; ++i) {
    double o = dpp_f64<0xB1>(x[i]);  // quad_perm [1, 0, 3, 2]
    x[i] = (e & 1) ? o - x[i] : x[i] + o;
    o = dpp_f64<0x4E>(x[i]);  // quad_perm [2, 3, 0, 1]
    x[i] = (e & 2) ? o - x[i] : x[i] + o;
    o = dpp_f64<0x141>(x[i]);  // row_half_mirror
    x[i] = (e & 4) ? o - x[i] : x[i] + o;
    o = dpp_f64<0x140>(x[i]);  // row_mirror
    x[i] = (e & 8) ? o - x[i] : x[i] + o;
    double lo, hi;
    swap_f64<16>(x[i], &lo, &hi);
    x[i] = (e & 16) ? lo - hi : lo + hi;
    swap_f64<32>(x[i], &lo, &hi);
    x[i] = (e & 32) ? lo - hi : lo + hi;
  }
  if constexpr (D == 128) {
    const double u = x[0], v = x[1];
    x[0] = u + v;
    x[1] = u - v;
  }
}

template <int D>
__device__ __forceinline__ double wave_absmax_f64(const double (&x)[D / 64]) {
  double m = 0.0;
#pragma unroll
  for (int i = 0; i < D / 64; ++i) m = fmax(m, fabs(x[i]));
  m = fmax(m, dpp_f64<0xB1>(m));
  m = fmax(m, dpp_f64<0x4E>(m));
  m = fmax(m, dpp_f64<0x141>(m));
  m = fmax(m, dpp_f64<0x140>(m));
  double lo, hi;
  swap_f64<16>(m, &lo, &hi);
  m = fmax(lo, hi);
  swap_f64<32>(m, &lo, &hi);
  return fmax(lo, hi);
}

__device__ __forceinline__ void split_value(double x, double s, int8_t* a, int8_t* b) {
  if (s > 0.0) {
    const double y = x / s;
    const double ai = rint(y);
    const double bi = fmin(fmax(rint(256.0 * (y - ai)), -128.0), 127.0);
    *a = static_cast<int8_t>(ai);
    *b = static_cast<int8_t>(bi);
  } else {
    *a = 0;
    *b = 0;
  }
}

}  // namespace fold
