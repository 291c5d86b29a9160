// One wave's 1024-point transform in double precision, for the expansion of
// summed grids (HIP only).  Same passes and lane layout as the FP32 transform
// in ispl_fft.h; every pass in geometric twiddle form, every factor an entry of
// a table in double.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "ispl_fft.h"

namespace ispl {

struct complex64d {
  double x, y;
};

__device__ __forceinline__ complex64d cmuladd(complex64d a, complex64d w, complex64d b) {
  return {fma(w.x, b.x, fma(-w.y, b.y, a.x)), fma(w.x, b.y, fma(w.y, b.x, a.y))};
}
__device__ __forceinline__ complex64d twice_minus(complex64d a, complex64d s) {
  return {fma(2.0, a.x, -s.x), fma(2.0, a.y, -s.y)};
}
__device__ __forceinline__ void dft4_geo(complex64d& a0, complex64d& a1, complex64d& a2,
                                         complex64d& a3, complex64d t, complex64d t2) {
  const complex64d t02 = cmuladd(a0, t2, a2);
  const complex64d d02 = twice_minus(a0, t02);
  const complex64d t13 = cmuladd(a1, t2, a3);
  const complex64d u13 = twice_minus(a1, t13);
  a0 = cmuladd(t02, t, t13);
  a2 = twice_minus(t02, a0);
  a1 = cmuladd(d02, complex64d{t.y, -t.x}, u13);  // -i T
  a3 = twice_minus(d02, a1);
}

// Twiddle i of the double table: per lane, or the same for the whole wave.
__device__ __forceinline__ complex64d twiddle64(const double* tw, int i) {
  const double2 w = reinterpret_cast<const double2*>(tw)[i];
  return {w.x, w.y};
}
__device__ __forceinline__ complex64d uniform_twiddle64(const double* tw, int i) {
  typedef double f64x2 __attribute__((ext_vector_type(2)));
  using cptr = const __attribute__((address_space(4))) f64x2*;
  const f64x2 w = reinterpret_cast<cptr>(reinterpret_cast<uint64_t>(tw))[__builtin_amdgcn_readfirstlane(i)];
  return {w.x, w.y};
}

__device__ __forceinline__ complex64d cmul(complex64d a, complex64d b) {
  return {fma(a.x, b.x, -(a.y * b.y)), fma(a.x, b.y, a.y * b.x)};
}
__device__ __forceinline__ complex64d square(complex64d a) {
  return {fma(a.x, a.x, -(a.y * a.y)), 2.0 * (a.x * a.y)};
}

// sum_j v[j] P^j W_16^{j k} into v[k], natural order (see dft16_geo of the FP32
// form), from P, P^2, P^4 and P^8: P^j W_16^{k1} and its square by constants.
__device__ __forceinline__ void dft16_geo64(complex64d (&v)[16], complex64d p, complex64d p2,
                                            complex64d p4, complex64d p8) {
#pragma unroll
  for (int j1 = 0; j1 < 4; ++j1) dft4_geo(v[j1], v[j1 + 4], v[j1 + 8], v[j1 + 12], p4, p8);
  // W_16^{k1} and W_8^{k1}
  constexpr double c = 0.92387953251128675613, s = 0.38268343236508977173;  // cos, sin(pi / 8)
  constexpr double r = 0.70710678118654752440;                              // cos(pi / 4)
  dft4_geo(v[0], v[1], v[2], v[3], p, p2);
  dft4_geo(v[4], v[5], v[6], v[7], cmul(p, {c, -s}), cmul(p2, {r, -r}));
  dft4_geo(v[8], v[9], v[10], v[11], cmul(p, {r, -r}), {p2.y, -p2.x});
  dft4_geo(v[12], v[13], v[14], v[15], cmul(p, {s, -c}), cmul(p2, {-r, -r}));
  complex64d t[16];
#pragma unroll
  for (int i = 0; i < 16; ++i) t[i] = v[4 * (i & 3) + (i >> 2)];
#pragma unroll
  for (int i = 0; i < 16; ++i) v[i] = t[i];
}

// 1024-point transform of v (lane l: v[j] = f[l + 64 j]) with the factors of bin
// class kappa of n = 1024 S points; `tw` is the table of `table` >= n points, xd
// the wave's exchange buffer (XWAVE doubles: real and imaginary parts go
// through it one after the other).  sink(i, F): bin of register i = 4 t + kd.
template <typename Sink>
__device__ __forceinline__ void class_transform64(complex64d (&v)[16], double* xd, const double* tw,
                                                  int n, int table, int kappa, int lane, Sink sink) {
  const int step = table / n, mask = table - 1, S = n >> 10;
  const int ka = lane & 15, row = lane >> 4, q = step * (kappa + S * ka);
  // the lane's two twiddles; their powers are formed (each 64-lane gather holds the CU's
  // address unit for 64 cycles, and eight waves share it)
  const complex64d w = twiddle64(tw, q & mask), w16 = twiddle64(tw, (table >> 4) * row);
  {
    const int e = 64 * step * kappa;
    dft16_geo64(v, uniform_twiddle64(tw, e & mask), uniform_twiddle64(tw, (2 * e) & mask),
                uniform_twiddle64(tw, (4 * e) & mask), uniform_twiddle64(tw, (8 * e) & mask));
  }
  const int p2base = ka * XPITCH + row;
#pragma unroll
  for (int k = 0; k < 16; ++k) xd[k * XPITCH + lane] = v[k].x;
  wave_lds_sync();
#pragma unroll
  for (int m = 0; m < 16; ++m) v[m].x = xd[p2base + 4 * m];
  wave_lds_sync();
#pragma unroll
  for (int k = 0; k < 16; ++k) xd[k * XPITCH + lane] = v[k].y;
  wave_lds_sync();
#pragma unroll
  for (int m = 0; m < 16; ++m) v[m].y = xd[p2base + 4 * m];
  const complex64d p4 = square(square(w)), p8 = square(p4), p16 = square(p8);
  dft16_geo64(v, p4, p8, p16, square(p16));
  wave_lds_sync();
#pragma unroll
  for (int k = 0; k < 16; ++k) xd[64 * k + lane] = v[k].x;
  wave_lds_sync();
#pragma unroll
  for (int t = 0; t < 4; ++t)
#pragma unroll
    for (int r = 0; r < 4; ++r) v[4 * t + r].x = xd[64 * (4 * row + t) + 16 * r + ka];
  wave_lds_sync();
#pragma unroll
  for (int k = 0; k < 16; ++k) xd[64 * k + lane] = v[k].y;
  wave_lds_sync();
#pragma unroll
  for (int t = 0; t < 4; ++t)
#pragma unroll
    for (int r = 0; r < 4; ++r) v[4 * t + r].y = xd[64 * (4 * row + t) + 16 * r + ka];
  wave_lds_sync();
  const complex64d w3 = cmul(w, w16);  // W^q W_64^{kc}, kc = 4 row + t
  // W_64^t
  constexpr double c64[4] = {1.0, 0.99518472667219688624, 0.98078528040323044913, 0.95694033573220886494};
  constexpr double s64[4] = {0.0, 0.09801714032956060199, 0.19509032201612826785, 0.29028467725446236764};
#pragma unroll
  for (int t = 0; t < 4; ++t) {
    const complex64d f = t == 0 ? w3 : cmul(w3, {c64[t], -s64[t]});
    dft4_geo(v[4 * t], v[4 * t + 1], v[4 * t + 2], v[4 * t + 3], f, square(f));
#pragma unroll
    for (int kd = 0; kd < 4; ++kd) sink(4 * t + kd, v[4 * t + kd]);
  }
}

}  // namespace ispl
