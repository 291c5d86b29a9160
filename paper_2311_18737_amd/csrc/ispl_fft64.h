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

// sum_j v[j] P^j W_16^{j k} into v[k] for P = W_N^e (see dft16_geo and
// load_geo of the FP32 form); tw(i) is W_N^{i mod N}.
template <typename TW>
__device__ __forceinline__ void dft16_geo64(complex64d (&v)[16], int e, int n_fft, TW tw) {
  const int n16 = n_fft >> 4;
  {
    const complex64d g = tw(4 * e), g2 = tw(8 * e);
#pragma unroll
    for (int j1 = 0; j1 < 4; ++j1) dft4_geo(v[j1], v[j1 + 4], v[j1 + 8], v[j1 + 12], g, g2);
  }
#pragma unroll
  for (int k1 = 0; k1 < 4; ++k1)
    dft4_geo(v[4 * k1], v[4 * k1 + 1], v[4 * k1 + 2], v[4 * k1 + 3], tw(e + k1 * n16),
             tw(2 * e + 2 * k1 * n16));
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
  dft16_geo64(v, 64 * step * kappa, table,
              [&](int i) { return uniform_twiddle64(tw, i & mask); });
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
  dft16_geo64(v, 4 * q, table, [&](int i) { return twiddle64(tw, i & mask); });
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
#pragma unroll
  for (int t = 0; t < 4; ++t) {
    const int e = q + (table >> 6) * (4 * row + t);  // W_n^{q} W_64^{kc}
    dft4_geo(v[4 * t], v[4 * t + 1], v[4 * t + 2], v[4 * t + 3], twiddle64(tw, e & mask),
             twiddle64(tw, (2 * e) & mask));
#pragma unroll
    for (int kd = 0; kd < 4; ++kd) sink(4 * t + kd, v[4 * t + kd]);
  }
}

}  // namespace ispl
