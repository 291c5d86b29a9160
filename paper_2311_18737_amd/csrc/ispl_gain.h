// Gain of the grid transforms (host and device).
//
// The transforms of the pulse loop take their twiddles from an FP32 table.  The
// rounding of the few factors on a bin's path scales the bin of a narrow line by a
// fixed 1 + d, |d| up to about 5e-8: harmless where bins are results, but the
// expansion of a summed grid spreads the error of a strong point over its
// neighbours (see ispl_grid.hip).  A radix-4 stage weighs its inputs by
// (1, t, t2, t t2) with rounded t and t2 in the place of (1, T, T^2, T^3); the inputs
// of all but the first pass are samples closer together than a line's envelope changes,
// so the line's bin is off by the mean of the four ratios, (1 + t / T)(1 + t2 / T^2) / 4,
// and by the product of these over the stages.
#pragma once

#include <math.h>
#include <stdint.h>

#include "ispl_internal.h"

namespace ispl {

struct GainProduct {
  double x, y;

  ISPL_HOST_DEVICE void times(double a, double b) {
    const double t = x * a - y * b;
    y = x * b + y * a;
    x = t;
  }
  // One plus the ratio of w = (wr, wi), rounded, to the unit vector (c, s), halved.
  ISPL_HOST_DEVICE void half(float wr, float wi, double c, double s) {
    times(0.5 * (1.0 + wr * c + wi * s), 0.5 * (wi * c - wr * s));
  }
};

// 1 / |gain|^2 of point k of a grid of `len` points (128 ... 16384), from the table
// W_N^i, i < n_fft, in double (its rounded entries are the kernels' FP32 table).
ISPL_HOST_DEVICE inline double grid_gain(const double* tw64, int32_t n_fft, int32_t len, int32_t k) {
  const int32_t mask = n_fft - 1, step = n_fft / len, n16 = n_fft >> 4;
  GainProduct g{1.0, 0.0};
  auto half = [&](int32_t i) {
    const double c = tw64[2 * (i & mask)], s = tw64[2 * (i & mask) + 1];
    g.half(static_cast<float>(c), static_cast<float>(s), c, s);
  };
  auto stage = [&](int32_t i) {  // ratio W_N^i, its square from the table too
    half(i);
    half(2 * i);
  };
  auto progression = [&](int32_t e, int32_t out) {  // dft16_geo of ratio W_N^e, output `out`
    stage(4 * e);
    stage(e + (out & 3) * n16);
  };
  // first pass: constants
  const int32_t classes = len > SUB ? len / SUB : 1, cls = k & (classes - 1);
  const int32_t radix = len > 2 * SUB ? classes : len > SUB ? 16 : len / 64;
  const int32_t col = len > 2 * SUB ? cls : len > SUB ? (k >> 1) & 15 : k & (radix - 1);
  if (len == 2 * SUB && cls == 1) {  // dft16_w32: W_8 (its square exact), then W_32 W_16^col
    const double c = tw64[2 * (n_fft >> 3)], s = tw64[2 * (n_fft >> 3) + 1];
    g.half(static_cast<float>(c), static_cast<float>(s), c, s);
    stage((n_fft >> 5) + (col & 3) * n16);
  } else if (radix == 8 && (col & 1)) {  // mean over W_8^j, j < 4
    const double c = tw64[2 * (n_fft >> 3)], s = tw64[2 * (n_fft >> 3) + 1];
    g.half(static_cast<float>(c), static_cast<float>(s), c, s);
  } else if (radix == 16) {  // mean over W_16^{j q}, j < 4
    double mx = 0.0, my = 0.0;
    for (int32_t j = 0; j < 4; ++j) {
      const int32_t i = (j * (col & 3) * n16) & mask;
      const double c = tw64[2 * i], s = tw64[2 * i + 1];
      const float wr = static_cast<float>(c), wi = static_cast<float>(s);
      mx += 0.25 * (wr * c + wi * s);
      my += 0.25 * (wi * c - wr * s);
    }
    g.times(mx, my);
  }
  // the wave's 1024 points: column q, then bins (kc, kd) of it
  int32_t q, kc;
  if (len > 2 * SUB) {
    const int32_t kb = k / classes, ka = kb & 15;
    progression(64 * step * cls, ka);
    q = cls + classes * ka;
    kc = (kb >> 4) & 15;
  } else if (len > SUB) {
    q = cls + 2 * col;
    kc = (k >> 5) & 15;
  } else {
    q = col;
    kc = (k / radix) & 15;
  }
  progression(4 * step * q, kc);
  const int32_t e = step * q + (n_fft >> 6) * kc;
  if (len > 2 * SUB) {  // T^2 is formed from the rounded T
    const double c = tw64[2 * (e & mask)], s = tw64[2 * (e & mask) + 1];
    const float x = static_cast<float>(c), y = static_cast<float>(s);
    half(e);
    g.half(fmaf(x, x, -y * y), 2.f * x * y, tw64[2 * ((2 * e) & mask)], tw64[2 * ((2 * e) & mask) + 1]);
  } else {
    stage(e);
  }
  return 1.0 / (g.x * g.x + g.y * g.y);
}

}  // namespace ispl
