// Building blocks of the transform kernels (HIP only; never included by
// host-only translation units): the 16- and 4-point DFTs with folded twiddles,
// one wave's 1024-point transform, sample conversion, the XCD-contiguous block
// numbering.  ispl_kernels.hip describes the transform's layout.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "ispl_internal.h"

namespace ispl {

// Per-wave exchange buffer: 16 rows of 64 complex at a pitch of 65, so that
// the pass-2 reads (16 rows, one column, per 16 lanes) hit 16 different bank
// pairs and the pass-1 writes (one row, 64 columns) are contiguous.
constexpr int XPITCH = 65;
constexpr int XWAVE = 16 * XPITCH;  // float2 of one wave's exchange buffer

// A value the compiler must keep in a VGPR: VALU instructions whose operands
// are all VGPRs (or inline constants) can dual-issue on gfx950, those reading
// an SGPR cannot.
__device__ __forceinline__ float in_vgpr(float x) {
  float r;
  asm volatile("v_mov_b32 %0, %1" : "=v"(r) : "v"(x));
  return r;
}

__device__ __forceinline__ float2 cmul(float2 a, float2 b) {
  return make_float2(fmaf(a.x, b.x, -(a.y * b.y)), fmaf(a.x, b.y, a.y * b.x));
}

__device__ __forceinline__ float2 conj_mul(float2 c, float2 x) {  // conj(c) * x
  return make_float2(fmaf(c.x, x.x, c.y * x.y), fmaf(c.x, x.y, -(c.y * x.x)));
}

// a + w b, two fused multiply-adds per component.
__device__ __forceinline__ float2 cmuladd(float2 a, float2 w, float2 b) {
  return make_float2(fmaf(w.x, b.x, fmaf(-w.y, b.y, a.x)), fmaf(w.x, b.y, fmaf(w.y, b.x, a.y)));
}

// 2 a - s: with s = a + w b this is a - w b at one FMA per component.
__device__ __forceinline__ float2 twice_minus(float2 a, float2 s) {
  return make_float2(fmaf(2.f, a.x, -s.x), fmaf(2.f, a.y, -s.y));
}

// Second layer of a 4-point forward DFT from s02 = x0 + x2, d02 = x0 - x2,
// s13 = x1 + x3, d13 = x1 - x3; outputs in natural order.
__device__ __forceinline__ void dft4_tail(float2 s02, float2 d02, float2 s13, float2 d13,
                                          float2& y0, float2& y1, float2& y2, float2& y3) {
  y0 = make_float2(s02.x + s13.x, s02.y + s13.y);
  y2 = make_float2(s02.x - s13.x, s02.y - s13.y);
  y1 = make_float2(d02.x + d13.y, d02.y - d13.x);  // d02 - i d13
  y3 = make_float2(d02.x - d13.y, d02.y + d13.x);  // d02 + i d13
}

// 4-point forward DFT in place, natural order in and out.
__device__ __forceinline__ void dft4(float2& a0, float2& a1, float2& a2, float2& a3) {
  const float2 s02 = make_float2(a0.x + a2.x, a0.y + a2.y);
  const float2 d02 = make_float2(a0.x - a2.x, a0.y - a2.y);
  const float2 s13 = make_float2(a1.x + a3.x, a1.y + a3.y);
  const float2 d13 = make_float2(a1.x - a3.x, a1.y - a3.y);
  dft4_tail(s02, d02, s13, d13, a0, a1, a2, a3);
}

// DFT4 of (a0, w1 a1, w2 a2, w3 a3): the twiddle products fold into the first
// butterfly layer as multiply-adds (a + w b, then 2 a - (a + w b)).
__device__ __forceinline__ void dft4_w123(float2& a0, float2& a1, float2& a2, float2& a3,
                                          float2 w1, float2 w2, float2 w3) {
  const float2 s02 = cmuladd(a0, w2, a2);
  const float2 d02 = twice_minus(a0, s02);
  const float2 p1 = cmul(a1, w1);
  const float2 s13 = cmuladd(p1, w3, a3);
  const float2 d13 = twice_minus(p1, s13);
  dft4_tail(s02, d02, s13, d13, a0, a1, a2, a3);
}

// DFT4 of (w0 a0, w1 a1, w2 a2, w3 a3).
__device__ __forceinline__ void dft4_w0123(float2& a0, float2& a1, float2& a2, float2& a3,
                                           float2 w0, float2 w1, float2 w2, float2 w3) {
  a0 = cmul(a0, w0);
  dft4_w123(a0, a1, a2, a3, w1, w2, w3);
}

constexpr float kC8 = 0.923879532511286756f;  // cos(pi / 8)
constexpr float kS8 = 0.382683432365089772f;  // sin(pi / 8)
constexpr float kR2 = 0.707106781186547524f;  // cos(pi / 4)

// Constants of the 16-point DFT, held in VGPRs for the whole kernel.
struct Dft16Consts {
  float c8, s8, r2;
};

__device__ __forceinline__ Dft16Consts dft16_consts() {
  return Dft16Consts{in_vgpr(kC8), in_vgpr(kS8), in_vgpr(kR2)};
}

// Second stage of a 16-point DFT (j = j1 + 4 j2, k = k1 + 4 k2): after the
// DFT4s over j2, v[j1 + 4 k1] holds a[j1][k1]; twiddle W_16^{j1 k1} and DFT4
// over j1, then leave X[k] in v[k].  W_16^m = exp(-2 pi i m / 16).
__device__ __forceinline__ void dft16_stage_b(float2 (&v)[16], const Dft16Consts& k) {
  const float2 w1 = make_float2(k.c8, -k.s8), w2 = make_float2(k.r2, -k.r2);
  const float2 w3 = make_float2(k.s8, -k.c8), w9 = make_float2(-k.c8, k.s8);
  const float2 w6 = make_float2(-k.r2, -k.r2);
  dft4(v[0], v[1], v[2], v[3]);                       // k1 = 0: W^0, W^0, W^0, W^0
  dft4_w123(v[4], v[5], v[6], v[7], w1, w2, w3);      // k1 = 1: W^0, W^1, W^2, W^3
  {                                                   // k1 = 2: W^0, W^2, W^4, W^6
    const float2 a0 = v[8], a2 = v[10];
    const float2 s02 = make_float2(a0.x + a2.y, a0.y - a2.x);  // a0 + (-i) a2
    const float2 d02 = make_float2(a0.x - a2.y, a0.y + a2.x);
    const float2 p1 = make_float2(k.r2 * (v[9].x + v[9].y), k.r2 * (v[9].y - v[9].x));
    const float2 s13 = cmuladd(p1, w6, v[11]);
    const float2 d13 = twice_minus(p1, s13);
    dft4_tail(s02, d02, s13, d13, v[8], v[9], v[10], v[11]);
  }
  dft4_w123(v[12], v[13], v[14], v[15], w3, w6, w9);  // k1 = 3: W^0, W^3, W^6, W^9
  // position 4 k1 + k2 holds X[k1 + 4 k2]
  float2 t[16];
#pragma unroll
  for (int i = 0; i < 16; ++i) t[i] = v[4 * (i & 3) + (i >> 2)];
#pragma unroll
  for (int i = 0; i < 16; ++i) v[i] = t[i];
}

// 16-point forward DFT of (w[j] v[j]) with w[0] = 1.
__device__ __forceinline__ void dft16_pre1(float2 (&v)[16], const float2 (&w)[16],
                                           const Dft16Consts& k) {
  dft4_w123(v[0], v[4], v[8], v[12], w[4], w[8], w[12]);
#pragma unroll
  for (int j1 = 1; j1 < 4; ++j1)
    dft4_w0123(v[j1], v[j1 + 4], v[j1 + 8], v[j1 + 12], w[j1], w[j1 + 4], w[j1 + 8], w[j1 + 12]);
  dft16_stage_b(v, k);
}

// 16-point forward DFT of v.
__device__ __forceinline__ void dft16(float2 (&v)[16], const Dft16Consts& k) {
#pragma unroll
  for (int j1 = 0; j1 < 4; ++j1) dft4(v[j1], v[j1 + 4], v[j1 + 8], v[j1 + 12]);
  dft16_stage_b(v, k);
}

// 16-point DFT of v when v[4..15] are zero: the first radix-4 stage then
// only replicates v[j1] (the 4-point DFT of (a, 0, 0, 0) is (a, a, a, a)).
__device__ __forceinline__ void dft16_first4(float2 (&v)[16], const Dft16Consts& k) {
#pragma unroll
  for (int j1 = 0; j1 < 4; ++j1) v[j1 + 4] = v[j1 + 8] = v[j1 + 12] = v[j1];
  dft16_stage_b(v, k);
}

// 16-point forward DFT of (w[j] v[j]).
__device__ __forceinline__ void dft16_pre(float2 (&v)[16], const float2 (&w)[16],
                                          const Dft16Consts& k) {
#pragma unroll
  for (int j1 = 0; j1 < 4; ++j1)
    dft4_w0123(v[j1], v[j1 + 4], v[j1 + 8], v[j1 + 12], w[j1], w[j1 + 4], w[j1 + 8], w[j1 + 12]);
  dft16_stage_b(v, k);
}

// Orders this wave's LDS accesses around a cross-lane exchange.  LDS requests
// of one wave are served in issue order, so only the compiler needs fencing.
__device__ __forceinline__ void wave_lds_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// 4 x 4 transpose between the four 16-lane rows of a wave and four registers
// (v_permlane16_swap / v_permlane32_swap): on entry register g of row r holds
// M[r][g], on exit register r of row g does.
__device__ __forceinline__ void row_transpose4(float (&m)[4]) {
  const auto s01 = __builtin_amdgcn_permlane16_swap(__float_as_uint(m[0]), __float_as_uint(m[1]),
                                                    false, false);
  const auto s23 = __builtin_amdgcn_permlane16_swap(__float_as_uint(m[2]), __float_as_uint(m[3]),
                                                    false, false);
  const auto s02 = __builtin_amdgcn_permlane32_swap(s01[0], s23[0], false, false);
  const auto s13 = __builtin_amdgcn_permlane32_swap(s01[1], s23[1], false, false);
  m[0] = __uint_as_float(s02[0]);
  m[1] = __uint_as_float(s13[0]);
  m[2] = __uint_as_float(s02[1]);
  m[3] = __uint_as_float(s13[1]);
}

template <int ST>
struct SampleIO;

// The same global-memory pointer, read from the first active lane: for
// values that are uniform over the workgroup, so that they stay in scalar
// registers and loads through them take a scalar base and a 32-bit lane offset.
// Element types are read as builtin types (complex64 as a 2-vector), since
// the class types cannot be loaded through an address-space pointer.
typedef float f32x2 __attribute__((ext_vector_type(2)));
template <typename T>
struct Builtin {
  using type = T;
};
template <>
struct Builtin<float2> {
  using type = f32x2;
};
template <typename T>
using gptr = const __attribute__((address_space(1))) typename Builtin<T>::type*;
template <typename T>
__device__ __forceinline__ gptr<T> uniform_ptr(const T* p) {
  const uint64_t v = reinterpret_cast<uint64_t>(p);
  const uint32_t lo = __builtin_amdgcn_readfirstlane(static_cast<uint32_t>(v));
  const uint32_t hi = __builtin_amdgcn_readfirstlane(static_cast<uint32_t>(v >> 32));
  return reinterpret_cast<gptr<T>>((static_cast<uint64_t>(hi) << 32) | lo);
}
__device__ __forceinline__ uint32_t from_builtin(uint32_t v) { return v; }
__device__ __forceinline__ float2 from_builtin(f32x2 v) { return make_float2(v.x, v.y); }

template <>
struct SampleIO<0> {  // complex64
  using raw_t = float2;
  __device__ static raw_t load(const void* base, int64_t i) {
    return reinterpret_cast<const float2*>(base)[i];
  }
  __device__ static raw_t zero() { return make_float2(0.f, 0.f); }
  __device__ static float2 cvt(raw_t r) { return r; }
};

template <>
struct SampleIO<1> {  // int16 (re, im) pairs; int16 -> float is exact
  using raw_t = uint32_t;
  __device__ static raw_t load(const void* base, int64_t i) {
    return reinterpret_cast<const uint32_t*>(base)[i];
  }
  __device__ static raw_t zero() { return 0u; }
  __device__ static float2 cvt(raw_t r) {
    return make_float2(static_cast<float>(static_cast<int16_t>(r & 0xffffu)),
                       static_cast<float>(static_cast<int32_t>(r) >> 16));
  }
};

// DFT4 of (a0, T a1, T^2 a2, T^3 a3), twiddles in geometric progression: with
// t02 = a0 + T^2 a2 and t13 = a1 + T^2 a3 the outputs are t02 +- T t13 and
// (a0 - T^2 a2) -+ i T (a1 - T^2 a3), so only T and T^2 are needed and every
// product folds into a multiply-add (24 operations, as for three free twiddles).
__device__ __forceinline__ void dft4_geo(float2& a0, float2& a1, float2& a2, float2& a3, float2 t,
                                         float2 t2) {
  const float2 t02 = cmuladd(a0, t2, a2);
  const float2 d02 = twice_minus(a0, t02);
  const float2 t13 = cmuladd(a1, t2, a3);
  const float2 u13 = twice_minus(a1, t13);
  a0 = cmuladd(t02, t, t13);
  a2 = twice_minus(t02, a0);
  a1 = cmuladd(d02, make_float2(t.y, -t.x), u13);  // -i T
  a3 = twice_minus(d02, a1);
}

// Twiddles of a 16-point DFT whose inputs carry the factors P^j (j < 16):
// with j = j1 + 4 j2 the first stage is a DFT4 over j2 with ratio G = P^4, the
// second a DFT4 over j1 with ratio H_k1 = P W_16^{k1}; each as (ratio, ratio^2).
struct GeoTwiddles {
  float2 g, g2;
  float2 h[4], h2[4];
};

// sum_j v[j] P^j W_16^{j k} into v[k], for the progression of `w`.
__device__ __forceinline__ void dft16_geo(float2 (&v)[16], const GeoTwiddles& w) {
#pragma unroll
  for (int j1 = 0; j1 < 4; ++j1) dft4_geo(v[j1], v[j1 + 4], v[j1 + 8], v[j1 + 12], w.g, w.g2);
  // v[j1 + 4 k1] holds the first-stage output k1 of group j1
#pragma unroll
  for (int k1 = 0; k1 < 4; ++k1)
    dft4_geo(v[4 * k1], v[4 * k1 + 1], v[4 * k1 + 2], v[4 * k1 + 3], w.h[k1], w.h2[k1]);
  // position 4 k1 + k2 holds X[k1 + 4 k2]
  float2 t[16];
#pragma unroll
  for (int i = 0; i < 16; ++i) t[i] = v[4 * (i & 3) + (i >> 2)];
#pragma unroll
  for (int i = 0; i < 16; ++i) v[i] = t[i];
}

// GeoTwiddles of the progression P = W_N^e (all from the table, so every
// factor is correctly rounded): G = W_N^{4 e}, H_k1 = W_N^{e + k1 N / 16}.
__device__ __forceinline__ void load_geo(GeoTwiddles& w, const float2* __restrict__ tw, int n_fft,
                                         int e) {
  const int nmask = n_fft - 1, n16 = n_fft >> 4;
  w.g = tw[(4 * e) & nmask];
  w.g2 = tw[(8 * e) & nmask];
#pragma unroll
  for (int k1 = 0; k1 < 4; ++k1) {
    w.h[k1] = tw[(e + k1 * n16) & nmask];
    w.h2[k1] = tw[(2 * e + 2 * k1 * n16) & nmask];
  }
}

// Twiddles of one wave's 1024-point transform of bin class kappa: the wave
// produces bins kappa + S kb (S = N / 1024, kb < 1024) of the N-point
// spectrum, so its input carries the factor W_N^{kappa n} on top of the
// 1024-point DFT kernel W_N^{S kb n}.  Fixed over the pulse loop.
struct WaveTwiddles {
  float2 pre[16];    // pass 1: W_N^{64 kappa j}, the same for every lane
  float2 tw2[16];    // pass 2: W_N^{l (kappa + S ka)} for the pass-1 lane l = row + 4 m
  float2 tw3[4][3];  // pass 3: W_64^{r kc}, r = 1..3, kc = 4 row + t
};

__device__ __forceinline__ void load_wave_twiddles(WaveTwiddles& w, const float2* __restrict__ tw,
                                                   int n_fft, int kappa, int lane) {
  const int nmask = n_fft - 1, S = n_fft >> 10;
  const int ka = lane & 15, row = lane >> 4;
#pragma unroll
  for (int j = 0; j < 16; ++j) {
    w.pre[j] = tw[(64 * kappa * j) & nmask];
    w.tw2[j] = tw[((row + 4 * j) * (kappa + S * ka)) & nmask];
  }
#pragma unroll
  for (int t = 0; t < 4; ++t)
#pragma unroll
    for (int r = 1; r < 4; ++r) w.tw3[t][r - 1] = tw[((n_fft >> 6) * r * (4 * row + t)) & nmask];
}

// The same transform with passes 2 and 3 in geometric form (36 instead of 56
// registers of per-lane twiddles; the long-code kernels need the room).  With
// q = kappa + S ka, lane (ka, r) weighs u_ka[r + 4 m] in pass 2 by
// W_N^{(r + 4 m) q} = W_N^{r q} (W_N^{4 q})^m: a progression of ratio W_N^{4 q},
// whose common factor W_N^{r q} moves into pass 3, where the 4-point DFT over r
// then weighs term r by (W_N^{q} W_64^{kc})^r = T_kc^r, T_kc = W_N^{q + 16 S kc},
// kc = 4 row + t.
struct WaveTwiddlesGeo {
  float2 pre[16];            // pass 1, as above
  GeoTwiddles p2;            // pass 2: progression W_N^{4 q}
  float2 t3[4], t3sq[4];     // pass 3: T_kc and T_kc^2
};

__device__ __forceinline__ void load_wave_twiddles(WaveTwiddlesGeo& w,
                                                   const float2* __restrict__ tw, int n_fft,
                                                   int kappa, int lane) {
  const int nmask = n_fft - 1, S = n_fft >> 10;
  const int ka = lane & 15, row = lane >> 4;
  const int q = kappa + S * ka;
#pragma unroll
  for (int j = 0; j < 16; ++j) w.pre[j] = tw[(64 * kappa * j) & nmask];
  load_geo(w.p2, tw, n_fft, 4 * q);
#pragma unroll
  for (int t = 0; t < 4; ++t) {
    const int e = q + 16 * S * (4 * row + t);
    w.t3[t] = tw[e & nmask];
    w.t3sq[t] = tw[(2 * e) & nmask];
  }
}

// Twiddles of passes 2 and 3 alone (pass 1 has constant factors or its own).
struct GridTwiddles {
  GeoTwiddles p2;
  float2 t3[4], t3sq[4];
};
// The same, with pass 3's row exchange through LDS.
struct GridTwiddlesRows : GridTwiddles {};
// The same with T_kc^2 formed for each transform (8 registers less).
struct GridTwiddlesRows1 {
  GeoTwiddles p2;
  float2 t3[4];
};
// The same with pass 3's factors in LDS too: t3[64 t] = (T_kc, T_kc^2) of this
// lane (16 registers less, for kernels that keep the next pulse's samples in flight).
struct GridTwiddlesLds {
  GeoTwiddles p2;
  const float4* t3;
};
// Pass 2's factors of one lane's column in LDS: p2[0] = (G, G^2), p2[16 (1 + k1)] =
// (H_k1, H_k1^2); 20 registers less, for kernels whose sums take 32.
struct GeoLds {
  const float4* p;
};
__device__ __forceinline__ void dft16_geo(float2 (&v)[16], const GeoLds& w) {
  {
    const float4 g = w.p[0];
#pragma unroll
    for (int j1 = 0; j1 < 4; ++j1)
      dft4_geo(v[j1], v[j1 + 4], v[j1 + 8], v[j1 + 12], make_float2(g.x, g.y), make_float2(g.z, g.w));
  }
#pragma unroll
  for (int k1 = 0; k1 < 4; ++k1) {
    const float4 h = w.p[16 * (1 + k1)];
    dft4_geo(v[4 * k1], v[4 * k1 + 1], v[4 * k1 + 2], v[4 * k1 + 3], make_float2(h.x, h.y),
             make_float2(h.z, h.w));
  }
  float2 t[16];
#pragma unroll
  for (int i = 0; i < 16; ++i) t[i] = v[4 * (i & 3) + (i >> 2)];
#pragma unroll
  for (int i = 0; i < 16; ++i) v[i] = t[i];
}
// Part t < 5 of the progression P = W_N^e as GeoLds reads it.
__device__ __forceinline__ float4 geo_part(const float2* __restrict__ tw, int n_fft, int e, int t) {
  const int nmask = n_fft - 1, i = t == 0 ? 4 * e : e + (t - 1) * (n_fft >> 4);
  const float2 u = tw[i & nmask], u2 = tw[(2 * i) & nmask];
  return make_float4(u.x, u.y, u2.x, u2.y);
}
// Both in LDS.
struct GridTwiddlesLds2 {
  GeoLds p2;
  const float4* t3;
};
// Pass 2's in LDS, pass 3's T_kc in registers and squared for each transform.
struct GridTwiddlesRows2 {
  GeoLds p2;
  float2 t3[4];
};

template <typename TW>
inline constexpr bool kGeo = false;
template <>
inline constexpr bool kGeo<WaveTwiddlesGeo> = true;
template <>
inline constexpr bool kGeo<GridTwiddles> = true;
template <>
inline constexpr bool kGeo<GridTwiddlesLds> = true;
template <>
inline constexpr bool kGeo<GridTwiddlesRows> = true;
template <>
inline constexpr bool kGeo<GridTwiddlesRows1> = true;
template <>
inline constexpr bool kGeo<GridTwiddlesLds2> = true;
template <>
inline constexpr bool kGeo<GridTwiddlesRows2> = true;
template <typename TW>
inline constexpr bool kLds3 = false;
template <>
inline constexpr bool kLds3<GridTwiddlesLds> = true;
template <>
inline constexpr bool kLds3<GridTwiddlesLds2> = true;
template <typename TW>
inline constexpr bool kRowsLds = kLds3<TW>;
template <>
inline constexpr bool kRowsLds<GridTwiddlesRows> = true;
template <>
inline constexpr bool kRowsLds<GridTwiddlesRows1> = true;
template <>
inline constexpr bool kRowsLds<GridTwiddlesRows2> = true;
template <typename TW>
inline constexpr bool kSquare3 = false;
template <>
inline constexpr bool kSquare3<GridTwiddlesRows1> = true;
template <>
inline constexpr bool kSquare3<GridTwiddlesRows2> = true;

// One wave's 1024-point transform and power accumulation.  On entry lane l
// holds f[l + 64 j] in v[j]; xw is the wave's exchange buffer.  On exit
// acc[4 t + kd] += |F[kb]|^2 for kb = ka + 16 (4 row + t) + 256 kd, with
// ka = lane & 15, row = lane >> 4 (F including the bin-class factors).
// K0: the wave's bin class is 0 (N = 1024), so the pass-1 factors are all 1.
// F4 (with K0): only v[0..3] carry samples (L <= 256); v[4..15] are not read.
struct NoHook {
  __device__ void operator()() const {}
};

// Passes 2 and 3 of one wave: on entry the pass-1 outputs lie in v (row k of
// the exchange in v[k]); sink(i, F) receives the bin of register i = 4 t + kd.
// `after_exchange` runs right after this wave has issued the reads of its
// pass-2 inputs: from then until the next call the exchange buffer is free.
template <typename TW, typename Hook, typename Sink>
__device__ __forceinline__ void wave_passes_23(float2 (&v)[16], float2* xw, const TW& w,
                                               const Dft16Consts& dk, int lane,
                                               Hook after_exchange, Sink sink) {
  const int ka = lane & 15, row = lane >> 4;
#pragma unroll
  for (int k = 0; k < 16; ++k) xw[k * XPITCH + lane] = v[k];
  wave_lds_sync();

  // pass 2: lane (ka, r) twiddles u_ka[r + 4 m] and transforms over m, giving
  // the partial bins v_{ka,r}[kc]
  const int p2base = ka * XPITCH + row;
#pragma unroll
  for (int m = 0; m < 16; ++m) v[m] = xw[p2base + 4 * m];
  after_exchange();
  if constexpr (kGeo<TW>)
    dft16_geo(v, w.p2);
  else
    dft16_pre(v, w.tw2, dk);

  // pass 3: the 4-point DFT over r runs across the four 16-lane rows.  For
  // each t a row transpose hands row g the four values v_{ka,r}[4 g + t],
  // r = 0..3; then twiddle W_64^{r kc}, DFT over r.
  if constexpr (kRowsLds<TW>) {
    // rows exchange through LDS: a v_permlane swap holds the VALU for 8 cycles
#pragma unroll
    for (int k = 0; k < 16; ++k) xw[64 * k + lane] = v[k];
    wave_lds_sync();
#pragma unroll
    for (int t = 0; t < 4; ++t)
#pragma unroll
      for (int r = 0; r < 4; ++r) v[4 * t + r] = xw[64 * (4 * row + t) + 16 * r + ka];
  }
#pragma unroll
  for (int t = 0; t < 4; ++t) {
    float2 c0, c1, c2, c3;
    if constexpr (kRowsLds<TW>) {
      c0 = v[4 * t], c1 = v[4 * t + 1], c2 = v[4 * t + 2], c3 = v[4 * t + 3];
    } else {
      float re[4] = {v[t].x, v[4 + t].x, v[8 + t].x, v[12 + t].x};
      float im[4] = {v[t].y, v[4 + t].y, v[8 + t].y, v[12 + t].y};
      row_transpose4(re);
      row_transpose4(im);
      c0 = make_float2(re[0], im[0]), c1 = make_float2(re[1], im[1]);
      c2 = make_float2(re[2], im[2]), c3 = make_float2(re[3], im[3]);
    }
    if constexpr (kLds3<TW>) {
      const float4 q = w.t3[64 * t];
      dft4_geo(c0, c1, c2, c3, make_float2(q.x, q.y), make_float2(q.z, q.w));
    } else if constexpr (kSquare3<TW>) {
      float2 u = w.t3[t];
      asm volatile("" : "+v"(u.x), "+v"(u.y));  // (or the squares would be kept across pulses)
      dft4_geo(c0, c1, c2, c3, u, make_float2(fmaf(u.x, u.x, -u.y * u.y), 2.f * u.x * u.y));
    } else if constexpr (kGeo<TW>) {
      dft4_geo(c0, c1, c2, c3, w.t3[t], w.t3sq[t]);
    } else {
      dft4_w123(c0, c1, c2, c3, w.tw3[t][0], w.tw3[t][1], w.tw3[t][2]);
    }
    sink(4 * t + 0, c0);
    sink(4 * t + 1, c1);
    sink(4 * t + 2, c2);
    sink(4 * t + 3, c3);
  }
}

// The running power sums of a wave's 16 bins per lane.
struct PowerSink {
  float (&acc)[16];
  __device__ __forceinline__ void operator()(int i, float2 c) const {
    acc[i] = fmaf(c.y, c.y, fmaf(c.x, c.x, acc[i]));
  }
};

// The same in double: squares and sums of FP32 bins lose nothing to rounding or to the
// range of FP32.
struct PowerSink64 {
  double (&acc)[16];
  __device__ __forceinline__ void operator()(int i, float2 c) const {
    const double x = c.x, y = c.y;
    acc[i] = fma(y, y, fma(x, x, acc[i]));
  }
};

template <bool K0 = false, bool F4 = false, typename TW = WaveTwiddles, typename Hook = NoHook>
__device__ __forceinline__ void wave_fft_accumulate(float2 (&v)[16], float2* xw, const TW& w,
                                                    const Dft16Consts& dk, float (&acc)[16],
                                                    int lane, Hook after_exchange = Hook{}) {
  // pass 1: pre-twiddle and 16-point DFT over the stride-64 samples of a lane
  static_assert(!F4 || K0, "four non-zero inputs only in bin class 0");
  if constexpr (F4)
    dft16_first4(v, dk);
  else if constexpr (K0)
    dft16(v, dk);
  else
    dft16_pre1(v, w.pre, dk);
  wave_passes_23(v, xw, w, dk, lane, after_exchange, PowerSink{acc});
}

// Workgroups are dealt to the 8 XCDs round-robin; renumber them so that each
// XCD runs a contiguous range of (gate, bin group, chunk) work items and
// neighbouring gates, whose windows overlap, share that XCD's L2.
__device__ __forceinline__ int xcd_block_id() {
  const int nblk = gridDim.x;
  const int xcd = blockIdx.x & 7, slot = blockIdx.x >> 3;
  const int per = nblk >> 3, extra = nblk & 7;
  return xcd < extra ? xcd * (per + 1) + slot : extra * (per + 1) + (xcd - extra) * per + slot;
}

}  // namespace ispl
