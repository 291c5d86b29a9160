// Folded integration (gfx950): the spectrum of a code of L samples through a
// transform of M >= 2 L - 1 points instead of N.
//
// |X(f)|^2 of a row of L samples is a trigonometric polynomial of degree
// L - 1 (its coefficients are the row's autocorrelation), and so is its sum over pulses:
// S at any M >= 2 L - 1 equispaced frequencies determines S everywhere.  So
// the pulse loop (Section 3.2: decode, transform, |X|^2, sum) runs on the grid
// of M = 2^m >= 2 L - 1 points, and once per gate the summed grid is taken to
// the N bins: an inverse DFT gives the lags r[n], |n| < L, and
//
//   S[k] = r[0] + 2 Re sum_{0 < n < L} r[n] W_N^{k n}.
//
// At L = 1000, N = 16384 the pulse loop has 2 instead of 16 transforms of 1024
// points per pulse and gate: 1000 pulses x 1000 gates (int16 samples) take 1.72 instead of
// 11.45 ms.  The grid's mean is taken out before the inverse transform and r[0]
// added back last, so rounding in the two transforms is relative to the
// spectrum's fluctuation about its mean, not to the mean; the sums of a gate's
// pulses are split over 8 or 16 waves, which halves their rounding (relative error against
// FP64 1.8e-7 there, 6.1e-7 before).

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>

#include "ispl_fft.h"
#include "ispl_internal.h"

namespace ispl {
namespace {

typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

// ---------------------------------------------------------------------------
// Grid pass, L <= 1024.
//
// One wave transforms 1024 values at a time: Q = 1024 / M pulses of M points
// (M <= 1024), or one of the two bin classes k mod 2 of one pulse (M = 2048).
// With M = 64 J, a lane holds samples l + 64 j, j < J, of each of its pulses:
//   pass 1  J-point DFTs over j; L <= M / 2, so half of the inputs are zero;
//   pass 2  lane (t, k1, r), t < Q, k1 < J: 16-point DFT over m of
//           u_{t,k1}[r + 4 m] W_M^{(r + 4 m) k1};
//   pass 3  4-point DFT over r: bins k1 + J (kc + 16 kd).
// Passes 2 and 3 are those of one 1024-point transform with k1 in the place of
// its ka, in geometric twiddle form.  Waves share nothing during the pulse loop (no
// barrier): each takes its own run of pulses, and the workgroup's sums meet in
// LDS at the end.
//
// What bounds it is VALU issue (M = 2048: 580 VALU instructions per wave and
// pulse at 0.30 per SIMD and cycle).  Register-only probes at four waves per
// SIMD: two-operand (4-byte) instructions issue at 0.43 per cycle, three-operand
// ones (8 bytes) at 0.34, and conversions, shifts and anything reading a scalar
// register at 0.22, a v_permlane swap at 0.12.  Hence pass 3's exchange between
// lane rows goes through LDS (12 % fewer cycles than with swaps), the code
// bits are brought up by additions, and pass 3's twiddles lie in LDS, which keeps
// four waves per SIMD with the next pulse's samples in flight.

// Samples through a buffer descriptor: reads past the end of the code return
// zero, so the row is zero-padded by the load itself.
__device__ __forceinline__ auto row_desc(const void* base, int64_t elem, int size, int elems) {
  const uint64_t v = reinterpret_cast<uint64_t>(base) + static_cast<uint64_t>(elem) * size;
  const uint32_t lo = __builtin_amdgcn_readfirstlane(static_cast<uint32_t>(v));
  const uint32_t hi = __builtin_amdgcn_readfirstlane(static_cast<uint32_t>(v >> 32));
  return __builtin_amdgcn_make_buffer_rsrc(
      reinterpret_cast<void*>((static_cast<uint64_t>(hi) << 32) | lo), 0,
      __builtin_amdgcn_readfirstlane(elems * size), 0x00020000);
}

template <int ST>
struct BufferSample;
template <>
struct BufferSample<0> {
  using raw_t = u32x2;
  static constexpr int SIZE = 8;
  template <typename D>
  __device__ static raw_t load(D d, int byte) {
    return __builtin_amdgcn_raw_buffer_load_b64(d, byte, 0, 0);
  }
  __device__ static float2 cvt(raw_t r) {
    return make_float2(__uint_as_float(r.x), __uint_as_float(r.y));
  }
};
template <>
struct BufferSample<1> {
  using raw_t = uint32_t;
  static constexpr int SIZE = 4;
  template <typename D>
  __device__ static raw_t load(D d, int byte) {
    return __builtin_amdgcn_raw_buffer_load_b32(d, byte, 0, 0);
  }
  __device__ static float2 cvt(raw_t r) { return SampleIO<1>::cvt(r); }
};

// 8-point DFT of (v0, v1, v2, v3, 0, 0, 0, 0): even outputs are the 4-point
// DFT of v, odd ones that of v_j W_8^j.
__device__ __forceinline__ void dft8_first4(float2* v, const Dft16Consts& k) {
  float2 e0 = v[0], e1 = v[1], e2 = v[2], e3 = v[3];
  float2 o0 = v[0];
  float2 o1 = make_float2(k.r2 * (v[1].x + v[1].y), k.r2 * (v[1].y - v[1].x));   // W_8
  float2 o2 = make_float2(v[2].y, -v[2].x);                                      // -i
  float2 o3 = make_float2(k.r2 * (v[3].y - v[3].x), -k.r2 * (v[3].x + v[3].y));  // W_8^3
  dft4(e0, e1, e2, e3);
  dft4(o0, o1, o2, o3);
  v[0] = e0, v[1] = o0, v[2] = e1, v[3] = o1, v[4] = e2, v[5] = o2, v[6] = e3, v[7] = o3;
}

// 16-point DFT of v when v[8..15] are zero.
__device__ __forceinline__ void dft16_first8(float2 (&v)[16], const Dft16Consts& k) {
#pragma unroll
  for (int j = 0; j < 4; ++j) {  // 4-point DFT of (a, b, 0, 0)
    const float2 a = v[j], b = v[j + 4];
    v[j] = make_float2(a.x + b.x, a.y + b.y);
    v[j + 4] = make_float2(a.x + b.y, a.y - b.x);
    v[j + 8] = make_float2(a.x - b.x, a.y - b.y);
    v[j + 12] = make_float2(a.x - b.y, a.y + b.x);
  }
  dft16_stage_b(v, k);
}

// Pass 1 of Q transforms side by side, transform t in v[t J .. t J + J - 1],
// its first J / 2 inputs set.
template <int Q>
__device__ __forceinline__ void grid_pass1(float2 (&v)[16], const Dft16Consts& k) {
  if constexpr (Q == 1) {
    dft16_first8(v, k);
  } else if constexpr (Q == 2) {
    dft8_first4(v, k);
    dft8_first4(v + 8, k);
  } else if constexpr (Q == 4) {
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      const float2 a = v[4 * t], b = v[4 * t + 1];
      v[4 * t] = make_float2(a.x + b.x, a.y + b.y);
      v[4 * t + 1] = make_float2(a.x + b.y, a.y - b.x);
      v[4 * t + 2] = make_float2(a.x - b.x, a.y - b.y);
      v[4 * t + 3] = make_float2(a.x - b.y, a.y + b.x);
    }
  } else {
#pragma unroll
    for (int t = 0; t < 8; ++t) v[2 * t + 1] = v[2 * t];
  }
}

// 16-point DFT of v[j] W_32^j (bin class 1 of 2048 points), in geometric form with
// constant ratios: W_8 and W_4 in the first stage, W_32 W_16^{k1} in the second.
__device__ __forceinline__ void dft16_w32(float2 (&v)[16], const Dft16Consts& k) {
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const float2 a0 = v[j], a1 = v[j + 4], a2 = v[j + 8], a3 = v[j + 12];
    const float2 t02 = make_float2(a0.x + a2.y, a0.y - a2.x);  // a0 - i a2
    const float2 d02 = make_float2(a0.x - a2.y, a0.y + a2.x);
    const float2 t13 = make_float2(a1.x + a3.y, a1.y - a3.x);
    const float2 u13 = make_float2(a1.x - a3.y, a1.y + a3.x);
    // T = W_8 = r2 (1 - i), -i T = r2 (-1 - i)
    v[j] = make_float2(fmaf(k.r2, t13.x + t13.y, t02.x), fmaf(k.r2, t13.y - t13.x, t02.y));
    v[j + 8] = twice_minus(t02, v[j]);
    v[j + 4] = make_float2(fmaf(k.r2, u13.y - u13.x, d02.x), fmaf(-k.r2, u13.x + u13.y, d02.y));
    v[j + 12] = twice_minus(d02, v[j + 4]);
  }
  // W_32^{1 + 2 k1}: cos, sin of (1 + 2 k1) pi / 16; squares W_16^{1 + 2 k1}
  constexpr float c1 = 0.980785280403230449f, s1 = 0.195090322016128268f;
  constexpr float c3 = 0.831469612302545237f, s3 = 0.555570233019602225f;
  dft4_geo(v[0], v[1], v[2], v[3], make_float2(c1, -s1), make_float2(k.c8, -k.s8));
  dft4_geo(v[4], v[5], v[6], v[7], make_float2(c3, -s3), make_float2(k.s8, -k.c8));
  dft4_geo(v[8], v[9], v[10], v[11], make_float2(s3, -c3), make_float2(-k.s8, -k.c8));
  dft4_geo(v[12], v[13], v[14], v[15], make_float2(s1, -c1), make_float2(-k.c8, -k.s8));
  float2 t[16];
#pragma unroll
  for (int i = 0; i < 16; ++i) t[i] = v[4 * (i & 3) + (i >> 2)];
#pragma unroll
  for (int i = 0; i < 16; ++i) v[i] = t[i];
}

// Code rows as sign bits: word lane of a row holds in bit 31 - j whether code
// sample lane + 64 j is -1; binary[row] tells whether the whole row is
// +-1 + 0i.  One wave per row, all its loads in flight at once.
__global__ void __launch_bounds__(256)
pack_grid_bits(const float2* __restrict__ tx, int32_t rows, int32_t code_len,
               uint32_t* __restrict__ bits, int32_t* __restrict__ binary) {
  const int row = 4 * static_cast<int>(blockIdx.x) + static_cast<int>(threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  if (row >= rows) return;  // whole waves
  const auto d = row_desc(tx, static_cast<int64_t>(row) * code_len, 8, code_len);
  u32x2 c[16];
#pragma unroll
  for (int j = 0; j < 16; ++j)
    c[j] = __builtin_amdgcn_raw_buffer_load_b64(d, (lane + 64 * j) * 8, 0, 0);
  uint32_t word = 0;
  bool ok = true;
#pragma unroll
  for (int j = 0; j < 16; ++j) {
    const float x = __uint_as_float(c[j].x), y = __uint_as_float(c[j].y);
    ok = ok && (lane + 64 * j >= code_len || ((x == 1.f || x == -1.f) && y == 0.f));
    word |= (x < 0.f ? 1u : 0u) << (31 - j);
  }
  bits[64 * row + lane] = word;
  const bool all = __all(ok);
  if (lane == 0) binary[row] = all ? 1 : 0;
}

// LOGM: log2 of the grid; W: waves per workgroup.  The workgroup's waves take
// W runs of pulses (LOGM = 11: W / 2 runs, each by one wave per bin class); with
// C chunks the run count is C times that.
template <int LOGM, int ST, int W>
__global__ void __launch_bounds__(64 * W, 4) grid_spectra(FoldArgs a) {
  constexpr int M = 1 << LOGM;
  constexpr int CLS = M > SUB ? M / SUB : 1;    // bin classes
  constexpr int Q = M < SUB ? SUB / M : 1;      // pulses per step
  constexpr int J = CLS > 1 ? 16 : M / 64;      // pass-1 points per pulse
  constexpr int JL = CLS > 1 ? 16 : J / 2;      // of which loaded
  constexpr int RUNS = W / CLS;
  // samples per pulse fetched a step ahead (all that four waves per SIMD have registers for)
  constexpr int JP = CLS > 1 ? (ST == 0 ? 6 : 10) : JL;
  static_assert(CLS <= 2 && W % CLS == 0, "at most two bin classes");
  using IO = BufferSample<ST>;
  __shared__ float2 xs[W * XWAVE];
  __shared__ float4 t3s[CLS][4][64];  // pass-3 twiddles of each class

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int cls = CLS > 1 ? wave & 1 : 0;
  const int run = wave / CLS;
  const int bid = a.gate_list ? static_cast<int>(blockIdx.x) : xcd_block_id();
  const int c = bid % a.chunks, slot = bid / a.chunks;
  int g = a.slot0 + slot;
  if (a.gate_list) {
    if (g >= *a.gate_count) return;  // uniform, before any barrier
    g = a.gate_list[g];
    if (g < 0 || g >= a.n_gates) return;
  }
  const int L = a.code_len;
  const float2* __restrict__ tw = reinterpret_cast<const float2*>(a.twiddle);
  // pass-2 column k1 of this lane (bins k1 + (M / 64) (kc + 16 kd)) and its
  // progressions W_M^{4 k1 m} (pass 2) and (W_M^{k1} W_64^{kc})^r (pass 3)
  GridTwiddlesLds wt;
  {
    const int step = a.n_fft >> LOGM, k1 = CLS > 1 ? cls + CLS * (lane & 15) : lane & (J - 1);
    load_geo(wt.p2, tw, a.n_fft, 4 * step * k1);
    if (wave < CLS) {
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        const int e = step * k1 + (a.n_fft >> 6) * (4 * (lane >> 4) + t);
        const float2 u = tw[e & (a.n_fft - 1)], u2 = tw[(2 * e) & (a.n_fft - 1)];
        t3s[wave][t][lane] = make_float4(u.x, u.y, u2.x, u2.y);
      }
    }
    wt.t3 = &t3s[cls][0][lane];
    __syncthreads();
  }
  const Dft16Consts dk = dft16_consts();
  float acc[16];
#pragma unroll
  for (int i = 0; i < 16; ++i) acc[i] = 0.f;

  const int64_t gate_off = static_cast<int64_t>(a.first_gate) + static_cast<int64_t>(g) * a.gate_step;
  const int steps = (a.n_pulses + Q - 1) / Q;
  const int64_t s = static_cast<int64_t>(c) * RUNS + run, all = static_cast<int64_t>(a.chunks) * RUNS;
  const int i0 = static_cast<int>(s * steps / all), i1 = static_cast<int>((s + 1) * steps / all);
  float2* xw = xs + wave * XWAVE;

  typename IO::raw_t raw[Q * JL];
  uint32_t bits[Q];
  // samples j0 <= j < j1 of each pulse of step i (zero past the last pulse)
  auto fetch = [&](int i, int j0, int j1) {
#pragma unroll
    for (int t = 0; t < Q; ++t) {
      const int p = i * Q + t;
      const auto d = row_desc(a.samples, static_cast<int64_t>(p) * a.stride + gate_off, IO::SIZE,
                              p < a.n_pulses && i < i1 ? L : 0);
#pragma unroll
      for (int j = 0; j < JL; ++j)
        if (j >= j0 && j < j1) raw[t * JL + j] = IO::load(d, (lane + 64 * j) * IO::SIZE);
    }
  };
  auto fetch_bits = [&](int i) {
#pragma unroll
    for (int t = 0; t < Q; ++t) {
      const int p = min(i * Q + t, a.n_pulses - 1);
      bits[t] = a.code_bits[(a.tx_per_pulse ? 64 * p : 0) + lane];
    }
  };
  auto transform = [&](float2 (&v)[16]) {
    if constexpr (CLS == 1)
      grid_pass1<Q>(v, dk);
    else if (cls == 0)
      dft16(v, dk);
    else
      dft16_w32(v, dk);
    wave_passes_23(v, xw, wt, dk, lane, NoHook{}, PowerSink{acc});
  };

  // codes of this wave's pulses all +-1: conj(c) x is a sign flip
  bool binary = a.code_bits != nullptr;
  if (binary) {
    if (a.tx_per_pulse) {
      bool ok = true;
      for (int p = i0 * Q + lane; p < min(i1 * Q, a.n_pulses); p += 64)
        ok = ok && a.code_binary[p] != 0;
      binary = __all(ok);
    } else {
      binary = a.code_binary[0] != 0;
    }
  }
  if (binary) {
    if (i0 < i1) {
      fetch(i0, 0, JP);
      fetch_bits(i0);
    }
    for (int i = i0; i < i1; ++i) {
      float2 v[16];
      if constexpr (JP < JL) fetch(i, JP, JL);
#pragma unroll
      for (int t = 0; t < Q; ++t) {
        uint32_t b = bits[t];  // bit 31 - j: sample j's sign, brought to the top by b + b (a shift
                               // does not pair with other waves' instructions, an add does)
#pragma unroll
        for (int j = 0; j < JL; ++j) {
          const float2 x = IO::cvt(raw[t * JL + j]);
          const uint32_t sgn = b & 0x80000000u;
          v[t * J + j] = make_float2(__uint_as_float(__float_as_uint(x.x) ^ sgn),
                                     __uint_as_float(__float_as_uint(x.y) ^ sgn));
          asm("v_add_u32 %0, %0, %0" : "+v"(b));
        }
      }
      __builtin_amdgcn_sched_barrier(0);
      fetch(i + 1, 0, JP);
      fetch_bits(i + 1);
      transform(v);
    }
  } else {
    for (int i = i0; i < i1; ++i) {
      float2 v[16];
      fetch(i, 0, JL);
#pragma unroll
      for (int t = 0; t < Q; ++t) {
        const int p = i * Q + t;
        const auto d = row_desc(a.tx, a.tx_per_pulse ? static_cast<int64_t>(p) * L : 0, 8,
                                p < a.n_pulses ? L : 0);
#pragma unroll
        for (int j = 0; j < JL; ++j) {
          const u32x2 cr = __builtin_amdgcn_raw_buffer_load_b64(d, (lane + 64 * j) * 8, 0, 0);
          v[t * J + j] = conj_mul(make_float2(__uint_as_float(cr.x), __uint_as_float(cr.y)),
                                  IO::cvt(raw[t * JL + j]));
        }
      }
      transform(v);
    }
  }

  // the workgroup's sums: each wave lays its bins out in its own region, then
  // every bin is added over runs and side-by-side transforms in fixed order
  wave_lds_sync();
  float* st = reinterpret_cast<float*>(xw);
  {
    const int ka = lane & 15, row = lane >> 4;
    const int base = CLS > 1 ? ka : (ka / J) * M + (ka & (J - 1));
#pragma unroll
    for (int t = 0; t < 4; ++t)
#pragma unroll
      for (int kd = 0; kd < 4; ++kd)
        st[base + J * (4 * row + t + 16 * kd)] = acc[4 * t + kd];
  }
  __syncthreads();
  const float* all_st = reinterpret_cast<const float*>(xs);
  // the chunk's partial row; on a grid of all N bins by gate, and with one
  // chunk the gate's row of the result itself
  const bool whole = a.grid_len == a.n_fft, last = whole && a.chunks == 1;
  float* out = last ? a.out + static_cast<int64_t>(g) * M
                    : a.grid + (static_cast<int64_t>(c) * a.rows + (whole ? g : slot)) * M;
  const bool add = last && a.accumulate;
  for (int e = tid; e < M; e += 64 * W) {
    float sum = 0.f;
#pragma unroll
    for (int r = 0; r < RUNS; ++r) {
      const float* wst = all_st + (CLS > 1 ? r * CLS + (e & (CLS - 1)) : r) * (2 * XWAVE);
      if constexpr (CLS > 1) {
        sum += wst[e / CLS];
      } else {
#pragma unroll
        for (int t = 0; t < Q; ++t) sum += wst[t * M + e];
      }
    }
    out[e] = add ? out[e] + sum : sum;
  }
}

// ---------------------------------------------------------------------------
// Expansion of the summed grid to N = 1024 R bins, L <= 1024.
//
// With the two-sided lags R[n] = rho[n] + i tau[n] (rho even, tau odd) and the
// real sequence q[n] = rho[n] + tau[n], H[k] = sum_{0 < |n| < L} q[n] W_N^{k n}
// gives two bins at once, S[k] = r0 + Re H - Im H and S[-k] = r0 + Re H + Im H.  Folded
// to 1024 points, bin class k1 (bins k1 + R kk) is the 1024-point transform of
//   h[n] = q[n] + e^{2 pi i k1 / R} q[n - 1024], 0 <= n < 1024,
// with the class's twiddles, and also yields class R - k1: the classes
// 0 ... R / 2 are all the transforms there are.  Bins on the grid are copied.
//
// One workgroup of eight waves per gate (two fit a compute unit): all waves sum
// the gate's chunk partials, wave 0 runs the inverse transform (for M < 1024
// also class 0, which makes the grid one of 1024 points), then each wave transforms one class and
// lays its two rows out in its own exchange buffer, from which the workgroup
// stores whole rows.  Everything between the partials and the result stays in LDS.

// Factors of passes 2 and 3 for bin class kappa of n = 1024 S points; `tw` is
// the table of `table` >= n points.
__device__ __forceinline__ void load_class_twiddles(GridTwiddles& w, const float2* __restrict__ tw,
                                                    int n, int table, int kappa, int lane) {
  const int step = table / n, mask = table - 1, S = n >> 10;
  const int row = lane >> 4, q = kappa + S * (lane & 15);
  load_geo(w.p2, tw, table, 4 * step * q);
#pragma unroll
  for (int t = 0; t < 4; ++t) {
    const int e = step * (q + 16 * S * (4 * row + t));
    w.t3[t] = tw[e & mask];
    w.t3sq[t] = tw[(2 * e) & mask];
  }
}

// Bin kb of register i of a lane after passes 2 and 3, and its place in a
// staged row of 1024 floats (the four 16-lane rows of a wave on different banks).
__device__ __forceinline__ int bin_of(int i, int lane) {
  return (lane & 15) + 16 * (4 * (lane >> 4) + (i >> 2)) + 256 * (i & 3);
}
__device__ __forceinline__ int staged(int kb) { return kb ^ ((kb >> 2) & 48); }

constexpr int EXP_WAVES = 8;
constexpr int MIRROR = 1040;   // second staged row of a wave's region
static_assert(MIRROR + SUB <= 2 * XWAVE, "two rows per region");

// Twiddle i of the table for a wave-uniform i, by a scalar load (the table is
// constant while a kernel runs).
__device__ __forceinline__ float2 uniform_twiddle(const float2* tw, int i) {
  using cptr = const __attribute__((address_space(4))) f32x2*;
  const f32x2 w = reinterpret_cast<cptr>(reinterpret_cast<uint64_t>(tw))[__builtin_amdgcn_readfirstlane(i)];
  return make_float2(w.x, w.y);
}

struct alignas(4) Float4u {
  float v[4];
};

// Whether the grid's sums can be expanded: finite, and far enough from the ends
// of the FP32 range that the transforms stay inside it.
__device__ __forceinline__ bool expandable(float mean) {
  return mean == 0.f || (mean > 1e-30f && mean < 1e30f);
}

// The N bins of gate g straight from its pulses, for a grid that cannot be
// expanded (a power beyond the FP32 range or near its lower end, NaN): bins then
// come out as the direct transform leaves them.
template <int ST>
__device__ void direct_row(const FoldArgs& a, int g, float2* xs, const Dft16Consts& dk, int tid) {
  using IO = BufferSample<ST>;
  constexpr int W = EXP_WAVES;
  const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int N = a.n_fft, R = N / SUB, L = a.code_len;
  const float2* __restrict__ tw = reinterpret_cast<const float2*>(a.twiddle);
  const int64_t gate_off = static_cast<int64_t>(a.first_gate) + static_cast<int64_t>(g) * a.gate_step;
  float2* xw = xs + wave * XWAVE;
  float* xf = reinterpret_cast<float*>(xs);
  float* out = a.out + static_cast<int64_t>(g) * N;
  for (int c0 = 0; c0 < R; c0 += W) {
    const int n_cls = min(W, R - c0), k1 = c0 + wave;
    __syncthreads();  // the regions are free
    if (wave < n_cls) {
      WaveTwiddlesGeo w;
      load_wave_twiddles(w, tw, N, k1, lane);
      float acc[16];
#pragma unroll
      for (int i = 0; i < 16; ++i) acc[i] = 0.f;
#pragma unroll 1
      for (int p = 0; p < a.n_pulses; ++p) {
        const auto ds = row_desc(a.samples, static_cast<int64_t>(p) * a.stride + gate_off, IO::SIZE, L);
        const auto dc = row_desc(a.tx, a.tx_per_pulse ? static_cast<int64_t>(p) * L : 0, 8, L);
        float2 v[16];
#pragma unroll
        for (int j = 0; j < 16; ++j) {
          const auto x = IO::load(ds, (lane + 64 * j) * IO::SIZE);
          const u32x2 cr = __builtin_amdgcn_raw_buffer_load_b64(dc, (lane + 64 * j) * 8, 0, 0);
          v[j] = conj_mul(make_float2(__uint_as_float(cr.x), __uint_as_float(cr.y)), IO::cvt(x));
        }
        wave_fft_accumulate(v, xw, w, dk, acc, lane);
      }
      wave_lds_sync();
#pragma unroll
      for (int i = 0; i < 16; ++i) xf[wave * 2 * XWAVE + bin_of(i, lane)] = acc[i];
    }
    __syncthreads();
    for (int k = tid; k < N; k += 64 * W) {
      const int i = (k & (R - 1)) - c0;
      if (i < 0 || i >= n_cls) continue;
      const float s = xf[i * 2 * XWAVE + k / R];
      out[k] = a.accumulate ? out[k] + s : s;
    }
  }
}

template <int ST>
__global__ void __launch_bounds__(64 * EXP_WAVES, 4) expand_grid(FoldArgs a) {
  constexpr int W = EXP_WAVES, NT = 64 * W;
  constexpr int UP = SUB + 4;  // aux: 1024-point grid of M < 1024
  __shared__ __attribute__((aligned(16))) float2 xs[W * XWAVE];
  __shared__ __attribute__((aligned(16))) float aux[2 * SUB + 8];
  __shared__ float red[W];

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int M = a.grid_len, N = a.n_fft, L = a.code_len, R = N / SUB;
  const int lr = __builtin_ctz(R);
  const float2* __restrict__ tw = reinterpret_cast<const float2*>(a.twiddle);
  const Dft16Consts dk = dft16_consts();
  float* xf = reinterpret_cast<float*>(xs);
  float2* xw = xs + wave * XWAVE;

  const int slot = a.gate_list ? static_cast<int>(blockIdx.x) : xcd_block_id();
  int g = a.slot0 + slot;
  if (a.gate_list) {
    if (g >= *a.gate_count) return;  // uniform, before any barrier
    g = a.gate_list[g];
    if (g < 0 || g >= a.n_gates) return;
  }

  // the classes 1, 2, ... last (class 0, and R / 2 at M = 2048, lie on the
  // grid), one per wave and round; at M = 2048 wave 0 runs the inverse transform only
  const bool wide = M == 2 * SUB;
  const int last = wide ? R / 2 - 1 : R / 2, per_round = wide ? W - 1 : W;
  const int task = wide ? wave - 1 : wave;
  const bool one_round = last <= per_round;

  // ---- the grid, chunk sums in ascending order, into aux; its mean
  float part = 0.f;
  {
    const float* row = a.grid + static_cast<int64_t>(slot) * M;
    const int64_t cs = static_cast<int64_t>(a.rows) * M;
    for (int k = 4 * tid; k < M; k += 4 * NT) {
      float4 s = *reinterpret_cast<const float4*>(row + k);
      for (int c0 = 1; c0 < a.chunks; c0 += 8) {
        float4 q[8];
#pragma unroll
        for (int u = 0; u < 8; ++u)
          q[u] = *reinterpret_cast<const float4*>(row + min(c0 + u, a.chunks - 1) * cs + k);
#pragma unroll
        for (int u = 0; u < 8; ++u)
          if (c0 + u < a.chunks) {
            s.x += q[u].x;
            s.y += q[u].y;
            s.z += q[u].z;
            s.w += q[u].w;
          }
      }
      *reinterpret_cast<float4*>(aux + k) = s;
      part += (s.x + s.y) + (s.z + s.w);
    }
  }
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) part += __shfl_xor(part, off);
  if (lane == 0) red[wave] = part;
  __syncthreads();
  float mean = 0.f;
#pragma unroll
  for (int i = 0; i < W; ++i) mean += red[i];
  mean *= 1.f / static_cast<float>(M);
  const bool ok = expandable(mean);

  // ---- lags: up to conjugation and 1 / M the forward DFT of the real grid,
  // M <= 1024 zero-interleaved to 1024 points (which repeats its spectrum),
  // M = 2048 as 1024 complex points z[2 a] + i z[2 a + 1]; with r = conj(F) / M
  // qs[n] = (q[n], q[-n]) = (Re r + Im r, Re r - Im r), n < M / 2, and one zero
  // more: behind the grid in aux, at M = 2048 in wave 0's own region
  const float scale = 1.f / static_cast<float>(M);
  float2* qs = wide ? xs : reinterpret_cast<float2*>(aux + M);
  if (wave == 0) {
    GridTwiddles w;
    load_class_twiddles(w, tw, SUB, N, 0, lane);
    float2 v[16];
    if (wide) {
#pragma unroll
      for (int j = 0; j < 16; ++j) {
        const float2 p = reinterpret_cast<const float2*>(aux)[lane + 64 * j];
        v[j] = make_float2(p.x - mean, p.y - mean);
      }
      dft16(v, dk);
      // (this wave's reads of its exchange buffer are all issued by then)
      wave_passes_23(v, xw, w, dk, lane, NoHook{},
                     [&](int i, float2 f) { xw[bin_of(i, lane)] = f; });
    } else {
      const int lup = __builtin_ctz(SUB / M), up = (1 << lup) - 1;
#pragma unroll
      for (int j = 0; j < 16; ++j) {
        const int n = lane + 64 * j;
        v[j] = make_float2((n & up) == 0 ? aux[n >> lup] - mean : 0.f, 0.f);
      }
      dft16(v, dk);
      wave_passes_23(v, xw, w, dk, lane, NoHook{},
                     [&](int i, float2 f) { xw[bin_of(i, lane)] = f; });
      wave_lds_sync();
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        const int n = lane + 64 * j;
        const float2 f = n > 0 && n < L ? xw[n] : make_float2(0.f, 0.f);
        if (n < M / 2) qs[n] = make_float2(scale * (f.x - f.y), scale * (f.x + f.y));
      }
      if (lane == 0) qs[M / 2] = make_float2(0.f, 0.f);
      if (M < SUB) {  // class 0
        wave_lds_sync();
#pragma unroll
        for (int j = 0; j < 16; ++j) {
          const int n = lane + 64 * j, m = SUB - n;
          const float qp = 64 * j < M / 2 ? qs[n].x : 0.f;
          const float qm = 64 * (15 - j) < M / 2 ? qs[m].y : 0.f;
          v[j] = make_float2(qp + qm, 0.f);
        }
        wave_lds_sync();
        dft16(v, dk);
        wave_passes_23(v, xw, w, dk, lane, NoHook{}, [&](int i, float2 F) {
          const int k = bin_of(i, lane);
          float s = F.x - F.y + mean;
          s = s < 0.f ? 0.f : s;  // S >= 0: a rounded zero stays one
          aux[UP + k] = (k & up) == 0 ? aux[k >> lup] : s;
        });
      }
    }
  }
  if (wide) {
    __syncthreads();
    // thread n turns F[n], F[1024 - n] into the lags n and 1024 - n in place
    static_assert(NT == SUB / 2, "a pair of lags per thread, thread 0 also the middle one");
    {
      const float2 A = xs[tid], B = xs[tid == 0 ? SUB / 2 : SUB - tid];
      auto lag = [&](int n, float2 p, float2 m) {  // p = F[n], m = F[1024 - n]
        float2 f = make_float2(0.f, 0.f);
        if (n > 0 && n < L) {
          const float2 E = make_float2(0.5f * (p.x + m.x), 0.5f * (p.y - m.y));
          const float2 O = make_float2(0.5f * (p.y + m.y), 0.5f * (m.x - p.x));
          f = cmuladd(E, tw[n * (N / (2 * SUB))], O);
        }
        qs[n] = make_float2(scale * (f.x - f.y), scale * (f.x + f.y));
      };
      lag(tid, A, B);
      lag(SUB - tid, B, A);  // tid = 0: the zero past the last lag
      if (tid == 0) lag(SUB / 2, B, B);
    }
  }

  // ---- the classes
  const float* grid = M < SUB ? aux + UP : aux;
  const int lratio = __builtin_ctz(N / max(M, SUB)), rmask = (1 << lratio) - 1;
  for (int z0 = 1; z0 == 1 || z0 <= last; z0 += per_round) {
    const int n_cls = min(per_round, last - z0 + 1);  // 0: every bin is on the grid
    const bool mine = task >= 0 && task < n_cls;
    const int k1 = z0 + task;
    GridTwiddles w;
    float2 pre[16];
    float2 rot = make_float2(1.f, 0.f);  // e^{2 pi i k1 / R}
    if (mine) {
      load_class_twiddles(w, tw, N, N, k1, lane);
#pragma unroll
      for (int j = 0; j < 16; ++j) pre[j] = uniform_twiddle(tw, (64 * k1 * j) & (N - 1));
      const float2 r = uniform_twiddle(tw, (SUB * k1) & (N - 1));
      rot = make_float2(r.x, -r.y);
    }
    __syncthreads();  // the lags (first round) are written, the regions free
    if (mine) {
      float2 v[16];
#pragma unroll
      for (int j = 0; j < 16; ++j) {  // q[n] and q[n - 1024], n = lane + 64 j
        const int n = lane + 64 * j, m = SUB - n;
        const float qp = 64 * j < M / 2 ? qs[n].x : 0.f;
        const float qm = 64 * (15 - j) < M / 2 ? qs[m].y : 0.f;
        v[j] = make_float2(fmaf(rot.x, qm, qp), rot.y * qm);
      }
      dft16_pre1(v, pre, dk);
      float* own = reinterpret_cast<float*>(xw);
      wave_passes_23(v, xw, w, dk, lane, NoHook{}, [&](int i, float2 f) {
        // staged(bin_of(i, lane)), with the register's kd as a constant offset
        const int r4 = lane >> 4;
        const int at = (lane & 15) + 64 * r4 + 16 * ((i >> 2) ^ r4);
        own[at + 256 * (i & 3)] = f.x - f.y;
        own[at + 256 * (i & 3) + MIRROR] = f.x + f.y;
      });
    }
    __syncthreads();
    if (ok) {
      // the four bins k = 4 tid + u (+ 4 NT per step) this thread stores:
      // their staged rows, or -1: not of this round, or grid points
      int base[4];
      bool grid_pt[4], mirror[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int k = 4 * tid + u, cl = k & (R - 1);
        grid_pt[u] = (k & rmask) == 0;
        mirror[u] = 2 * cl > R;
        const int i = (mirror[u] ? R - cl : cl) - z0;
        base[u] = i >= 0 && i < n_cls
                      ? (i + (wide ? 1 : 0)) * 2 * XWAVE + (mirror[u] ? MIRROR : 0)
                      : -1;
        if (grid_pt[u]) base[u] = z0 == 1 ? 0 : -1;
      }
      float* out = a.out + static_cast<int64_t>(g) * N;
      for (int k0 = 4 * tid; k0 < N; k0 += 4 * NT) {
        Float4u s;
        if (a.accumulate) s = *reinterpret_cast<const Float4u*>(out + k0);
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          float x = 0.f;
          if (grid_pt[u]) {
            x = grid[(k0 + u) >> lratio];
          } else if (base[u] >= 0) {
            // class R - k1 holds bin -(k1 + R kk), i.e. its own entry 1023 - kk
            const int kb = (k0 + u) >> lr;
            x = xf[base[u] + staged(mirror[u] ? SUB - 1 - kb : kb)] + mean;
            x = x < 0.f ? 0.f : x;
          }
          s.v[u] = a.accumulate ? s.v[u] + x : x;
        }
        if (one_round) {
          *reinterpret_cast<Float4u*>(out + k0) = s;
        } else {
#pragma unroll
          for (int u = 0; u < 4; ++u)
            if (base[u] >= 0) out[k0 + u] = s.v[u];
        }
      }
    }
    if (z0 + per_round <= last) __syncthreads();
  }
  if (!ok) direct_row<ST>(a, g, xs, dk, tid);
}

template <int LOGM, int ST>
hipError_t launch_grid_w(const FoldArgs& a, hipStream_t s) {
  const dim3 grid(static_cast<unsigned>(a.rows) * static_cast<unsigned>(a.chunks));
  switch (a.waves) {
    case 8: hipLaunchKernelGGL((grid_spectra<LOGM, ST, 8>), grid, dim3(512), 0, s, a); break;
    case 16: hipLaunchKernelGGL((grid_spectra<LOGM, ST, 16>), grid, dim3(1024), 0, s, a); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

template <int ST>
hipError_t launch_grid(const FoldArgs& a, hipStream_t s) {
  switch (a.grid_len) {
    case 128: return launch_grid_w<7, ST>(a, s);
    case 256: return launch_grid_w<8, ST>(a, s);
    case 512: return launch_grid_w<9, ST>(a, s);
    case 1024: return launch_grid_w<10, ST>(a, s);
    case 2048: return launch_grid_w<11, ST>(a, s);
    default: return hipErrorInvalidValue;
  }
}

template <int ST>
hipError_t launch_expand(const FoldArgs& a, hipStream_t s) {
  hipLaunchKernelGGL(expand_grid<ST>, dim3(static_cast<unsigned>(a.rows)), dim3(64 * EXP_WAVES), 0,
                     s, a);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_folded(const FusedArgs& f, hipStream_t s) {
  FoldArgs a{};
  a.samples = f.samples;
  a.tx = f.tx;
  a.twiddle = f.twiddle;
  a.grid = f.grid;
  a.out = f.out;
  a.stride = f.stride;
  a.n_fft = f.n_fft;
  a.grid_len = f.grid_len;
  a.code_len = f.code_len;
  a.n_gates = f.n_gates;
  a.gate_step = f.gate_step;
  a.first_gate = f.first_gate;
  a.n_pulses = f.n_pulses;
  a.chunks = f.grid_chunks;
  a.waves = f.grid_waves;
  a.tx_per_pulse = f.tx_per_pulse;
  a.accumulate = f.accumulate;
  a.gate_list = f.gate_list;
  a.gate_count = f.gate_count;
  if (f.grid_bits) {
    const int rows = f.tx_per_pulse ? f.n_pulses : 1;
    hipLaunchKernelGGL(pack_grid_bits, dim3(static_cast<unsigned>((rows + 3) / 4)), dim3(256), 0, s,
                       reinterpret_cast<const float2*>(f.tx), rows, f.code_len, f.grid_bits,
                       f.grid_binary);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    a.code_bits = f.grid_bits;
    a.code_binary = f.grid_binary;
  }
  if (a.grid_len == a.n_fft) {  // every bin is on the grid: partials by gate, no expansion
    a.rows = f.n_gates;
    hipError_t e = f.sample_type == 1 ? launch_grid<1>(a, s) : launch_grid<0>(a, s);
    if (e == hipSuccess && a.chunks > 1)
      e = launch_reduce_chunks(a.grid, a.out, static_cast<int64_t>(f.n_gates) * f.n_fft, a.chunks,
                               a.accumulate, a.n_fft, a.gate_list, a.gate_count, s);
    return e;
  }
  // as many gates at a time as the scratch holds
  for (int32_t s0 = 0; s0 < f.n_gates; s0 += f.grid_rows) {
    a.slot0 = s0;
    a.rows = std::min(f.n_gates - s0, f.grid_rows);
    hipError_t e = f.sample_type == 1 ? launch_grid<1>(a, s) : launch_grid<0>(a, s);
    if (e == hipSuccess)
      e = f.sample_type == 1 ? launch_expand<1>(a, s) : launch_expand<0>(a, s);
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

}  // namespace ispl
