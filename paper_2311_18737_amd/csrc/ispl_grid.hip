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
// points per pulse and gate: 1000 pulses x 1000 gates (int16 samples) take 1.92 instead of
// 11.45 ms.  The grid's mean is taken out before the inverse transform and r[0]
// added back last, so rounding in the two transforms is relative to the
// spectrum's fluctuation about its mean, not to the mean.
//
// What is wrong at a strong grid point is spread over its neighbours by the expansion, as
// 1 / (pi x distance): a direct transform's rounding stays at the line.  So the
// powers are squared and summed in double (7 to 10 % of the pass; sums of 32 pulses in FP32
// before that), and a point's sum is multiplied by the known gain of its FP32 twiddles
// (ispl_gain.h).  Largest error over max(S, mean S) with a line at -10 dB per sample, L = 1000 /
// 2000 / 4000: 4e-7 / 8e-7 / 1.7e-6 (FP32 sums 3.1e-6 / 7.5e-6 / 1.2e-5, double ones
// without the gain 2.0e-6 / 5.7e-6 / 1.7e-5; direct 5e-7); without a line 1.0e-7 to 1.4e-7, direct
// 4e-7 to 6e-7.  Gates with a line too strong for that are redone by direct transforms (peak_limit).

#include <float.h>
#include <math.h>
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

#include <algorithm>

#include "ispl_fft.h"
#include "ispl_fft64.h"
#include "ispl_gain.h"
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
// What bounds it is VALU issue (M = 2048: 600 VALU instructions per wave and
// pulse, 32 of them in double, at 0.29 per SIMD and cycle; a fifth of the waves' time goes to LDS).  Register-only probes at four waves per
// SIMD: two-operand (4-byte) instructions issue at 0.43 per cycle, three-operand
// ones (8 bytes) at 0.34, and conversions, shifts and anything reading a scalar
// register at 0.22, a v_permlane swap at 0.12.  Hence pass 3's exchange between
// lane rows goes through LDS (12 % fewer cycles than with swaps), the code
// bits are brought up by additions, and pass 3's twiddles lie in LDS (beside double sums, which
// take 32 registers, pass 2's too), which keeps four waves per SIMD with the next pulse's
// samples in flight.

// Pulses (or steps of several) that one FP32 sum takes before it is added to the
// row in memory, on a grid of all N bins (the rounding of a long sum grows with its length).
constexpr int RUN_STEPS = 32;

// `steps` cut into `n` runs, the first steps % n of them one longer (a 32-bit
// division: s * steps / n takes 64 bits and hundreds of instructions each).
struct RunSplit {
  uint32_t each, extra;
  __device__ RunSplit(int steps, int n)
      : each(static_cast<uint32_t>(steps) / static_cast<uint32_t>(n)),
        extra(static_cast<uint32_t>(steps) - each * static_cast<uint32_t>(n)) {}
  __device__ int begin(int s) const {
    return __builtin_amdgcn_readfirstlane(
        static_cast<int>(static_cast<uint32_t>(s) * each + min(static_cast<uint32_t>(s), extra)));
  }
  __device__ int longest() const { return static_cast<int>(each + (extra != 0 ? 1 : 0)); }
};

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

// x, recomputed by the compiler wherever it is used (values formed from it are
// not kept across a loop).
__device__ __forceinline__ int opaque(int x) {
  asm volatile("" : "+v"(x));
  return x;
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

// The gate of a workgroup's slot, or -1 (uniform, before any barrier).
__device__ __forceinline__ int gate_of(const FoldArgs& a, int slot) {
  const int g = a.slot0 + slot;
  if (!a.gate_list) return g;
  if (g >= *a.gate_count) return -1;
  const int listed = a.gate_list[g];
  return listed < a.n_gates ? listed : -1;
}

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

// Where chunk c of a gate's sums goes: the chunk's partial row by slot; on a grid of all N
// bins (WHOLE, FP32) by gate, and with one chunk the gate's row of the result itself.
template <bool WHOLE>
__device__ __forceinline__ auto out_row(const FoldArgs& a, int g, int slot, int c) {
  const int64_t row = static_cast<int64_t>(c) * a.rows + (WHOLE ? g : slot);
  if constexpr (WHOLE)
    return a.chunks == 1 ? a.out + static_cast<int64_t>(g) * a.grid_len : a.partial + row * a.grid_len;
  else
    return a.grid + row * a.grid_len;
}

// The gains of a grid's points (a context's are written on the host).
__global__ void __launch_bounds__(256)
build_gains(const double* __restrict__ tw64, int32_t n_fft, int32_t len, double* __restrict__ gain) {
  const int k = static_cast<int>(blockIdx.x * blockDim.x + threadIdx.x);
  if (k < len) gain[k] = grid_gain(tw64, n_fft, len, k);
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
  bits[64 * static_cast<int64_t>(row) + lane] = word;
  const bool all = __all(ok);
  if (lane == 0) binary[row] = all ? 1 : 0;
}

// LOGM: log2 of the grid; W: waves per workgroup.  The workgroup's waves take
// W runs of pulses (LOGM = 11: W / 2 runs, each by one wave per bin class); with
// C chunks the run count is C times that.  WHOLE: the grid is the N bins themselves, summed
// in FP32 as the direct transform's are.
template <int LOGM, int ST, int W, bool WHOLE>
__global__ void __launch_bounds__(64 * W, 4) grid_spectra(FoldArgs a) {
  constexpr int M = 1 << LOGM;
  constexpr int CLS = M > SUB ? M / SUB : 1;    // bin classes
  constexpr int Q = M < SUB ? SUB / M : 1;      // pulses per step
  constexpr int J = CLS > 1 ? 16 : M / 64;      // pass-1 points per pulse
  constexpr int JL = CLS > 1 ? 16 : J / 2;      // of which loaded
  constexpr int RUNS = W / CLS;
  // samples per pulse fetched a step ahead (all that four waves per SIMD have registers for)
  constexpr int JP = CLS > 1 ? (ST == 0 ? 6 : 12) : JL;
  using sum_t = std::conditional_t<WHOLE, float, double>;
  static_assert(CLS <= 2 && W % CLS == 0, "at most two bin classes");
  using IO = BufferSample<ST>;
  __shared__ float2 xs[W * XWAVE];
  __shared__ float4 t3s[CLS][4][64];  // pass-3 twiddles of each class
  __shared__ float4 p2s[WHOLE ? 1 : CLS][5][16];  // and pass 2's (beside double sums)

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int cls = CLS > 1 ? wave & 1 : 0;
  const int run = wave / CLS;
  if (a.redo_count && blockIdx.x == 0 && tid == 0) *a.redo_count = 0;  // (the expansion's list)
  const int bid = a.gate_list ? static_cast<int>(blockIdx.x) : xcd_block_id();
  const int c = bid % a.chunks, slot = bid / a.chunks;
  const int g = gate_of(a, slot);
  if (g < 0) return;
  if constexpr (!WHOLE)
    if (a.skip && a.skip[slot] != 0) return;
  const int L = a.code_len;
  const float2* __restrict__ tw = reinterpret_cast<const float2*>(a.twiddle);
  // pass-2 column k1 of this lane (bins k1 + (M / 64) (kc + 16 kd)) and its
  // progressions W_M^{4 k1 m} (pass 2) and (W_M^{k1} W_64^{kc})^r (pass 3)
  std::conditional_t<WHOLE, GridTwiddlesLds, GridTwiddlesLds2> wt;
  {
    const int step = a.n_fft >> LOGM, k1 = CLS > 1 ? cls + CLS * (lane & 15) : lane & (J - 1);
    if constexpr (WHOLE) load_geo(wt.p2, tw, a.n_fft, 4 * step * k1);
    if (wave < CLS) {
      if constexpr (!WHOLE)
        for (int t = lane >> 4; t < 5; t += 4)
          p2s[wave][t][lane & 15] = geo_part(tw, a.n_fft, 4 * step * k1, t);
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        const int e = step * k1 + (a.n_fft >> 6) * (4 * (lane >> 4) + t);
        const float2 u = tw[e & (a.n_fft - 1)], u2 = tw[(2 * e) & (a.n_fft - 1)];
        t3s[wave][t][lane] = make_float4(u.x, u.y, u2.x, u2.y);
      }
    }
    wt.t3 = &t3s[cls][0][lane];
    if constexpr (!WHOLE) wt.p2.p = &p2s[cls][0][lane & 15];
    __syncthreads();
  }
  const Dft16Consts dk = dft16_consts();
  sum_t acc[16];
#pragma unroll
  for (int i = 0; i < 16; ++i) acc[i] = 0;

  const int64_t gate_off = static_cast<int64_t>(a.first_gate) + static_cast<int64_t>(g) * a.gate_step;
  const RunSplit runs((a.n_pulses + Q - 1) / Q, a.chunks * RUNS);
  const int i0 = runs.begin(c * RUNS + run), i1 = runs.begin(c * RUNS + run + 1);
  float2* xw = xs + wave * XWAVE;

  typename IO::raw_t raw[Q * JL];
  uint32_t bits[Q];
  // samples j0 <= j < j1 of each pulse of step i (zero past the last pulse)
  auto fetch = [&](int i, int j0, int j1) {
    // formed here, the offsets fold into the loads; hoisted out of the loop they
    // would take a register each
    const int so = opaque(lane * IO::SIZE);
#pragma unroll
    for (int t = 0; t < Q; ++t) {
      const int p = i * Q + t;
      const auto d = row_desc(a.samples, static_cast<int64_t>(p) * a.stride + gate_off, IO::SIZE,
                              p < a.n_pulses && i < i1 ? L : 0);
#pragma unroll
      for (int j = 0; j < JL; ++j)
        if (j >= j0 && j < j1) raw[t * JL + j] = IO::load(d, so + 64 * IO::SIZE * j);
    }
  };
  auto fetch_bits = [&](int i) {
#pragma unroll
    for (int t = 0; t < Q; ++t) {
      const int p = min(i * Q + t, a.n_pulses - 1);
      bits[t] = a.code_bits[(a.tx_per_pulse ? 64 * static_cast<int64_t>(p) : 0) + lane];
    }
  };
  auto transform = [&](float2 (&v)[16]) {
    if constexpr (CLS == 1)
      grid_pass1<Q>(v, dk);
    else if (cls == 0)
      dft16(v, dk);
    else
      dft16_w32(v, dk);
    wave_passes_23(v, xw, wt, dk, lane, NoHook{},
                   std::conditional_t<WHOLE, PowerSink, PowerSink64>{acc});
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
  sum_t* out = out_row<WHOLE>(a, g, slot, c);
  bool add = WHOLE ? a.chunks == 1 && a.accumulate : a.add != 0;
  // at most RUN_STEPS steps go into one FP32 sum (the same number of sums for
  // every run, which meet at its end), all into one double
  const int per_sum = WHOLE ? RUN_STEPS : max(1, runs.longest());
  const int n_sums = WHOLE ? max(1, (runs.longest() + RUN_STEPS - 1) / RUN_STEPS) : 1;
  for (int u = 0; u < n_sums; ++u) {
  const int b0 = min(i0 + u * per_sum, i1), b1 = min(b0 + per_sum, i1);
  if (binary) {
    if (b0 < b1) {
      fetch(b0, 0, JP);
      fetch_bits(b0);
    }
    for (int i = b0; i < b1; ++i) {
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
    // (the two bin classes of M = 2048 have no registers for a prefetch beside the codes)
    if (CLS == 1 && b0 < b1) fetch(b0, 0, JL);
    for (int i = b0; i < b1; ++i) {
      float2 v[16];
      if constexpr (CLS > 1) fetch(i, 0, JL);
      const int co = opaque(lane * 8);
#pragma unroll
      for (int t = 0; t < Q; ++t) {
        const int p = i * Q + t;
        const auto d = row_desc(a.tx, a.tx_per_pulse ? static_cast<int64_t>(p) * L : 0, 8,
                                p < a.n_pulses ? L : 0);
#pragma unroll
        for (int j = 0; j < JL; ++j) {
          const u32x2 cr = __builtin_amdgcn_raw_buffer_load_b64(d, co + 512 * j, 0, 0);
          v[t * J + j] = conj_mul(make_float2(__uint_as_float(cr.x), __uint_as_float(cr.y)),
                                  IO::cvt(raw[t * JL + j]));
        }
      }
      if constexpr (CLS == 1) {
        __builtin_amdgcn_sched_barrier(0);
        fetch(i + 1, 0, JL);
      }
      transform(v);
    }
  }

  // the workgroup's sums: each wave lays its bins out in its own region, then
  // every bin is added over runs and side-by-side transforms in fixed order
  wave_lds_sync();
  // (addresses formed here each time: kept across the pulse loop they would
  // take its registers)
  const int ft = opaque(tid), fl = ft & 63;
  constexpr int REGION = XWAVE * sizeof(float2) / sizeof(sum_t);
  sum_t* st = reinterpret_cast<sum_t*>(xs) + (ft >> 6) * REGION;
  {
    const int ka = fl & 15, row = fl >> 4;
    const int base = CLS > 1 ? ka : (ka / J) * M + (ka & (J - 1));
#pragma unroll
    for (int t = 0; t < 4; ++t)
#pragma unroll
      for (int kd = 0; kd < 4; ++kd) {
        st[base + J * (4 * row + t + 16 * kd)] = acc[4 * t + kd];
        acc[4 * t + kd] = 0;
      }
  }
  __syncthreads();
  const sum_t* all_st = reinterpret_cast<const sum_t*>(xs);
  for (int e = ft; e < M; e += 64 * W) {
    constexpr int kSumUnroll = RUNS * Q > 64 ? 4 : RUNS;
    sum_t sum = 0;
#pragma unroll kSumUnroll
    for (int r = 0; r < RUNS; ++r) {
      const sum_t* wst = all_st + (CLS > 1 ? r * CLS + (e & (CLS - 1)) : r) * REGION;
      if constexpr (CLS > 1) {
        sum += wst[e / CLS];
      } else {
#pragma unroll
        for (int t = 0; t < Q; ++t) sum += wst[t * M + e];
      }
    }
    if constexpr (!WHOLE) sum *= a.gain[e];
    out[e] = add ? out[e] + sum : sum;
  }
  add = true;
  if (u + 1 < n_sums) __syncthreads();  // the regions are exchange buffers again
  }
}

// ---------------------------------------------------------------------------
// Grid pass, L > 1024: M = 1024 J points, J = 4 or 8 >= L / 512, and J = 16 where
// those are all the bins (L <= 8192).
//
// A workgroup of J waves transforms one pulse at a time.  With n = lg + 1024 j
// the first pass is a J-point DFT over j for every lg < 1024 (half of its inputs
// lie past the code), 16 / J values of lg per thread; an exchange through LDS hands wave k1 the
// outputs k1 of all lg, and its 1024-point transform with the factors
// W_M^{k1 lg} gives bins k1 + J kb.  The factors are a geometric progression in
// every pass, so none costs a multiplication of its own.
//
// Two barriers a pulse and the exchange bound it (J = 8, int16: 29 % of the waves' time waits for
// LDS, VALU issue 0.19 per SIMD and cycle); registers
// decide what is kept in flight: all eight int16 samples of the next pulse, half
// of the complex64 ones (all of them spill, and a reload waits for every load
// before it).  200 pulses x 500 gates at L = 4000, N = 16384, phase codes (int16)
// take 1.13 ms, 2.22 by direct transforms; 500 pulses x 2000 gates at L = 2000, N = 32768
// 5.1 instead of 31 ms.

// Code rows as sign bits for the long grid: word lg of a row holds in bit
// 31 - j whether code sample lg + 1024 j is -1.  One workgroup per row.
__global__ void __launch_bounds__(256)
pack_long_grid_bits(const float2* __restrict__ tx, int32_t code_len, uint32_t* __restrict__ bits,
                    int32_t* __restrict__ binary) {
  const int row = blockIdx.x;
  bool ok = true;
#pragma unroll
  for (int t = 0; t < 4; ++t) {
    const int lg = static_cast<int>(threadIdx.x) + 256 * t;
    u32x2 c[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      const auto d = row_desc(tx, static_cast<int64_t>(row) * code_len + SUB * j, 8,
                              max(0, code_len - SUB * j));
      c[j] = __builtin_amdgcn_raw_buffer_load_b64(d, 8 * lg, 0, 0);
    }
    uint32_t word = 0;
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      const float x = __uint_as_float(c[j].x), y = __uint_as_float(c[j].y);
      ok = ok && (lg + SUB * j >= code_len || ((x == 1.f || x == -1.f) && y == 0.f));
      word |= (x < 0.f ? 1u : 0u) << (31 - j);
    }
    bits[static_cast<int64_t>(row) * SUB + lg] = word;
  }
  ok = __syncthreads_and(ok);
  if (threadIdx.x == 0) binary[row] = ok ? 1 : 0;
}

// A long grid's sums: its chunks' partials, `elems` apart, in ascending order.
__global__ void __launch_bounds__(256)
sum_chunks(const double* __restrict__ partial, double* __restrict__ to, int64_t elems, int32_t chunks) {
  const int64_t step = static_cast<int64_t>(gridDim.x) * blockDim.x;
  for (int64_t i = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x; i < elems; i += step) {
    double s = 0.0;
    for (int c = 0; c < chunks; ++c) s += partial[c * elems + i];
    to[i] = s;
  }
}

template <int J, int ST, bool WHOLE>
__global__ void __launch_bounds__(64 * J, 4) grid_long(FoldArgs a) {
  constexpr int NT = 64 * J, PER = 16 / J, JL = J / 2;
  constexpr int JP = ST == 0 ? JL / 2 : JL;  // of each thread's samples, fetched a pulse ahead
  using IO = BufferSample<ST>;
  __shared__ float2 xs[J * XWAVE];
  using sum_t = std::conditional_t<WHOLE, float, double>;
  __shared__ GeoTwiddles p1s[J];  // pass-1 progression W_M^{64 k1} of each wave
  __shared__ float4 p2s[WHOLE ? 1 : J][5][16];  // pass 2's (beside double sums)

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  if (a.redo_count && blockIdx.x == 0 && tid == 0) *a.redo_count = 0;  // (the expansion's list)
  const int bid = a.gate_list ? static_cast<int>(blockIdx.x) : xcd_block_id();
  const int c = bid % a.chunks, slot = bid / a.chunks;
  const int g = gate_of(a, slot);
  if (g < 0) return;
  if constexpr (!WHOLE)
    if (a.skip && a.skip[slot] != 0) return;
  const int L = a.code_len, M = SUB * J, step = a.n_fft / M, nmask = a.n_fft - 1;
  const float2* __restrict__ tw = reinterpret_cast<const float2*>(a.twiddle);
  // (complex64 samples in flight take 16 registers)
  std::conditional_t<!WHOLE, GridTwiddlesRows2,
                     std::conditional_t<ST == 0, GridTwiddlesRows1, GridTwiddlesRows>> wt;
  {
    const int q = wave + J * (lane & 15);
    if constexpr (WHOLE) {
      load_geo(wt.p2, tw, a.n_fft, 4 * step * q);
    } else {
      for (int t = lane >> 4; t < 5; t += 4)
        p2s[wave][t][lane & 15] = geo_part(tw, a.n_fft, 4 * step * q, t);
      wt.p2.p = &p2s[wave][0][lane & 15];
    }
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      const int e = step * (q + 16 * J * (4 * (lane >> 4) + t));
      wt.t3[t] = tw[e & nmask];
      if constexpr (WHOLE && ST == 1) wt.t3sq[t] = tw[(2 * e) & nmask];
    }
    if (lane == 0) load_geo(p1s[wave], tw, a.n_fft, 64 * step * wave);
  }
  const Dft16Consts dk = dft16_consts();
  sum_t acc[16];
#pragma unroll
  for (int i = 0; i < 16; ++i) acc[i] = 0;

  const int64_t gate_off = static_cast<int64_t>(a.first_gate) + static_cast<int64_t>(g) * a.gate_step;
  const RunSplit runs(a.n_pulses, a.chunks);
  const int p0 = runs.begin(c), p1 = runs.begin(c + 1);
  float2* xw = xs + wave * XWAVE;

  typename IO::raw_t raw[8];  // sample tid + NT t + 1024 j in raw[t JL + j]
  uint32_t bits[PER];
  auto fetch = [&](int p, int j0, int j1) {
    const int so = opaque(tid * IO::SIZE);  // (as in grid_spectra)
#pragma unroll
    for (int j = 0; j < JL; ++j) {
      if (j < j0 || j >= j1) continue;
      const auto d = row_desc(a.samples, static_cast<int64_t>(p) * a.stride + gate_off + SUB * j,
                              IO::SIZE, p < p1 ? max(0, L - SUB * j) : 0);
#pragma unroll
      for (int t = 0; t < PER; ++t) raw[t * JL + j] = IO::load(d, so + NT * IO::SIZE * t);
    }
  };
  auto fetch_bits = [&](int p) {
    const uint32_t* row = a.code_bits + (a.tx_per_pulse ? static_cast<int64_t>(min(p, p1 - 1)) * SUB : 0);
#pragma unroll
    for (int t = 0; t < PER; ++t) bits[t] = row[tid + NT * t];
  };
  // first pass in place: outputs k1 of thread value t in v[t J + k1]
  auto first_pass = [&](float2 (&v)[16]) {
#pragma unroll
    for (int t = 0; t < PER; ++t) {
      if constexpr (J == 4) {
        const float2 x = v[4 * t], y = v[4 * t + 1];
        v[4 * t] = make_float2(x.x + y.x, x.y + y.y);
        v[4 * t + 1] = make_float2(x.x + y.y, x.y - y.x);
        v[4 * t + 2] = make_float2(x.x - y.x, x.y - y.y);
        v[4 * t + 3] = make_float2(x.x - y.y, x.y + y.x);
      } else if constexpr (J == 8) {
        dft8_first4(v + 8 * t, dk);
      } else {
        dft16_first8(v, dk);
      }
    }
  };
  auto transform = [&](float2 (&v)[16]) {
    __syncthreads();  // every wave has finished its exchanges of the previous pulse
#pragma unroll
    for (int t = 0; t < PER; ++t)
#pragma unroll
      for (int k = 0; k < J; ++k) xs[k * XWAVE + tid + NT * t] = v[t * J + k];
    __syncthreads();
#pragma unroll
    for (int i = 0; i < 16; ++i) v[i] = xw[lane + 64 * i];
    wave_lds_sync();  // read before this wave reuses its region for its own exchange
    dft16_geo(v, p1s[wave]);
    wave_passes_23(v, xw, wt, dk, lane, NoHook{},
                   std::conditional_t<WHOLE, PowerSink, PowerSink64>{acc});
  };

  // codes of this workgroup's pulses all +-1: conj(c) x is a sign flip
  bool binary = a.code_bits != nullptr;
  if (binary) {
    if (a.tx_per_pulse) {
      bool ok = true;
      for (int p = p0 + lane; p < p1; p += 64) ok = ok && a.code_binary[p] != 0;
      binary = __all(ok);  // every wave reads the same flags
    } else {
      binary = a.code_binary[0] != 0;
    }
  }
  sum_t* out = out_row<WHOLE>(a, g, slot, c);
  bool add = WHOLE ? a.chunks == 1 && a.accumulate : a.add != 0;
  const int per_sum = WHOLE ? RUN_STEPS : max(1, p1 - p0);  // (as in grid_spectra)
  for (int q0 = p0; q0 == p0 || q0 < p1; q0 += per_sum) {
    const int q1 = min(q0 + per_sum, p1);
    if (binary) {
      if (q0 < q1) {
        fetch(q0, 0, JP);
        fetch_bits(q0);
      }
      for (int p = q0; p < q1; ++p) {
        float2 v[16];
        if constexpr (JP < JL) fetch(p, JP, JL);
#pragma unroll
        for (int t = 0; t < PER; ++t) {
          uint32_t b = bits[t];
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
        fetch(p + 1, 0, JP);
        fetch_bits(p + 1);
        first_pass(v);
        transform(v);
      }
    } else {
      // (complex64 samples have no registers for a prefetch beside the codes)
      if (ST == 1 && q0 < q1) fetch(q0, 0, JL);
      for (int p = q0; p < q1; ++p) {
        float2 v[16];
        if constexpr (ST == 0) fetch(p, 0, JL);
        const int co = opaque(tid * 8);
#pragma unroll
        for (int j = 0; j < JL; ++j) {
          const auto d = row_desc(a.tx, (a.tx_per_pulse ? static_cast<int64_t>(p) * L : 0) + SUB * j, 8,
                                  max(0, L - SUB * j));
#pragma unroll
          for (int t = 0; t < PER; ++t) {
            const u32x2 cr = __builtin_amdgcn_raw_buffer_load_b64(d, co + 8 * NT * t, 0, 0);
            v[t * J + j] = conj_mul(make_float2(__uint_as_float(cr.x), __uint_as_float(cr.y)),
                                    IO::cvt(raw[t * JL + j]));
          }
        }
        if constexpr (ST == 1) {
          __builtin_amdgcn_sched_barrier(0);
          fetch(p + 1, 0, JL);
        }
        first_pass(v);
        transform(v);
      }
    }

    // the sums in bin order through LDS (bin k1 + J kb of wave k1), stored in runs
    __syncthreads();
    // (addresses formed here each time: kept across the pulse loop they would
    // take its registers)
    const int ft = opaque(tid), fl = ft & 63;
    constexpr int REGION = XWAVE * sizeof(float2) / sizeof(sum_t);
    sum_t* st = reinterpret_cast<sum_t*>(xs) + (ft >> 6) * REGION;
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      const int r4 = fl >> 4;
      st[(fl & 15) + 64 * r4 + 16 * ((i >> 2) ^ r4) + 256 * (i & 3)] = acc[i];  // staged(bin_of)
      acc[i] = 0;
    }
    __syncthreads();
    const sum_t* all_st = reinterpret_cast<const sum_t*>(xs);
    for (int e = ft; e < M; e += NT) {
      const int kb = e / J;
      sum_t s = all_st[(e & (J - 1)) * REGION + (kb ^ ((kb >> 2) & 48))];
      if constexpr (!WHOLE) s *= a.gain[e];
      out[e] = add ? out[e] + s : s;
    }
    add = true;  // (the next pulse's first barrier frees the regions)
  }
}

// ---------------------------------------------------------------------------
// Expansion of the summed grid to N = 1024 R bins.
//
// With the two-sided lags R[n] = rho[n] + i tau[n] (rho even, tau odd) and the
// real sequence q[n] = rho[n] + tau[n], H[k] = sum_{0 < |n| < L} q[n] W_N^{k n}
// gives two bins at once, S[k] = r0 + Re H - Im H and S[-k] = r0 + Re H + Im H.  Folded
// to 1024 points, bin class k1 (bins k1 + R kk) is the 1024-point transform of
//   h[n] = sum_s q[n + 1024 s] W_R^{k1 s} + q[n - 1024 (s + 1)] W_R^{-k1 (s + 1)},
// 0 <= n < 1024, s < max(1, M / 2048), with the class's twiddles, and also
// yields class R - k1: the classes 0 ... R / 2 are all the transforms there
// are.  Bins on the grid are copied, and classes wholly on it not transformed.
//
// One workgroup of eight waves per gate: all waves sum the gate's chunk
// partials, the inverse transform (up to M = 2048 by wave 0, for M < 1024 with
// class 0, which makes the grid one of 1024 points; longer grids as M / 2048 classes
// of one wave each) leaves q in LDS, then each wave transforms one class and
// lays its two rows out in its own exchange buffer, from which the workgroup
// stores whole rows.
//
// The transforms run in double precision: a line of power S_l leaves rounding of
// about 1e-7 S_l at its mirror frequency and other places of an FP32
// transform's structure, where S may be a hundred times smaller, which no direct
// transform does (1000 gates of N = 16384 take 71 us, in FP32 50).  The lags are double too: with
// FP32 lags a line at -10 dB left 7e-7 at L = 1000, now 4e-7.

// SG-point DFT in place, natural order (SG = 2 or 4).
template <int SG>
__device__ __forceinline__ void dft_small64(complex64d (&z)[SG]) {
  auto add = [](complex64d a, complex64d b) { return complex64d{a.x + b.x, a.y + b.y}; };
  auto sub = [](complex64d a, complex64d b) { return complex64d{a.x - b.x, a.y - b.y}; };
  auto four = [&](complex64d& a0, complex64d& a1, complex64d& a2, complex64d& a3) {
    const complex64d s02 = add(a0, a2), d02 = sub(a0, a2), s13 = add(a1, a3), d13 = sub(a1, a3);
    a0 = add(s02, s13);
    a2 = sub(s02, s13);
    a1 = complex64d{d02.x + d13.y, d02.y - d13.x};
    a3 = complex64d{d02.x - d13.y, d02.y + d13.x};
  };
  if constexpr (SG == 2) {
    const complex64d a = z[0], b = z[1];
    z[0] = add(a, b);
    z[1] = sub(a, b);
  } else {
    static_assert(SG == 4, "two or four segments");
    four(z[0], z[1], z[2], z[3]);
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

struct alignas(4) Float4u {
  float v[4];
};

// A gate's grid of m points: its mean, largest and smallest value.
struct GridStats {
  double sum = 0.0;
  float hi = 0.f, lo = FLT_MAX;
  __device__ __forceinline__ void add(double v) {
    sum += v;
    hi = fmaxf(hi, static_cast<float>(v));
    lo = fminf(lo, static_cast<float>(v));
  }
  // Over the workgroup, from each thread's part; sum becomes the mean.
  __device__ __forceinline__ void reduce(double* red, float2* red_ends, int m) {
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) {
      sum += __shfl_xor(sum, off);
      hi = fmaxf(hi, __shfl_xor(hi, off));
      lo = fminf(lo, __shfl_xor(lo, off));
    }
    if ((threadIdx.x & 63) == 0) {
      red[threadIdx.x >> 6] = sum;
      red_ends[threadIdx.x >> 6] = make_float2(hi, lo);
    }
    __syncthreads();
    sum = 0.0;
#pragma unroll
    for (int i = 0; i < EXP_WAVES; ++i) {
      sum += red[i];
      hi = fmaxf(hi, red_ends[i].x);
      lo = fminf(lo, red_ends[i].y);
    }
    sum /= static_cast<double>(m);
  }
  // Whether the bins follow from the grid at no more than a direct transform's error.  That is
  // about 7 roundings of sqrt(S mean S) in a bin of power S, the grid's about that of its largest
  // point, over the square root of the samples that a bin's rounding averages and whatever the
  // distance of the bin; so hi^2 <= limit mean lo, the limit as measured (peak_limit).
  // Infinite and NaN points fail.
  __device__ __forceinline__ bool usable(float limit) const {
    const double h = hi;
    return sum - sum == 0.0 && hi <= FLT_MAX && h * h <= limit * sum * lo;
  }
};

// Whether the gate's sums end with the probe's pulses.
__device__ __forceinline__ bool left_out(const FoldArgs& a, int slot) {
  return a.skip && a.skip[slot] != 0;
}

// Leaves gate g to the launches that follow (one thread per gate).
__device__ __forceinline__ void redo_gate(const FoldArgs& a, int g) {
  a.redo_list[atomicAdd(a.redo_count, 1)] = g;
}

// A gate's grid of M <= 2048 points into `to`, its chunk partials (cs apart)
// summed in ascending order; returns this thread's part of its statistics.
__device__ __forceinline__ GridStats gather_grid(const FoldArgs& a, const double* row, int64_t cs,
                                                 double* to, int tid) {
  GridStats part;
  for (int k = 2 * tid; k < a.grid_len; k += 2 * 64 * EXP_WAVES) {
    double2 s = *reinterpret_cast<const double2*>(row + k);
    for (int c0 = 1; c0 < a.chunks; c0 += 8) {
      double2 q[8];
#pragma unroll
      for (int u = 0; u < 8; ++u)
        q[u] = *reinterpret_cast<const double2*>(row + min(c0 + u, a.chunks - 1) * cs + k);
#pragma unroll
      for (int u = 0; u < 8; ++u)
        if (c0 + u < a.chunks) {
          s.x += q[u].x;
          s.y += q[u].y;
        }
    }
    *reinterpret_cast<double2*>(to + k) = s;
    part.add(s.x);
    part.add(s.y);
  }
  return part;
}

// After the first pulses of a long call: the gates whose largest point stands so far above the mean
// that they will be redone: hi <= 0.9 sqrt(limit) mean here, hi <= sqrt(limit mean lo) at the end, with
// lo about 0.8 mean.  (A gate left out that could have been expanded costs more than one summed for
// nothing: at 0.7, 500 gates of L = 1000 with -10 dB lines took 3793 us, without a probe 619.)  One
// workgroup per gate.
__global__ void __launch_bounds__(64 * EXP_WAVES) probe_grid(FoldArgs a, int32_t* __restrict__ skip) {
  __shared__ double red[EXP_WAVES];
  __shared__ float2 red_ends[EXP_WAVES];
  const int slot = blockIdx.x, M = a.grid_len;
  if (gate_of(a, slot) < 0) return;
  const double* row = a.grid + static_cast<int64_t>(slot) * M;
  const int64_t cs = static_cast<int64_t>(a.rows) * M;
  GridStats st;
  for (int k = 2 * static_cast<int>(threadIdx.x); k < M; k += 2 * 64 * EXP_WAVES) {
    double2 s = make_double2(0.0, 0.0);
    for (int c0 = 0; c0 < a.chunks; c0 += 8) {
      double2 q[8];
#pragma unroll
      for (int u = 0; u < 8; ++u)
        q[u] = *reinterpret_cast<const double2*>(row + min(c0 + u, a.chunks - 1) * cs + k);
#pragma unroll
      for (int u = 0; u < 8; ++u)
        if (c0 + u < a.chunks) {
          s.x += q[u].x;
          s.y += q[u].y;
        }
    }
    st.add(s.x);
    st.add(s.y);
  }
  st.reduce(red, red_ends, M);
  constexpr double MARGIN = 0.9;
  const double h = st.hi, most = MARGIN * st.sum;
  if (threadIdx.x == 0) skip[slot] = h * h <= a.peak_limit * most * most ? 0 : 1;
}

// SG: M / 2048 segments of 1024 lags each way (0: M <= 1024).  Two waves per SIMD:
// with four (two workgroups on a CU) the double-precision transforms spill, 71
// against 67 us at 1000 gates of N = 16384.
template <int SG>
__global__ void __launch_bounds__(64 * EXP_WAVES, 2) expand_grid(FoldArgs a) {
  constexpr int W = EXP_WAVES, NT = 64 * W;
  constexpr bool WIDE = SG == 1, LONG = SG > 1;
  __shared__ __attribute__((aligned(16))) float2 xs[W * XWAVE];
  __shared__ __attribute__((aligned(16))) double sums[LONG ? 1 : 2 * SUB];  // M <= 2048: the grid
  __shared__ float up_s[SG == 0 ? SUB : 1];      // M < 1024: the grid of 1024 points
  // q[n] and q[-n], n < M / 2, and one zero more (before that a transform's parts)
  __shared__ double qp[LONG ? SG * SUB + 1 : SUB + 1], qm[LONG ? SG * SUB + 1 : SUB + 1];
  __shared__ double red[W];
  __shared__ float2 red_ends[W];

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int M = a.grid_len, N = a.n_fft, L = a.code_len, R = N / SUB;
  const int lr = __builtin_ctz(R);
  const double* tw64 = a.twiddle64;
  float* xf = reinterpret_cast<float*>(xs);
  float2* xw = xs + wave * XWAVE;
  double* xd = reinterpret_cast<double*>(xw);

  const int bid = a.gate_list ? static_cast<int>(blockIdx.x) : xcd_block_id();
  const int slot = bid / a.blocks, share = bid % a.blocks;  // of the gate's rounds of classes
  const int g = gate_of(a, slot);
  if (g < 0) return;
  const double* const row = a.grid + static_cast<int64_t>(slot) * M;
  const int64_t cs = static_cast<int64_t>(a.rows) * M;
  const double scale = 1.0 / static_cast<double>(M);

  // With r = conj(DFT) / M the lags n are q[n] = Re r + Im r, q[-n] = Re r - Im r.
  auto put_lag = [&](int n, complex64d f) {
    qp[n] = scale * (f.x - f.y);
    qm[n] = scale * (f.x + f.y);
  };
  // The lags n and m = n_cpx - n in place of F[n], F[m] (F: the transform of the
  // complex points z[2 a] + i z[2 a + 1]).
  auto untangle = [&](int n, complex64d p, complex64d m) {
    complex64d f{0.0, 0.0};
    if (n > 0 && n < L) {
      const complex64d E{0.5 * (p.x + m.x), 0.5 * (p.y - m.y)};
      const complex64d O{0.5 * (p.y + m.y), 0.5 * (m.x - p.x)};
      f = cmuladd(E, twiddle64(tw64, n * (N / M)), O);
    }
    put_lag(n, f);
  };
  auto get = [&](int n) { return complex64d{qp[n], qm[n]}; };

  // the classes 1 ... R / 2 that do not lie on the grid (multiples of `ratio` do),
  // one per wave and round
  const int ratio = N / max(M, SUB), lratio = __builtin_ctz(ratio), rmask = ratio - 1;
  const int n_tasks = ratio == 1 ? 0 : R / 2 - ((R / 2) >> lratio);
  constexpr int PER_ROUND = W;
  auto class_of = [&](int task) { return task + 1 + task / rmask; };

  GridStats st;
  double mean;
  if constexpr (LONG) {
    // ---- the grid (its chunk sums are formed by then), two times SG complex points per thread, and the first pass of the inverse transform:
    // SG-point DFTs over points lg + 1024 j
    complex64d z[2][SG];
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
      for (int j = 0; j < SG; ++j) {
        const double2 s = reinterpret_cast<const double2*>(row)[tid + NT * t + SUB * j];
        z[t][j] = complex64d{s.x, s.y};
        st.add(s.x);
        st.add(s.y);
      }
    st.reduce(red, red_ends, M);
    if (!st.usable(a.peak_limit) || left_out(a, slot)) {  // uniform
      if (share == 0 && tid == 0) redo_gate(a, g);
      return;
    }
    mean = st.sum;
#pragma unroll
    for (int t = 0; t < 2; ++t) {
#pragma unroll
      for (int j = 0; j < SG; ++j) z[t][j] = complex64d{z[t][j].x - mean, z[t][j].y - mean};
      dft_small64(z[t]);
    }
    // class `wave` of the SG 1024-point complex transforms, real and imaginary
    // parts handed over one after the other
    complex64d v[16];
#pragma unroll
    for (int half = 0; half < 2; ++half) {
      if (half == 1) __syncthreads();
#pragma unroll
      for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int k = 0; k < SG; ++k)
          reinterpret_cast<double*>(xs + k * XWAVE)[tid + NT * t] = half == 0 ? z[t][k].x : z[t][k].y;
      __syncthreads();
      if (wave < SG)
#pragma unroll
        for (int j = 0; j < 16; ++j) (half == 0 ? v[j].x : v[j].y) = xd[lane + 64 * j];
    }
    if (wave < SG) {
      wave_lds_sync();
      class_transform64(v, xd, tw64, M / 2, N, wave, lane, [&](int i, complex64d f) {
        const int n = wave + SG * bin_of(i, lane);
        qp[n] = f.x;
        qm[n] = f.y;
      });
    }
    __syncthreads();
    constexpr int NC = SG * SUB;
    for (int n = tid; n <= NC / 2; n += NT) {
      const complex64d A = get(n), B = get(n == 0 ? 0 : NC - n);
      untangle(n, A, B);
      untangle(NC - n, B, A);  // n = 0: the zero past the last lag
    }
  } else {
    // ---- the grid, chunk sums in ascending order
    st = gather_grid(a, row, cs, sums, tid);
    st.reduce(red, red_ends, M);
    if (!st.usable(a.peak_limit) || left_out(a, slot)) {  // uniform
      if (share == 0 && tid == 0) redo_gate(a, g);
      return;
    }
    mean = st.sum;

    // ---- lags: up to conjugation and 1 / M the forward DFT of the real grid,
    // M <= 1024 zero-interleaved to 1024 points (which repeats its spectrum),
    // M = 2048 as complex points
    if (wave == 0) {
      complex64d v[16];
      auto to_lags = [&](int i, complex64d f) {
        qp[bin_of(i, lane)] = f.x;
        qm[bin_of(i, lane)] = f.y;
      };
      if constexpr (WIDE) {
#pragma unroll
        for (int j = 0; j < 16; ++j) {
          const double2 p = reinterpret_cast<const double2*>(sums)[lane + 64 * j];
          v[j] = complex64d{p.x - mean, p.y - mean};
        }
        class_transform64(v, xd, tw64, SUB, N, 0, lane, to_lags);
      } else {
        const int lup = __builtin_ctz(SUB / M), up = (1 << lup) - 1;
#pragma unroll
        for (int j = 0; j < 16; ++j) {
          const int n = lane + 64 * j;
          v[j] = complex64d{(n & up) == 0 ? sums[n >> lup] - mean : 0.0, 0.0};
        }
        class_transform64(v, xd, tw64, SUB, N, 0, lane, to_lags);
        wave_lds_sync();
#pragma unroll
        for (int j = 0; j < 8; ++j) {
          const int n = lane + 64 * j;
          if (n < M / 2) put_lag(n, n > 0 && n < L ? get(n) : complex64d{0.0, 0.0});
        }
        if (lane == 0) put_lag(M / 2, complex64d{0.0, 0.0});
        if (M < SUB) {  // class 0
          wave_lds_sync();
#pragma unroll
          for (int j = 0; j < 16; ++j) {
            const int n = lane + 64 * j, m = SUB - n;
            const double rp = 64 * j < M / 2 ? qp[n] : 0.0;
            const double rm = 64 * (15 - j) < M / 2 ? qm[m] : 0.0;
            v[j] = complex64d{rp + rm, 0.0};
          }
          class_transform64(v, xd, tw64, SUB, N, 0, lane, [&](int i, complex64d F) {
            const int k = bin_of(i, lane);
            const float s = static_cast<float>(F.x - F.y + mean);
            // S >= 0: a rounded zero stays one
            up_s[k] = (k & up) == 0 ? static_cast<float>(sums[k >> lup]) : s < 0.f ? 0.f : s;
          });
        }
      }
    }
    if constexpr (WIDE) {
      __syncthreads();
      static_assert(NT == SUB / 2, "a pair of lags per thread, thread 0 also the middle one");
      const complex64d A = get(tid), B = get(tid == 0 ? SUB / 2 : SUB - tid);
      untangle(tid, A, B);
      untangle(SUB - tid, B, A);  // tid = 0: the zero past the last lag
      if (tid == 0) untangle(SUB / 2, B, B);
    }
  }

  // ---- the classes
  auto grid_bin = [&](int k) -> float {
    if constexpr (LONG) return static_cast<float>(row[k]);
    if constexpr (SG == 0)
      if (M < SUB) return up_s[k];
    return static_cast<float>(sums[k]);
  };
  const bool one_round = n_tasks <= PER_ROUND;
  for (int z0 = PER_ROUND * share; z0 == 0 || z0 < n_tasks; z0 += PER_ROUND * a.blocks) {
    const int n_cls = min(PER_ROUND, n_tasks - z0);  // 0: every bin is on the grid
    const bool mine = wave < n_cls;
    const int k1 = mine ? class_of(z0 + wave) : 0;
    __syncthreads();  // the lags (first round) are written, the regions free
    if (mine) {
      complex64d v[16];
      const complex64d r1 = uniform_twiddle64(tw64, (SUB * k1) & (N - 1));  // W_R^{k1}
#pragma unroll
      for (int j = 0; j < 16; ++j) {  // q[n] and q[n - 1024], n = lane + 64 j
        const int n = lane + 64 * j, m = SUB - n;
        const double rp = LONG || 64 * j < M / 2 ? qp[n] : 0.0;
        const double rm = LONG || 64 * (15 - j) < M / 2 ? qm[m] : 0.0;
        v[j] = complex64d{fma(r1.x, rm, rp), -r1.y * rm};
      }
      if constexpr (LONG) {
#pragma unroll 1
        for (int s = 1; s < SG; ++s) {
          const complex64d f = uniform_twiddle64(tw64, (SUB * k1 * s) & (N - 1));
          const complex64d b = uniform_twiddle64(tw64, (SUB * k1 * (s + 1)) & (N - 1));
#pragma unroll
          for (int j = 0; j < 16; ++j) {
            const int n = lane + 64 * j + SUB * s, m = SUB * (s + 1) - lane - 64 * j;
            const double rp = qp[n], rm = qm[m];
            v[j].x = fma(b.x, rm, fma(f.x, rp, v[j].x));
            v[j].y = fma(-b.y, rm, fma(f.y, rp, v[j].y));
          }
        }
      }
      float* own = reinterpret_cast<float*>(xw);
      class_transform64(v, xd, tw64, N, N, k1, lane, [&](int i, complex64d f) {
        // staged(bin_of(i, lane)), with the register's kd as a constant offset
        const int r4 = lane >> 4;
        const int at = (lane & 15) + 64 * r4 + 16 * ((i >> 2) ^ r4);
        own[at + 256 * (i & 3)] = static_cast<float>(f.x - f.y + mean);
        own[at + 256 * (i & 3) + MIRROR] = static_cast<float>(f.x + f.y + mean);
      });
    }
    __syncthreads();
    {
      // the four bins k = 4 tid + u (+ 4 NT per step) this thread stores: their
      // staged rows, or -1: not of this round, or grid points
      int base[4];
      bool grid_pt[4], mirror[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int k = 4 * tid + u, cl = k & (R - 1);
        grid_pt[u] = (k & rmask) == 0;
        mirror[u] = 2 * cl > R;
        const int kc = mirror[u] ? R - cl : cl;
        const int i = kc - 1 - (kc >> lratio) - z0;
        base[u] = i >= 0 && i < n_cls ? i * 2 * XWAVE + (mirror[u] ? MIRROR : 0) : -1;
        if (grid_pt[u]) base[u] = z0 == 0 ? 0 : -1;
      }
      float* out = a.out + static_cast<int64_t>(g) * N;
      for (int k0 = 4 * tid; k0 < N; k0 += 4 * NT) {
        Float4u s;
        if (a.accumulate) s = *reinterpret_cast<const Float4u*>(out + k0);
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          float x = 0.f;
          if (grid_pt[u]) {
            x = grid_bin((k0 + u) >> lratio);
          } else if (base[u] >= 0) {
            // class R - k1 holds bin -(k1 + R kk), i.e. its own entry 1023 - kk
            const int kb = (k0 + u) >> lr;
            x = xf[base[u] + staged(mirror[u] ? SUB - 1 - kb : kb)];
            x = x < 0.f ? 0.f : x;  // S >= 0: a rounded zero stays one
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
    if (z0 + PER_ROUND * a.blocks < n_tasks) __syncthreads();
  }
}

// ---------------------------------------------------------------------------
// A window of K bins of the N-point spectrum from the summed grid (M <= 2048).
//
// The lags r[n] as in expand_grid, kept in double, then
//   S[k] = r0 + 2 Re sum_{0 < n < L} r[n] z^n,  z = W_N^k,
// by Horner's rule: wave w takes an eighth of the lags for 128 bins, two per lane
// (the lag is one broadcast LDS read for eight multiply-adds), the eighths
// meet in LDS.  4 K L double multiply-adds a gate are little beside a transform
// of N points and need no window-sized table.  1000 pulses x 1000 gates, L = 256, K = 256
// of N = 16384: the pulse pass 430 us, the windows 30; by matrix products (each
// pulse's K L) 1150.  Small calls are faster by products (the rule of the zoom plans).

template <bool WIDE>
__global__ void __launch_bounds__(64 * EXP_WAVES, 4) expand_window(FoldArgs a) {
  __shared__ __attribute__((aligned(16))) double grid[WIDE ? 2 * SUB : SUB];
  __shared__ __attribute__((aligned(16))) complex64d lags[SUB + 1];
  __shared__ __attribute__((aligned(16))) double xd[XWAVE];
  __shared__ double red[EXP_WAVES], sums[EXP_WAVES][128];
  __shared__ float2 red_ends[EXP_WAVES];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int M = a.grid_len, N = a.n_fft, L = a.code_len, K = a.n_bins;
  const int bid = a.gate_list ? static_cast<int>(blockIdx.x) : xcd_block_id();
  const int slot = bid / a.blocks, part = bid % a.blocks;  // of the window, in runs of 128 bins
  const int g = gate_of(a, slot);
  if (g < 0) return;
  const int r0 = K / 128 * part / a.blocks, r1 = K / 128 * (part + 1) / a.blocks;
  const int k0 = a.bin_start[g];
  const double* row = a.grid + static_cast<int64_t>(slot) * M;
  GridStats st = gather_grid(a, row, static_cast<int64_t>(a.rows) * M, grid, tid);
  st.reduce(red, red_ends, M);
  if (!st.usable(a.peak_limit) || left_out(a, slot)) {  // uniform
    if (part == 0 && tid == 0) redo_gate(a, g);
    return;
  }
  const double mean = st.sum;

  // z and z^n0 of the lane's two bins in the run from j0 on (for the first run read
  // before the lags are there)
  const int per = (L - 1 + EXP_WAVES - 1) / EXP_WAVES;
  const int n0 = 1 + wave * per, n1 = min(n0 + per, L);
  complex64d za, zb, sa, sb;
  auto load_factors = [&](int j0) {
    const uint32_t ka = static_cast<uint32_t>(k0 + j0 + lane), kb = ka + 64, mask = N - 1;
    za = twiddle64(a.twiddle64, ka & mask), sa = twiddle64(a.twiddle64, (ka * n0) & mask);
    zb = twiddle64(a.twiddle64, kb & mask), sb = twiddle64(a.twiddle64, (kb * n0) & mask);
  };
  if (wave > 0) load_factors(128 * r0);

  // lags[n] = r[n] = conj(DFT of the grid)[n] / M, 0 < n < L
  const double scale = 1.0 / static_cast<double>(M);
  if (wave == 0) {
    complex64d v[16];
    if constexpr (WIDE) {
#pragma unroll
      for (int j = 0; j < 16; ++j) {
        const double2 p = reinterpret_cast<const double2*>(grid)[lane + 64 * j];
        v[j] = complex64d{p.x - mean, p.y - mean};
      }
      class_transform64(v, xd, a.twiddle64, SUB, N, 0, lane,
                        [&](int i, complex64d f) { lags[bin_of(i, lane)] = f; });
    } else {
      const int lup = __builtin_ctz(SUB / M), up = (1 << lup) - 1;
#pragma unroll
      for (int j = 0; j < 16; ++j) {
        const int n = lane + 64 * j;
        v[j] = complex64d{(n & up) == 0 ? grid[n >> lup] - mean : 0.0, 0.0};
      }
      class_transform64(v, xd, a.twiddle64, SUB, N, 0, lane, [&](int i, complex64d f) {
        lags[bin_of(i, lane)] = complex64d{scale * f.x, -scale * f.y};
      });
    }
  }
  __syncthreads();
  if constexpr (WIDE) {  // from the transform of the complex points grid[2 a] + i grid[2 a + 1]
    auto untangle = [&](int n, complex64d p, complex64d m) {
      const complex64d E{0.5 * (p.x + m.x), 0.5 * (p.y - m.y)};
      const complex64d O{0.5 * (p.y + m.y), 0.5 * (m.x - p.x)};
      const complex64d f = cmuladd(E, twiddle64(a.twiddle64, n * (N / M)), O);
      lags[n] = complex64d{scale * f.x, -scale * f.y};
    };
    const int n = tid == 0 ? SUB / 2 : tid;  // a pair of lags per thread (n = 0 is not used)
    const complex64d A = lags[n], B = lags[SUB - n];
    __syncthreads();
    untangle(n, A, B);
    if (tid != 0) untangle(SUB - n, B, A);
    __syncthreads();
  }

  if (wave == 0) load_factors(128 * r0);  // (no registers for them beside the transform)
  float* out = a.out + static_cast<int64_t>(g) * K;
  for (int j0 = 128 * r0; j0 < 128 * r1; j0 += 128) {
    complex64d ha{0.0, 0.0}, hb{0.0, 0.0};
#pragma unroll 4
    for (int n = n1 - 1; n >= n0; --n) {
      const complex64d r = lags[n];
      ha = cmuladd(r, ha, za);
      hb = cmuladd(r, hb, zb);
    }
    sums[wave][lane] = ha.x * sa.x - ha.y * sa.y;
    sums[wave][lane + 64] = hb.x * sb.x - hb.y * sb.y;
    __syncthreads();
    if (tid < 128) {
      double s = sums[0][tid];
#pragma unroll
      for (int w = 1; w < EXP_WAVES; ++w) s += sums[w][tid];
      const float x = static_cast<float>(fma(2.0, s, mean));
      const float y = x < 0.f ? 0.f : x;  // S >= 0: a rounded zero stays one
      out[j0 + tid] = a.accumulate ? out[j0 + tid] + y : y;
    }
    if (j0 + 128 < 128 * r1) load_factors(j0 + 128);
    __syncthreads();
  }
}

template <int LOGM, int ST, bool WHOLE>
hipError_t launch_grid_w(const FoldArgs& a, hipStream_t s) {
  const dim3 grid(static_cast<unsigned>(a.rows) * static_cast<unsigned>(a.chunks));
  switch (a.waves) {
    case 8: hipLaunchKernelGGL((grid_spectra<LOGM, ST, 8, WHOLE>), grid, dim3(512), 0, s, a); break;
    case 16: hipLaunchKernelGGL((grid_spectra<LOGM, ST, 16, WHOLE>), grid, dim3(1024), 0, s, a); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

template <int ST>
hipError_t launch_grid(const FoldArgs& a, hipStream_t s) {
  const dim3 grid(static_cast<unsigned>(a.rows) * static_cast<unsigned>(a.chunks));
  if (a.partial) {  // the grid is the N bins (N >= 1024; longer codes: N >= 16384)
    switch (a.grid_len) {
      case 1024: return launch_grid_w<10, ST, true>(a, s);
      case 2048: return launch_grid_w<11, ST, true>(a, s);
      case 16384: hipLaunchKernelGGL((grid_long<16, ST, true>), grid, dim3(1024), 0, s, a); break;
      default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
  }
  switch (a.grid_len) {
    case 128: return launch_grid_w<7, ST, false>(a, s);
    case 256: return launch_grid_w<8, ST, false>(a, s);
    case 512: return launch_grid_w<9, ST, false>(a, s);
    case 1024: return launch_grid_w<10, ST, false>(a, s);
    case 2048: return launch_grid_w<11, ST, false>(a, s);
    case 4096: hipLaunchKernelGGL((grid_long<4, ST, false>), grid, dim3(256), 0, s, a); break;
    case 8192: hipLaunchKernelGGL((grid_long<8, ST, false>), grid, dim3(512), 0, s, a); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

hipError_t launch_expand(FoldArgs a, hipStream_t s) {
  // with fewer gates than compute units a gate's rounds of classes go to several
  // workgroups, each forming the lags (N = 65536, one gate: 93 us by one)
  const int ratio = a.n_fft / std::max(a.grid_len, SUB), half = a.n_fft / SUB / 2;
  const int tasks = ratio == 1 ? 0 : half - half / ratio;
  a.blocks = std::max(1, std::min((tasks + EXP_WAVES - 1) / EXP_WAVES, 256 / a.rows));
  const dim3 grid(static_cast<unsigned>(a.rows) * static_cast<unsigned>(a.blocks)), block(64 * EXP_WAVES);
  switch (a.grid_len / (2 * SUB)) {
    case 0: hipLaunchKernelGGL((expand_grid<0>), grid, block, 0, s, a); break;
    case 1: hipLaunchKernelGGL((expand_grid<1>), grid, block, 0, s, a); break;
    case 2: hipLaunchKernelGGL((expand_grid<2>), grid, block, 0, s, a); break;
    case 4: hipLaunchKernelGGL((expand_grid<4>), grid, block, 0, s, a); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

// A run of gates summed on the grid; with probe > 0 in two passes, the second without the gates
// whose first `probe` pulses show a line too strong (a.skip then tells the expansion).
hipError_t sum_grid(FoldArgs& a, int sample_type, int probe, int32_t* early, hipStream_t s) {
  if (probe <= 0 || probe >= a.n_pulses)
    return sample_type == 1 ? launch_grid<1>(a, s) : launch_grid<0>(a, s);
  FoldArgs first = a, rest = a;
  first.n_pulses = probe;
  first.skip = nullptr;
  hipError_t e = sample_type == 1 ? launch_grid<1>(first, s) : launch_grid<0>(first, s);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(probe_grid, dim3(static_cast<unsigned>(a.rows)), dim3(64 * EXP_WAVES), 0, s, a, early);
  e = hipGetLastError();
  if (e != hipSuccess) return e;
  rest.n_pulses = a.n_pulses - probe;
  rest.samples = static_cast<const char*>(a.samples) + probe * a.stride * (sample_type == 1 ? 4 : 8);
  if (a.tx_per_pulse) {
    rest.tx = a.tx + static_cast<int64_t>(2) * probe * a.code_len;
    if (a.code_bits) {
      rest.code_bits = a.code_bits + static_cast<int64_t>(probe) * (a.code_len > SUB ? SUB : 64);
      rest.code_binary = a.code_binary + probe;
    }
  }
  rest.skip = early;
  rest.add = 1;
  a.skip = early;
  return sample_type == 1 ? launch_grid<1>(rest, s) : launch_grid<0>(rest, s);
}

// Sign bits of the call's code rows, if it has room for them.
hipError_t pack_bits(FoldArgs& a, uint32_t* bits, int32_t* binary, hipStream_t s) {
  if (!bits) return hipSuccess;
  const int rows = a.tx_per_pulse ? a.n_pulses : 1;
  if (a.code_len > SUB)
    hipLaunchKernelGGL(pack_long_grid_bits, dim3(static_cast<unsigned>(rows)), dim3(256), 0, s,
                       reinterpret_cast<const float2*>(a.tx), a.code_len, bits, binary);
  else
    hipLaunchKernelGGL(pack_grid_bits, dim3(static_cast<unsigned>((rows + 3) / 4)), dim3(256), 0, s,
                       reinterpret_cast<const float2*>(a.tx), rows, a.code_len, bits, binary);
  a.code_bits = bits;
  a.code_binary = binary;
  return hipGetLastError();
}

hipError_t launch_window(const FoldArgs& a, hipStream_t s) {
  const dim3 grid(static_cast<unsigned>(a.rows) * static_cast<unsigned>(a.blocks)), block(64 * EXP_WAVES);
  if (a.grid_len > SUB)
    hipLaunchKernelGGL((expand_window<true>), grid, block, 0, s, a);
  else
    hipLaunchKernelGGL((expand_window<false>), grid, block, 0, s, a);
  return hipGetLastError();
}

// A grid with points hi, lo and mean is expanded while t = hi / sqrt(mean lo) <= 22 L^(1/4)
// (12 L^(1/4) for L > 1024, whose transforms have a pass more), less by (P / 32)^(1/4) for few
// pulses, over which rounding averages less.  Largest errors over max(S, mean S) there and of
// direct transforms, one line per gate (sets of 40 to 600 gates, complex64):
//   L =  128, P = 100   t =  74: 2.5e-7, 3.8e-7    t = 115: 3.0e-7, 3.9e-7
//   L =  256, P = 100   t =  62: 2.3e-7, 5.8e-7    t = 164: 6.4e-7, 6.0e-7
//   L =  256, P =   8   t =  33: 3.5e-7, 5.6e-7    t =  90: 5.9e-7, 5.3e-7
//   L = 1000, P = 100   t = 124: 4.0e-7, 4.5e-7    t = 233: 8.0e-7, 4.7e-7
//   L = 2000, P = 100   t =  83: 3.1e-7, 5.1e-7    t = 249: 8.5e-7, 5.3e-7
//   L = 4000, P =  60   t =  20: 1.6e-7, 4.1e-7    t = 170: 7.3e-7, 3.9e-7
// Noise alone has t = 20 to 40 at 3 pulses, 2 at 100.
float peak_limit(int code_len, int n_pulses) {
  const float c = code_len > SUB ? 12.f : 22.f;
  return c * c * std::sqrt(static_cast<float>(code_len) * std::min(1.f, static_cast<float>(n_pulses) / 32.f));
}

// Spectra of redone gates whose direct launch split its pulses into chunks, from the partials
// by list slot, the chunks in ascending order.
__global__ void __launch_bounds__(256)
sum_redone(DirectArgs a, int zgroups) {
  const int k = min(max(*a.gate_count, 0), a.n_gates);
  const int chunks = adaptive_chunks(k, zgroups, a.adapt_target, a.adapt_max_chunks, a.adapt_rows);
  if (chunks == 1) return;  // written by the launch itself
  const int64_t n = static_cast<int64_t>(k) * a.n_fft, step = static_cast<int64_t>(gridDim.x) * blockDim.x;
  for (int64_t i = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x; i < n; i += step) {
    float s = 0.f;
    for (int c = 0; c < chunks; ++c) s += a.adapt_partial[c * n + i];
    float* dst = a.out + static_cast<int64_t>(a.gate_list[i / a.n_fft]) * a.n_fft + i % a.n_fft;
    *dst = a.accumulate ? *dst + s : s;
  }
}

// The gates that the expansion has left over, by direct transforms: pulses split over as many
// workgroups as fill the chip for the number of gates there turn out to be, the partials in the
// grid scratch (no longer read).  With none left over the launches find an empty list: 1.6 us
// each.  (Recomputed by the gate's expansion workgroup, without a split, one such gate
// held up a call by 100 times its time.)
hipError_t redo_direct(const FusedArgs& f, hipStream_t s) {
  FusedArgs d = f;
  d.grid_len = 0;
  d.gate_list = f.redo_list;
  d.gate_count = f.redo_count;
  d.chunks = 1;
  d.adapt_partial = reinterpret_cast<float*>(f.grid);
  d.adapt_target = f.redo_target;
  d.adapt_max_chunks = f.redo_max_chunks;
  d.adapt_rows = f.redo_rows;
  hipError_t e = hipSuccess;
  if (d.code_bits) {
    e = launch_pack_code_bits_if(d.tx, d.tx_per_pulse ? d.n_pulses : 1, d.code_len,
                                 const_cast<uint16_t*>(d.code_bits),
                                 const_cast<int32_t*>(d.code_binary), f.redo_count, s);
    if (e != hipSuccess) return e;
  }
  e = launch_fused(d, s);
  if (e != hipSuccess || d.adapt_max_chunks == 1) return e;
  const int zgroups = d.sub_len == SUB ? (1 << d.log2_r) / d.waves_per_block : 1 << d.log2_r;
  hipLaunchKernelGGL(sum_redone, dim3(512), dim3(256), 0, s, static_cast<const DirectArgs&>(d), zgroups);
  return hipGetLastError();
}

// The same for zoom windows, by matrix products (their codes as complex numbers: a pass over all of
// them less).
hipError_t redo_products(const ZoomArgs& z, hipStream_t s) {
  ZoomArgs d = z;
  d.grid_len = 0;
  d.gate_list = z.redo_list;
  d.gate_count = z.redo_count;
  d.code_bits = nullptr;
  d.code_binary = nullptr;
  const hipError_t e = launch_zoom(d, s, true);
  if (e != hipSuccess || d.chunks == 1) return e;
  return launch_reduce_chunks(d.partial, d.out, static_cast<int64_t>(d.n_gates) * d.n_bins, d.chunks,
                              d.accumulate, d.n_bins, d.gate_list, d.gate_count, s);
}

}  // namespace

hipError_t launch_folded(const FusedArgs& f, hipStream_t s) {
  FoldArgs a{};
  a.samples = f.samples;
  a.tx = f.tx;
  a.twiddle = f.twiddle;
  a.twiddle64 = f.twiddle64;
  a.gain = f.grid_gain;
  a.grid = f.grid;
  a.partial = f.grid_len == f.n_fft ? reinterpret_cast<float*>(f.grid) : nullptr;
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
  a.redo_list = f.redo_list;
  a.redo_count = a.partial ? nullptr : f.redo_count;
  a.peak_limit = peak_limit(a.code_len, a.n_pulses);
  hipError_t e = pack_bits(a, f.grid_bits, f.grid_binary, s);
  if (e != hipSuccess) return e;
  if (a.grid_len == a.n_fft) {  // every bin is on the grid: partials by gate, no expansion
    a.rows = f.n_gates;
    e = f.sample_type == 1 ? launch_grid<1>(a, s) : launch_grid<0>(a, s);
    if (e == hipSuccess && a.chunks > 1 && !f.grid_defer)
      e = launch_reduce_chunks(a.partial, a.out, static_cast<int64_t>(f.n_gates) * f.n_fft, a.chunks,
                               a.accumulate, a.n_fft, a.gate_list, a.gate_count, s);
    return e;
  }
  if (f.grid_gain_missing) {
    hipLaunchKernelGGL(build_gains, dim3(static_cast<unsigned>((a.grid_len + 255) / 256)), dim3(256), 0,
                       s, a.twiddle64, a.n_fft, a.grid_len, f.grid_gain);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  // as many gates at a time as the scratch holds
  for (int32_t s0 = 0; s0 < f.n_gates; s0 += f.grid_rows) {
    a.slot0 = s0;
    a.rows = std::min(f.n_gates - s0, f.grid_rows);
    e = sum_grid(a, f.sample_type, f.probe_pulses, f.redo_early, s);
    FoldArgs x = a;
    if (e == hipSuccess && a.grid_len > 2 * SUB && a.chunks > 1) {
      // a long grid's chunk partials by a launch of their own, behind them (the expansion's
      // workgroups have too few threads for their latency: 80 pulses of one gate, 60 us more)
      const int64_t elems = static_cast<int64_t>(a.rows) * a.grid_len;
      x.grid = a.grid + a.chunks * elems;
      x.chunks = 1;
      const unsigned blocks = static_cast<unsigned>(std::min<int64_t>((elems + 255) / 256, 4096));
      hipLaunchKernelGGL(sum_chunks, dim3(blocks), dim3(256), 0, s, a.grid, x.grid, elems, a.chunks);
      e = hipGetLastError();
    }
    if (e == hipSuccess)
      e = launch_expand(x, s);
    if (e == hipSuccess) e = redo_direct(f, s);
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

hipError_t launch_zoom_folded(const ZoomArgs& z, hipStream_t s) {
  FoldArgs a{};
  a.samples = z.samples;
  a.tx = z.tx;
  a.twiddle = z.twiddle;
  a.twiddle64 = z.twiddle64;
  a.gain = z.grid_gain;
  a.grid = z.grid;
  a.out = z.out;
  a.stride = z.stride;
  a.n_fft = z.n_fft;
  a.grid_len = z.grid_len;
  a.code_len = z.code_len;
  a.n_gates = z.n_gates;
  a.gate_step = z.gate_step;
  a.first_gate = z.first_gate;
  a.n_pulses = z.n_pulses;
  a.chunks = z.grid_chunks;
  a.waves = z.grid_waves;
  a.tx_per_pulse = z.tx_per_pulse;
  a.accumulate = z.accumulate;
  a.gate_list = z.gate_list;
  a.gate_count = z.gate_count;
  a.redo_list = z.redo_list;
  a.redo_count = z.redo_count;
  // (BF16 products round 16 times as coarsely)
  a.peak_limit = (z.precision == 1 ? 1.f : 256.f) * peak_limit(a.code_len, a.n_pulses);
  a.bin_start = z.bin_start;
  a.n_bins = z.n_bins;
  hipError_t e = pack_bits(a, z.grid_bits, z.grid_binary, s);
  for (int32_t s0 = 0; e == hipSuccess && s0 < z.n_gates; s0 += z.grid_rows) {
    a.slot0 = s0;
    a.rows = std::min(z.n_gates - s0, z.grid_rows);
    // a workgroup or more per gate, up to two per CU (each forms the gate's lags)
    a.blocks = std::max(1, std::min(z.n_bins / 128, 512 / a.rows));
    e = sum_grid(a, z.sample_type, z.probe_pulses, z.redo_early, s);
    if (e == hipSuccess) e = launch_window(a, s);
    if (e == hipSuccess) e = redo_products(z, s);
  }
  return e;
}

}  // namespace ispl
