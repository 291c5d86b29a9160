// Device helpers shared by several kernel files (HIP only; never included by
// host-only translation units).
#pragma once

#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

namespace ispl {

// Sample i of a row: complex64, or an int16 (re, im) pair (exact in float).
__device__ __forceinline__ float2 load_any_sample(const void* base, int32_t sample_type,
                                                  int64_t i) {
  if (sample_type == 1) {
    const uint32_t r = reinterpret_cast<const uint32_t*>(base)[i];
    return make_float2(static_cast<float>(static_cast<int16_t>(r & 0xffffu)),
                       static_cast<float>(static_cast<int32_t>(r) >> 16));
  }
  return reinterpret_cast<const float2*>(base)[i];
}

// The exponent of a column whose largest |x|^2 and |c|^2 are mx and mc (see below).
__device__ __forceinline__ int column_exponent(float mx, float mc) {
  int e = 0;
  const float m = sqrtf(mx) * sqrtf(mc);
  if (m > 0.f && isfinite(m)) {
    int ex;
    frexpf(m, &ex);  // m < 2^ex
    e = 14 - ex;
  }
  return max(-60, min(60, e));
}

// FP16 column exponent of pulse p, computed by one workgroup of 256 threads:
// the e with max|x| max|c| 2^e < 2^14 over the samples [lo, hi) of the pulse
// row that some gate reads and over the pulse's code, so that no split FP16
// value of the zoom DFT overflows and the low halves stay normal down to about
// 2^-17 of that maximum.  Clamped to [-60, 60]; 0 for an all-zero pulse.
__device__ __forceinline__ void pulse_exponent_block(const void* __restrict__ samples,
                                                     int32_t sample_type,
                                                     const float* __restrict__ tx,
                                                     int64_t stride, int64_t lo, int64_t hi,
                                                     int32_t code_len, int32_t tx_per_pulse,
                                                     int p, int32_t* __restrict__ exps) {
  __shared__ float red[2][4];
  float mx = 0.f, mc = 0.f;
  const int64_t base = static_cast<int64_t>(p) * stride;
  // eight loads in flight per thread (indices clamped into the span, the
  // clamped ones counted as zero); the maximum does not depend on the order
  constexpr int U = 8;
  for (int64_t i0 = lo + threadIdx.x; i0 < hi; i0 += 256 * U) {
    float2 x[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int64_t i = i0 + 256 * u;
      x[u] = load_any_sample(samples, sample_type, base + (i < hi ? i : hi - 1));
    }
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (i0 + 256 * u < hi) mx = fmaxf(mx, x[u].x * x[u].x + x[u].y * x[u].y);
  }
  const float2* txp = reinterpret_cast<const float2*>(tx) +
                      (tx_per_pulse ? static_cast<int64_t>(p) * code_len : 0);
  for (int n0 = threadIdx.x; n0 < code_len; n0 += 256 * U) {
    float2 c[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int n = n0 + 256 * u;
      c[u] = txp[n < code_len ? n : code_len - 1];
    }
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (n0 + 256 * u < code_len) mc = fmaxf(mc, c[u].x * c[u].x + c[u].y * c[u].y);
  }
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) {
    mx = fmaxf(mx, __shfl_xor(mx, off));
    mc = fmaxf(mc, __shfl_xor(mc, off));
  }
  if ((threadIdx.x & 63) == 0) {
    red[0][threadIdx.x >> 6] = mx;
    red[1][threadIdx.x >> 6] = mc;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    mx = fmaxf(fmaxf(red[0][0], red[0][1]), fmaxf(red[0][2], red[0][3]));
    mc = fmaxf(fmaxf(red[1][0], red[1][1]), fmaxf(red[1][2], red[1][3]));
    exps[p] = column_exponent(mx, mc);
  }
}

// Largest |c|^2 and |x|^2 of a lane's samples of two gates at0 and at1 (the type known, so that all
// loads of a step are in flight).
template <int ST>
__device__ __forceinline__ void gate_maxima(const void* __restrict__ samples,
                                            const float2* __restrict__ txp, int64_t at0, int64_t at1,
                                            int32_t code_len, int lane, float& mc, float& m0, float& m1) {
  constexpr int U = 4;
  for (int n0 = lane; n0 < code_len; n0 += 64 * U) {
    float2 c[U], x[U], y[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {  // (past the end the last sample again)
      const int n = min(n0 + 64 * u, code_len - 1);
      c[u] = txp[n];
      x[u] = load_any_sample(samples, ST, at0 + n);
      y[u] = load_any_sample(samples, ST, at1 + n);
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      mc = fmaxf(mc, c[u].x * c[u].x + c[u].y * c[u].y);
      m0 = fmaxf(m0, x[u].x * x[u].x + x[u].y * x[u].y);
      m1 = fmaxf(m1, y[u].x * y[u].x + y[u].y * y[u].y);
    }
  }
}

// The same for each gate by itself, exps[n_gates p + g], so that a gate far weaker than the strongest
// of its pulse keeps its bits: the gates 8 group ... 8 group + 7 of pulse p, two per wave.
__device__ __forceinline__ void gate_exponents_block(const void* __restrict__ samples,
                                                     int32_t sample_type,
                                                     const float* __restrict__ tx, int64_t stride,
                                                     int32_t first_gate, int32_t gate_step,
                                                     int32_t n_gates, int32_t code_len,
                                                     int32_t tx_per_pulse, int p, int group,
                                                     int32_t* __restrict__ exps) {
  const int lane = threadIdx.x & 63, g0 = 8 * group + 2 * static_cast<int>(threadIdx.x >> 6);
  if (g0 >= n_gates) return;  // whole waves, no barrier
  const float2* txp = reinterpret_cast<const float2*>(tx) +
                      (tx_per_pulse ? static_cast<int64_t>(p) * code_len : 0);
  const int64_t at0 = static_cast<int64_t>(p) * stride + first_gate + static_cast<int64_t>(g0) * gate_step;
  const int64_t at1 = g0 + 1 < n_gates ? at0 + gate_step : at0;
  float mc = 0.f, m0 = 0.f, m1 = 0.f;
  if (sample_type == 1)
    gate_maxima<1>(samples, txp, at0, at1, code_len, lane, mc, m0, m1);
  else
    gate_maxima<0>(samples, txp, at0, at1, code_len, lane, mc, m0, m1);
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) {
    mc = fmaxf(mc, __shfl_xor(mc, off));
    m0 = fmaxf(m0, __shfl_xor(m0, off));
    m1 = fmaxf(m1, __shfl_xor(m1, off));
  }
  if (lane < 2 && g0 + lane < n_gates)
    exps[static_cast<int64_t>(n_gates) * p + g0 + lane] = column_exponent(lane == 0 ? m0 : m1, mc);
}

// Sign bits of pulse p's code for the zoom DFT, by one workgroup of 256
// threads: bit b of word w of bits[p] is set when code[32 w + b] == -1 + 0i
// (positions past L read as +1), and binary[p] = 1 when every code of the row
// is exactly +-1 + 0i (0: the zoom then reads the row as complex codes).
// words * 32 must be a multiple of 64 (one ballot of a wave gives two words).
// With a code shared by all pulses only row 0 exists (p == 0 writes it).
__device__ __forceinline__ void code_bits_block(const float* __restrict__ tx, int32_t code_len,
                                                int32_t tx_per_pulse, int32_t words, int p,
                                                uint32_t* __restrict__ bits,
                                                int32_t* __restrict__ binary) {
  if (!tx_per_pulse && p != 0) return;  // uniform over the workgroup
  const float2* txp = reinterpret_cast<const float2*>(tx) +
                      (tx_per_pulse ? static_cast<int64_t>(p) * code_len : 0);
  const int lane = threadIdx.x & 63;
  bool ok = true;
  for (int n0 = 64 * (threadIdx.x >> 6); n0 < 32 * words; n0 += 256) {  // wave-uniform
    const int n = n0 + lane;
    bool neg = false;
    if (n < code_len) {
      const float2 c = txp[n];
      ok = ok && c.y == 0.f && (c.x == 1.f || c.x == -1.f);
      neg = c.x < 0.f;
    }
    const uint64_t m = __ballot(neg);
    if (lane == 0) {
      uint32_t* w = bits + static_cast<int64_t>(p) * words + n0 / 32;
      w[0] = static_cast<uint32_t>(m);
      w[1] = static_cast<uint32_t>(m >> 32);
    }
  }
  ok = __syncthreads_and(ok);
  if (threadIdx.x == 0) binary[p] = ok ? 1 : 0;
}

}  // namespace ispl
