// Window-proposal network of the learned zoom: training kernels (FP32: the
// 32 -> 32 layers on the matrix cores' FP32 products, the rest on the vector ALUs).
//
// The network maps one gate's coarse spectrum feature
// x[t] = log(max(S[t] / mean S, 1e-30)), t < T = 1024, to one logit per coarse bin through four circular 7-tap 1-D
// convolutions, 1 -> 32 -> 32 -> 32 -> 1 channels with ReLU after the first
// three.  Training minimises the softmax cross entropy against a two-hot
// target at the line's coarse position u (1 - frac(u) on floor(u), frac(u)
// on floor(u) + 1, modulo T).  Per-gate weight gradients are summed over the
// batch in a fixed order (no atomics), so a training step is bit-reproducible.

#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include "ispl_internal.h"

namespace ispl {
namespace {

constexpr int T = NET_LEN;      // 1024 positions
constexpr int TAPS = 7;
constexpr int PAD = 3;
constexpr int NT = 256;         // threads: four consecutive positions each
static_assert(T == 4 * NT, "one thread per four positions");

__device__ __forceinline__ float4 ld4(const float* p) { return *reinterpret_cast<const float4*>(p); }

// The 10 values v[(4 j - 3 + i) mod T], i < 10, of row `row` (length T, in LDS).
__device__ __forceinline__ void window10(const float* row, int j, float (&w)[10]) {
  const float4 l = ld4(row + ((4 * j - 4) & (T - 1)));
  const float4 m = ld4(row + 4 * j);
  const float4 r = ld4(row + ((4 * j + 4) & (T - 1)));
  w[0] = l.y; w[1] = l.z; w[2] = l.w;
  w[3] = m.x; w[4] = m.y; w[5] = m.z; w[6] = m.w;
  w[7] = r.x; w[8] = r.y; w[9] = r.z;
}

// ---------------------------------------------------------------------------
// 32 -> 32 layers and their data gradients as FP32 matrix products
// (v_mfma_f32_32x32x2_f32): rows are the 32 output channels, columns 32
// positions, the reduction 16 channel pairs x 7 taps.
//
// One workgroup of eight waves per 256 positions of a gate, one 32-position
// tile per wave.  The inputs (with the 3 + 3 neighbours, wrapped) and the
// weights lie in LDS; a step's operands are one 4-byte read each, which the
// 64-cycle products of four waves per SIMD (two workgroups per CU) hide.  At 256
// gates a layer takes 43 to 46 us (128-position workgroups 50; on the vector ALUs, one
// workgroup per gate, 150 to 230), the products alone 24, its bytes 15.
// Weight rows have an odd pitch, input rows one of half the banks.
constexpr int TILE = 256;
constexpr int TNT = 2 * TILE;      // threads: a wave per 32 positions
constexpr int ROW = 288;           // pitch of an input row; entry i is position t0 - 4 + i
constexpr int USED = TILE + 8;     // entries of it
constexpr int WPITCH = 32 * TAPS + 1;

typedef float f32x16t __attribute__((ext_vector_type(16)));

// Row (channel) of accumulator i in lane half h.
__device__ __forceinline__ int acc_row(int i, int h) { return 8 * (i >> 2) + 4 * h + (i & 3); }

enum ConvKind {
  kFirstTwo,  // layers 1 and 2: in = x [B][T]; layer 1 is also written to a1
  kForward,   // a 32 -> 32 layer with ReLU
  kData       // its data gradient: in = dz, da[ci][t] = sum_{co,k} W[co][ci][k] dz[co][t - k + 3],
              // out = da where a1 (the layer's input activation) > 0, else 0
};

template <ConvKind KIND>
__global__ void __launch_bounds__(TNT) conv_tile(const float* __restrict__ in,
                                                const float* __restrict__ params, int w_off,
                                                float* __restrict__ a1, float* __restrict__ out) {
  __shared__ __attribute__((aligned(16))) float in_s[32][ROW];
  __shared__ float w_s[32 * WPITCH];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int b = blockIdx.x / (T / TILE), t0 = TILE * (blockIdx.x % (T / TILE));
  const float* W = params + w_off;
  const int64_t rows = static_cast<int64_t>(b) * 32 * T;

#pragma unroll
  for (int i = 0; i < 32 * 32 * TAPS / TNT; ++i) {
    const int e = tid + TNT * i, r = e / (32 * TAPS);
    w_s[e + r] = W[e];
  }
  if constexpr (KIND == kFirstTwo) {
    __shared__ float x_s[USED + 8];  // entry i is position t0 - 8 + i
    if (tid < USED + 8) x_s[tid] = in[static_cast<int64_t>(b) * T + ((t0 - 8 + tid) & (T - 1))];
    __syncthreads();
    const float* W1 = params;
    for (int e = tid; e < 32 * USED; e += TNT) {
      const int co = e / USED, i = e % USED;
      float z = W1[32 * TAPS + co];
#pragma unroll
      for (int k = 0; k < TAPS; ++k) z = fmaf(W1[co * TAPS + k], x_s[i + k + 1], z);
      z = fmaxf(z, 0.f);
      in_s[co][i] = z;
      if (i >= 4 && i < 4 + TILE) a1[rows + co * T + t0 - 4 + i] = z;
    }
  } else {
#pragma unroll
    for (int u = 0; u < (32 * USED / 4 + TNT - 1) / TNT; ++u) {
      const int e = tid + TNT * u;
      if (e < 32 * USED / 4) {
        const int r = e / (USED / 4), i = 4 * (e % (USED / 4));
        *reinterpret_cast<float4*>(&in_s[r][i]) = ld4(in + rows + r * T + ((t0 - 4 + i) & (T - 1)));
      }
    }
  }
  __syncthreads();

  const int col = lane & 31, h = lane >> 5;
  f32x16t acc;
#pragma unroll
  for (int i = 0; i < 16; ++i) acc[i] = KIND == kData ? 0.f : W[32 * 32 * TAPS + acc_row(i, h)];
  // product step (pair c, tap k): channel 2 c + h of both operands
  const float* wp = w_s + (KIND == kData ? h * WPITCH + col * TAPS : col * WPITCH + h * TAPS);
  const float* ip = &in_s[h][32 * wave + col];
#pragma unroll 4
  for (int c = 0; c < 16; ++c)
#pragma unroll
    for (int k = 0; k < TAPS; ++k)
      acc = __builtin_amdgcn_mfma_f32_32x32x2f32(
          wp[(KIND == kData ? 2 * WPITCH : 2 * TAPS) * c + k],
          ip[2 * ROW * c + (KIND == kData ? 7 - k : 1 + k)], acc, 0, 0, 0);
  const int64_t at = rows + t0 + 32 * wave + col;
#pragma unroll
  for (int i = 0; i < 16; ++i) {
    const int64_t o = at + acc_row(i, h) * T;
    if constexpr (KIND == kData)
      out[o] = a1[o] > 0.f ? acc[i] : 0.f;
    else
      out[o] = fmaxf(acc[i], 0.f);
  }
}

// Sums over the 64 lanes of 64 values per lane, value i left in lane i: each
// step hands half of the values to the lane's partner (63 exchanges, not 6 x 64).
template <int N = 32>
__device__ __forceinline__ float lane_sums(float (&v)[64], int lane) {
  const bool up = (lane & N) != 0;
#pragma unroll
  for (int i = 0; i < N; ++i) {
    const float keep = up ? v[i + N] : v[i], send = up ? v[i] : v[i + N];
    v[i] = keep + __shfl_xor(send, N);
  }
  if constexpr (N > 1)
    return lane_sums<N / 2>(v, lane);
  else
    return v[0];
}

// ---------------------------------------------------------------------------
// Weight gradients dW[co][ci][k] = sum_t dz[co][t] a[ci][(t + k - 3) mod T],
// db[co] = sum_t dz[co][t] of one gate, written to that gate's row of the partial
// buffer (layer segment at w_off, flat parameter order).
//
// A 32 -> 32 layer: seven FP32 matrix products (one per tap) over the
// positions, all seven accumulators in registers.  Wave w takes positions 128 w ...
// 128 w + 127, lane half h their half 64 h ..., so that each lane walks its own
// rows of dz and a in order: 16-byte loads, no LDS, and the taps' operands are a
// sliding window over a in registers.  At 256 gates the three layers take 100 us (the
// vector ALU form with a (co, ci) pair's taps per thread 530), of which the products are
// 48; accumulators leave two waves per SIMD, so a workgroup's first loads are not hidden.
constexpr int WG_WAVES = 8;

__device__ void weight_grad32(const float* __restrict__ dz, const float* __restrict__ a,
                              float* __restrict__ out, float (&buf)[2][WG_WAVES][1024]) {
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int r = lane & 31, h = lane >> 5;
  const int t0 = 128 * wave + 64 * h;
  const float* dr = dz + r * T + t0;
  const float* ar = a + r * T;
  f32x16t acc[TAPS];
#pragma unroll
  for (int k = 0; k < TAPS; ++k)
#pragma unroll
    for (int i = 0; i < 16; ++i) acc[k][i] = 0.f;
  float db = 0.f;
  // sixteen positions at a time, the next ones in flight
  float w[22], next[16], dv[16], dn[16];  // w[i]: position base - 3 + i of a
  auto load16 = [](float (&to)[16], const float* from) {
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const float4 f = ld4(from + 4 * q);
      to[4 * q] = f.x, to[4 * q + 1] = f.y, to[4 * q + 2] = f.z, to[4 * q + 3] = f.w;
    }
  };
  {
    const float4 l = ld4(ar + ((t0 - 4) & (T - 1)));
    w[0] = l.y, w[1] = l.z, w[2] = l.w;
  }
  load16(next, ar + t0);
  load16(dn, dr);
#pragma unroll 1
  for (int it = 0; it < 4; ++it) {
#pragma unroll
    for (int i = 0; i < 16; ++i) w[3 + i] = next[i], dv[i] = dn[i];
    load16(next, ar + ((t0 + 16 * it + 16) & (T - 1)));
    if (it < 3) load16(dn, dr + 16 * it + 16);
#pragma unroll
    for (int j = 0; j < 16; ++j) {
      if (j == 13) w[19] = next[0], w[20] = next[1], w[21] = next[2];
#pragma unroll
      for (int k = 0; k < TAPS; ++k)
        acc[k] = __builtin_amdgcn_mfma_f32_32x32x2f32(dv[j], w[j + k], acc[k], 0, 0, 0);
      db += dv[j];
    }
    w[0] = w[16], w[1] = w[17], w[2] = w[18];
  }
  // the waves' sums, tap by tap through LDS
  float sum[TAPS][2];
#pragma unroll
  for (int k = 0; k < TAPS; ++k) {
    float (&half)[WG_WAVES][1024] = buf[k & 1];
#pragma unroll
    for (int i = 0; i < 16; ++i) half[wave][32 * acc_row(i, h) + r] = acc[k][i];
    __syncthreads();
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      float s = 0.f;
#pragma unroll
      for (int w = 0; w < WG_WAVES; ++w) s += half[w][tid + 512 * u];
      sum[k][u] = s;
    }
  }
  db += __shfl_xor(db, 32);
  __syncthreads();  // (both halves read)
  float* flat = &buf[0][0][0];
  float* bias = &buf[1][0][0];
  static_assert(32 * 32 * TAPS <= WG_WAVES * 1024, "a gate's weights in one half");
#pragma unroll
  for (int k = 0; k < TAPS; ++k)
#pragma unroll
    for (int u = 0; u < 2; ++u) flat[(tid + 512 * u) * TAPS + k] = sum[k][u];
  if (lane < 32) bias[32 * wave + lane] = db;
  __syncthreads();
  for (int i = tid; i < 32 * 32 * TAPS; i += 64 * WG_WAVES) out[i] = flat[i];
  if (tid < 32) {
    float s = 0.f;
#pragma unroll
    for (int w = 0; w < WG_WAVES; ++w) s += bias[32 * w + tid];
    out[32 * 32 * TAPS + tid] = s;
  }
}

// Layer 1 (one input channel): four output channels per wave, 16 positions per lane.
__device__ void weight_grad1(const float* __restrict__ dz, const float* __restrict__ x,
                             float* __restrict__ out) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  float v[64];  // 8 values (taps, bias) of 4 channels; the upper half stays zero
#pragma unroll
  for (int i = 0; i < 64; ++i) v[i] = 0.f;
#pragma unroll
  for (int s = 0; s < 4; ++s) {
    const int j = lane + 64 * s;
    float w[10];
    window10(x, j, w);
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      const float4 d4 = ld4(dz + (4 * wave + c) * T + 4 * j);
      const float d[4] = {d4.x, d4.y, d4.z, d4.w};
#pragma unroll
      for (int m = 0; m < 4; ++m) {
#pragma unroll
        for (int k = 0; k < TAPS; ++k) v[8 * c + k] = fmaf(d[m], w[m + k], v[8 * c + k]);
        v[8 * c + 7] += d[m];
      }
    }
  }
  const float s = lane_sums(v, lane);
  const int co = 4 * wave + (lane >> 3), k = lane & 7;
  if (lane < 32) out[k < TAPS ? co * TAPS + k : 32 * TAPS + co] = s;
}

// Layers 3, 2 and 1 in one launch (the long ones first).
__global__ void __launch_bounds__(64 * WG_WAVES)
weight_grads(const float* __restrict__ dz3, const float* __restrict__ a2,
             const float* __restrict__ dz2, const float* __restrict__ a1,
             const float* __restrict__ dz1, const float* __restrict__ x, int batch, int off3,
             int off2, int off1, int n_params, float* __restrict__ part) {
  __shared__ float buf[2][WG_WAVES][1024];
  const int layer = blockIdx.x / batch, b = blockIdx.x % batch;
  const int64_t rows = static_cast<int64_t>(b) * 32 * T;
  float* out = part + static_cast<int64_t>(b) * n_params;
  if (layer == 2)
    weight_grad1(dz1 + rows, x + static_cast<int64_t>(b) * T, out + off1);
  else
    weight_grad32((layer == 0 ? dz3 : dz2) + rows, (layer == 0 ? a2 : a1) + rows,
                  out + (layer == 0 ? off3 : off2), buf);
}

// Fixed-order block reduction helpers (256 threads).
__device__ float block_sum(float v, float* red) {
  for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off);
  __syncthreads();
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
  __syncthreads();
  return (red[0] + red[1]) + (red[2] + red[3]);
}

// Sum or maximum over a workgroup of 16 waves, in a fixed order.
template <bool MAX>
__device__ __forceinline__ float block16(float v, float* red) {
  for (int off = 32; off > 0; off >>= 1) {
    const float o = __shfl_xor(v, off);
    v = MAX ? fmaxf(v, o) : v + o;
  }
  __syncthreads();
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
  __syncthreads();
  float r = red[0];
#pragma unroll
  for (int i = 1; i < 16; ++i) r = MAX ? fmaxf(r, red[i]) : r + red[i];
  return r;
}

// Layer 4 (32 -> 1) of one gate: logits; with GRAD instead the softmax cross
// entropy against the two-hot target at coarse position target_pos[b] (loss[b]) and,
// with dz4 = softmax - target, the gradients of the layer's weights (into the gate's
// partial row) and its data gradient dz3, in one pass over a3 each: four
// kernels and two passes of 128 KB per gate less.  1024 threads: four positions of
// eight channels each.
template <bool GRAD>
__global__ void __launch_bounds__(1024) last_layer(const float* __restrict__ a3,
                                                   const float* __restrict__ params, int w_off,
                                                   const float* __restrict__ target_pos,
                                                   float* __restrict__ logits,
                                                   float* __restrict__ loss, int n_params,
                                                   float* __restrict__ part,
                                                   float* __restrict__ dz3) {
  __shared__ __attribute__((aligned(16))) float z_s[4][T];
  __shared__ __attribute__((aligned(16))) float d_s[T];
  __shared__ float red[16], wsum[16][64];
  const int b = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int j = tid & (NT - 1), grp = __builtin_amdgcn_readfirstlane(tid / NT);
  const float* W = params + w_off;
  const int64_t rows = static_cast<int64_t>(b) * 32 * T;
  const float* a = a3 + rows + 8 * grp * T;
  const float* wg = W + 8 * grp * TAPS;
  {
    float acc[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int c = 0; c < 8; ++c) {
      float w[10];
      window10(a + c * T, j, w);
#pragma unroll
      for (int k = 0; k < TAPS; ++k)
#pragma unroll
        for (int m = 0; m < 4; ++m) acc[m] = fmaf(wg[c * TAPS + k], w[m + k], acc[m]);
    }
    *reinterpret_cast<float4*>(&z_s[grp][4 * j]) = make_float4(acc[0], acc[1], acc[2], acc[3]);
  }
  __syncthreads();
  const float z = W[32 * TAPS] + ((z_s[0][tid] + z_s[1][tid]) + (z_s[2][tid] + z_s[3][tid]));
  if constexpr (!GRAD) {
    logits[static_cast<int64_t>(b) * T + tid] = z;
  } else {
    const float mx = block16<true>(z, red);
    const float e = expf(z - mx);
    const float sum = block16<false>(e, red);
    const float u = target_pos[b];
    const float fl = floorf(u);
    const float f = u - fl;
    const int lo = static_cast<int>(fl) & (T - 1), hi = (lo + 1) & (T - 1);
    const float tgt = (tid == lo ? 1.f - f : 0.f) + (tid == hi ? f : 0.f);
    d_s[tid] = e * (1.f / sum) - tgt;
    z_s[0][tid] = z;  // (read by this thread alone before)
    __syncthreads();
    if (tid == 0) {
      const float lse = mx + logf(sum);  // -log p[t] = lse - z[t]
      loss[b] = (1.f - f) * (lse - z_s[0][lo]) + f * (lse - z_s[0][hi]);
    }
    float dw[10];  // dw[i] = dz4[4 j - 3 + i]
    window10(d_s, j, dw);
    float v[64];   // 7 taps of 8 channels; 56: the bias
#pragma unroll
    for (int i = 0; i < 64; ++i) v[i] = 0.f;
    float* dst = dz3 + rows + 8 * grp * T;
#pragma unroll
    for (int c = 0; c < 8; ++c) {
      float w[10];
      window10(a + c * T, j, w);
      float o[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int k = 0; k < TAPS; ++k)
#pragma unroll
        for (int m = 0; m < 4; ++m) {
          v[c * TAPS + k] = fmaf(dw[m + 3], w[m + k], v[c * TAPS + k]);
          o[m] = fmaf(wg[c * TAPS + k], dw[m - k + 6], o[m]);
        }
      *reinterpret_cast<float4*>(dst + c * T + 4 * j) =
          make_float4(w[3] > 0.f ? o[0] : 0.f, w[4] > 0.f ? o[1] : 0.f, w[5] > 0.f ? o[2] : 0.f,
                      w[6] > 0.f ? o[3] : 0.f);
    }
    v[56] = (dw[3] + dw[4]) + (dw[5] + dw[6]);
    wsum[wave][lane] = lane_sums(v, lane);
    __syncthreads();
    if (tid < 32 * TAPS + 1) {  // waves 4 grp ... 4 grp + 3 hold channels 8 grp ...
      const int q = tid < 32 * TAPS ? tid / 56 : 0, i = tid < 32 * TAPS ? tid % 56 : 56;
      part[static_cast<int64_t>(b) * n_params + w_off + tid] =
          (wsum[4 * q][i] + wsum[4 * q + 1][i]) + (wsum[4 * q + 2][i] + wsum[4 * q + 3][i]);
    }
  }
}

// grad[i] = (1 / B) sum_b part[b][i], and in the last workgroup the mean of the
// losses: 32 columns and 8 interleaved runs of rows per workgroup, the runs'
// sums added in order.  (One thread per column has 59 workgroups walk the
// rows: 62 us at 256 rows.)
__global__ void __launch_bounds__(256) mean_rows(const float* __restrict__ part, int rows,
                                                 int cols, const float* __restrict__ loss,
                                                 float* __restrict__ out,
                                                 float* __restrict__ loss_mean) {
  __shared__ float run_s[8][32];
  const int c = threadIdx.x & 31, run = threadIdx.x >> 5;
  const bool of_loss = blockIdx.x == gridDim.x - 1;
  const int i = of_loss ? c : 32 * static_cast<int>(blockIdx.x) + c, n = of_loss ? 1 : cols;
  const float* src = of_loss ? loss : part;
  float s = 0.f;
  if (i < n) {
    int r = run;
    for (; r + 24 < rows; r += 32) {
      float q[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) q[u] = src[static_cast<int64_t>(r + 8 * u) * n + i];
#pragma unroll
      for (int u = 0; u < 4; ++u) s += q[u];
    }
    for (; r < rows; r += 8) s += src[static_cast<int64_t>(r) * n + i];
  }
  run_s[run][c] = s;
  __syncthreads();
  if (run == 0 && i < n) {
    s = run_s[0][c];
#pragma unroll
    for (int u = 1; u < 8; ++u) s += run_s[u][c];
    (of_loss ? loss_mean : out)[i] = s / static_cast<float>(rows);
  }
}

__global__ void __launch_bounds__(256) adam_update(float* __restrict__ params,
                                                   const float* __restrict__ grad,
                                                   float* __restrict__ m, float* __restrict__ v,
                                                   int n, float lr, float beta1, float beta2,
                                                   float eps, float corr1, float corr2) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const float g = grad[i];
  const float mi = beta1 * m[i] + (1.f - beta1) * g;
  const float vi = beta2 * v[i] + (1.f - beta2) * g * g;
  m[i] = mi;
  v[i] = vi;
  params[i] -= lr * (mi / corr1) / (sqrtf(vi / corr2) + eps);
}

// x[t] = log(max(S[t] / mean S, 1e-30)) per row.
__global__ void __launch_bounds__(NT) log_features(const float* __restrict__ spectra,
                                                   float* __restrict__ out) {
  __shared__ float red[4];
  const int b = blockIdx.x, j = threadIdx.x;
  const float4 s = ld4(spectra + static_cast<int64_t>(b) * T + 4 * j);
  const float mean = block_sum((s.x + s.y) + (s.z + s.w), red) / static_cast<float>(T);
  const float inv = 1.f / mean;
  float4 o;
  o.x = logf(fmaxf(s.x * inv, 1e-30f));
  o.y = logf(fmaxf(s.y * inv, 1e-30f));
  o.z = logf(fmaxf(s.z * inv, 1e-30f));
  o.w = logf(fmaxf(s.w * inv, 1e-30f));
  *reinterpret_cast<float4*>(out + static_cast<int64_t>(b) * T + 4 * j) = o;
}

}  // namespace

// Parameter layout (floats): W1[32][1][7] b1[32] W2[32][32][7] b2[32]
// W3[32][32][7] b3[32] W4[1][32][7] b4[1].
constexpr int L1_OFF = 0, L2_OFF = 256, L3_OFF = 7456, L4_OFF = 14656;
static_assert(L4_OFF + 225 == NET_PARAMS, "parameter layout");

hipError_t launch_net_features(const float* spectra, int rows, float* out, hipStream_t s) {
  hipLaunchKernelGGL(log_features, dim3(rows), dim3(NT), 0, s, spectra, out);
  return hipGetLastError();
}

namespace {

// layers 1 to 3: a1, a2, a3
void launch_trunk(const NetWork& w, const float* x, int batch, hipStream_t s) {
  const dim3 tiles(batch * (T / TILE));
  hipLaunchKernelGGL((conv_tile<kFirstTwo>), tiles, dim3(TNT), 0, s, x, w.params, L2_OFF, w.a1, w.a2);
  hipLaunchKernelGGL((conv_tile<kForward>), tiles, dim3(TNT), 0, s, w.a2, w.params, L3_OFF,
                     static_cast<float*>(nullptr), w.a3);
}

}  // namespace

hipError_t launch_net_forward_f32(const NetWork& w, const float* x, int batch, float* logits,
                                  hipStream_t s) {
  launch_trunk(w, x, batch, s);
  hipLaunchKernelGGL((last_layer<false>), dim3(batch), dim3(1024), 0, s, w.a3, w.params, L4_OFF,
                     static_cast<const float*>(nullptr), logits, static_cast<float*>(nullptr), 0,
                     static_cast<float*>(nullptr), static_cast<float*>(nullptr));
  return hipGetLastError();
}

hipError_t launch_net_loss_grad(const NetWork& w, const float* x, const float* target_pos,
                                int batch, float* grad, float* loss_mean, hipStream_t s) {
  launch_trunk(w, x, batch, s);
  hipLaunchKernelGGL((last_layer<true>), dim3(batch), dim3(1024), 0, s, w.a3, w.params, L4_OFF,
                     target_pos, static_cast<float*>(nullptr), w.loss, NET_PARAMS, w.part, w.dzA);
  // data gradients: dz3 in dzA, dz2 in dzB, dz1 in a3 (no longer needed)
  const dim3 tiles(batch * (T / TILE));
  hipLaunchKernelGGL((conv_tile<kData>), tiles, dim3(TNT), 0, s, w.dzA, w.params, L3_OFF, w.a2, w.dzB);
  hipLaunchKernelGGL((conv_tile<kData>), tiles, dim3(TNT), 0, s, w.dzB, w.params, L2_OFF, w.a1, w.a3);
  hipLaunchKernelGGL(weight_grads, dim3(3 * batch), dim3(64 * WG_WAVES), 0, s, w.dzA, w.a2, w.dzB,
                     w.a1, w.a3, x, batch, L3_OFF, L2_OFF, L1_OFF, NET_PARAMS, w.part);
  hipLaunchKernelGGL(mean_rows, dim3((NET_PARAMS + 31) / 32 + 1), dim3(256), 0, s, w.part, batch,
                     NET_PARAMS, w.loss, grad, loss_mean);
  return hipGetLastError();
}

hipError_t launch_adam(float* params, const float* grad, float* m, float* v, int n, float lr,
                       int step, hipStream_t s) {
  const float b1 = 0.9f, b2 = 0.999f;
  const float c1 = 1.f - powf(b1, static_cast<float>(step));
  const float c2 = 1.f - powf(b2, static_cast<float>(step));
  hipLaunchKernelGGL(adam_update, dim3((n + 255) / 256), dim3(256), 0, s, params, grad, m, v, n,
                     lr, b1, b2, 1e-8f, c1, c2);
  return hipGetLastError();
}

}  // namespace ispl

// ---------------------------------------------------------------------------
// Inference on the matrix cores: BF16 weights and activations, FP32
// accumulation.  One workgroup (4 waves) per gate keeps the whole gate in
// LDS: the input row, and two [T][32] BF16 activation buffers used in turn.
// Layers 1-3 are GEMMs D[co][t] = sum_k A[co][k] B[k][t] on
// v_mfma_f32_32x32x16_bf16: layer 1 with k = tap (7 of 16 used), layers 2 and
// 3 with k = 32 tap + ci (14 k-steps); each wave holds its A fragments in
// registers for the whole layer and sweeps eight 32-position tiles.  Layer 4
// (one output channel) runs on the vector ALUs.  Activation rows are 64 bytes
// (32 channels); the four 16-byte channel groups of row t are stored at group
// position g ^ ((t >> 1) & 3), which puts the eight 16-byte accesses of
// consecutive rows that one LDS cycle serves on distinct banks.

namespace ispl {
namespace {

typedef __bf16 nbf16x8 __attribute__((ext_vector_type(8)));
typedef float nf32x16 __attribute__((ext_vector_type(16)));

struct alignas(16) Frag8 {
  uint32_t w[4];
};

__device__ __forceinline__ uint32_t to_bf16(float x) {  // round to nearest even
  uint32_t u = __float_as_uint(x);
  u += 0x7fffu + ((u >> 16) & 1u);
  return u >> 16;
}
__device__ __forceinline__ float from_bf16(uint32_t h) { return __uint_as_float(h << 16); }

// 2-byte index of channel ci of row t in a swizzled [T][32] activation buffer
__device__ __forceinline__ int act_idx(int t, int ci) {
  return t * 32 + 8 * ((ci >> 3) ^ ((t >> 1) & 3)) + (ci & 7);
}

// Weight tables of the matrix-core layers.  w1[ln]: layer 1's A fragment,
// W1[co = ln % 32][k = 8 (ln / 32) + i] for k < 7, zero above.  w2, w3 [ks][ln]:
// the 8 BF16 values W[co = ln % 32][ci][kk] with k = 16 ks + 8 (ln / 32) + i,
// kk = k / 32, ci = k % 32.  w4: BF16-rounded W4[ci][kk] as floats.  Biases FP32.
struct NetBf16 {
  Frag8 w1[64];
  Frag8 w2[14][64];
  Frag8 w3[14][64];
  float w4[32 * 7];
  float b1[32], b2[32], b3[32], b4;
};

__global__ void __launch_bounds__(256) prep_bf16(const float* __restrict__ p, NetBf16* out) {
  const int tid = threadIdx.x;
  for (int e = tid; e < 2 * 14 * 64; e += 256) {
    const int layer = e / (14 * 64), ks = (e / 64) % 14, ln = e % 64;
    const float* W = p + (layer == 0 ? 256 : 7456);
    Frag8 f;
    for (int i = 0; i < 8; i += 2) {
      uint32_t half[2];
      for (int u = 0; u < 2; ++u) {
        const int k = 16 * ks + 8 * (ln / 32) + i + u, kk = k / 32, ci = k % 32, co = ln % 32;
        half[u] = to_bf16(W[(co * 32 + ci) * 7 + kk]);
      }
      f.w[i / 2] = half[0] | (half[1] << 16);
    }
    (layer == 0 ? out->w2 : out->w3)[ks][ln] = f;
  }
  if (tid < 64) {
    Frag8 f;
    for (int i = 0; i < 8; i += 2) {
      uint32_t half[2];
      for (int u = 0; u < 2; ++u) {
        const int k = 8 * (tid / 32) + i + u, co = tid % 32;
        half[u] = k < 7 ? to_bf16(p[co * 7 + k]) : 0u;
      }
      f.w[i / 2] = half[0] | (half[1] << 16);
    }
    out->w1[tid] = f;
  }
  for (int e = tid; e < 224; e += 256) out->w4[e] = from_bf16(to_bf16(p[14656 + e]));
  if (tid < 32) {
    out->b1[tid] = p[224 + tid];
    out->b2[tid] = p[7424 + tid];
    out->b3[tid] = p[14624 + tid];
  }
  if (tid == 0) out->b4 = p[14880];
}

// The 16 biases of this lane's accumulator rows: bv[r] = bias[co(r)] with
// co(r) = (r % 4) + 8 (r / 4) + 4 h (h = lane / 32), loaded once per layer.
__device__ __forceinline__ void load_bias(const float* bias, int h, float (&bv)[16]) {
#pragma unroll
  for (int r = 0; r < 16; ++r) bv[r] = bias[(r & 3) + 8 * (r >> 2) + 4 * h];
}

// bias + ReLU of one 32 x 32 accumulator tile (D[co][t], t = this lane's
// column), rounded to BF16 and stored as four 8-byte groups.
__device__ __forceinline__ void store_tile(const nf32x16& acc, const float (&bv)[16], int h, int t,
                                           uint16_t* dst) {
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int co = 8 * q + 4 * h;
    const uint32_t v01 = to_bf16(fmaxf(acc[4 * q + 0] + bv[4 * q + 0], 0.f)) |
                         (to_bf16(fmaxf(acc[4 * q + 1] + bv[4 * q + 1], 0.f)) << 16);
    const uint32_t v23 = to_bf16(fmaxf(acc[4 * q + 2] + bv[4 * q + 2], 0.f)) |
                         (to_bf16(fmaxf(acc[4 * q + 3] + bv[4 * q + 3], 0.f)) << 16);
    *reinterpret_cast<uint2*>(dst + act_idx(t, co)) = make_uint2(v01, v23);
  }
}

// Forward workgroup: FW_WAVES waves, each owning FW_SPAN consecutive positions
// of the matrix-core layers.  The input stage (features) runs on the first
// FW_IN_THREADS threads, two positions each, whatever FW_WAVES is, so its
// reduction order (and hence every result) does not depend on the tiling.
constexpr int FW_WAVES = 16;
constexpr int FW_THREADS = 64 * FW_WAVES;
constexpr int FW_SPAN = T / FW_WAVES;   // 64 positions per wave
constexpr int FW_PAIRS = FW_SPAN / 64;  // pairs of 32-position tiles per wave
constexpr int FW_PER_THREAD = T / FW_THREADS;
constexpr int FW_IN_THREADS = T / 2;
constexpr int FW_IN_WAVES = FW_IN_THREADS / 64;
static_assert(FW_SPAN % 64 == 0 && T % FW_THREADS == 0, "forward tiling");

// One 32-channel layer: each wave sweeps its positions as pairs of
// 32-position tiles; the two tiles' accumulation chains are interleaved and
// the B fragments of the next k-step are read from LDS one step ahead, so
// neither the matrix-core latency nor the LDS latency stalls a lone wave.
__device__ __forceinline__ void mfma_layer(const uint16_t* __restrict__ src, uint16_t* __restrict__ dst,
                                           const Frag8 (*__restrict__ wt)[64], const float* bias,
                                           int wave, int lane) {
  const int h = lane >> 5, c = lane & 31;
  Frag8 afr[14];
#pragma unroll
  for (int ks = 0; ks < 14; ++ks) afr[ks] = wt[ks][lane];
  float bv[16];
  load_bias(bias, h, bv);
  auto bfrag = [&](int t, int ks) {
    const int kk = ks >> 1, ci0 = 16 * (ks & 1) + 8 * h;
    const int row = (t + kk - PAD) & (T - 1);
    return *reinterpret_cast<const Frag8*>(src + act_idx(row, ci0));
  };
  for (int pair = 0; pair < FW_PAIRS; ++pair) {
    const int t0 = FW_SPAN * wave + 64 * pair + c, t1 = t0 + 32;  // this lane's two columns
    nf32x16 acc0, acc1;
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      acc0[r] = 0.f;
      acc1[r] = 0.f;
    }
    Frag8 b0 = bfrag(t0, 0), b1 = bfrag(t1, 0);
#pragma unroll
    for (int ks = 0; ks < 14; ++ks) {
      Frag8 n0 = b0, n1 = b1;
      if (ks + 1 < 14) {
        n0 = bfrag(t0, ks + 1);
        n1 = bfrag(t1, ks + 1);
      }
      acc0 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(nbf16x8, afr[ks]),
                                                     __builtin_bit_cast(nbf16x8, b0), acc0, 0, 0, 0);
      acc1 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(nbf16x8, afr[ks]),
                                                     __builtin_bit_cast(nbf16x8, b1), acc1, 0, 0, 0);
      b0 = n0;
      b1 = n1;
    }
    store_tile(acc0, bv, h, t0, dst);
    store_tile(acc1, bv, h, t1, dst);
  }
}

// FROM_SPECTRA: the input rows are coarse spectra and the features
// log(max(S / mean S, 1e-30)) are formed here (as log_features does).  With
// chunks > 1 the spectra are still split over pulse chunks ([chunks][batch][T]
// partials): each row is summed in ascending chunk order, as the separate
// chunk reduction does, and written to x_out before use.
template <bool FROM_SPECTRA>
__global__ void __launch_bounds__(FW_THREADS) net_forward_bf16(const float* __restrict__ x,
                                                               const NetBf16* __restrict__ nw,
                                                               float* __restrict__ logits,
                                                               const float* __restrict__ partial,
                                                               int32_t chunks,
                                                               float* __restrict__ x_out) {
  __shared__ __attribute__((aligned(16))) float xs[T];
  __shared__ __attribute__((aligned(16))) uint16_t act0[T * 32];
  __shared__ __attribute__((aligned(16))) uint16_t act1[T * 32];
  __shared__ float red[FW_IN_WAVES];
  __shared__ float w4s[32 * TAPS];  // layer-4 weights, read by every lane
  const int g = blockIdx.x, j = threadIdx.x, lane = j & 63;
  const int wave = __builtin_amdgcn_readfirstlane(j >> 6);
  const int h = lane >> 5, c = lane & 31;
  if (j < 32 * TAPS) w4s[j] = nw->w4[j];
  // input stage: thread j < FW_IN_THREADS holds positions 2 j, 2 j + 1
  const bool in = j < FW_IN_THREADS;  // whole waves
  float2 v = make_float2(0.f, 0.f);
  if (!in) {
  } else if (FROM_SPECTRA && chunks > 1) {
    const int64_t cs = static_cast<int64_t>(gridDim.x) * T;
    const float2* pr = reinterpret_cast<const float2*>(partial + static_cast<int64_t>(g) * T) + j;
    v = make_float2(0.f, 0.f);
    // eight loads in flight, then the sums in ascending chunk order
    for (int c0 = 0; c0 < chunks; c0 += 8) {
      float2 q[8];
#pragma unroll
      for (int u = 0; u < 8; ++u)
        q[u] = c0 + u < chunks ? pr[(c0 + u) * (cs / 2)] : make_float2(0.f, 0.f);
#pragma unroll
      for (int u = 0; u < 8; ++u)
        if (c0 + u < chunks) {
          v.x += q[u].x;
          v.y += q[u].y;
        }
    }
    reinterpret_cast<float2*>(x_out + static_cast<int64_t>(g) * T)[j] = v;
  } else {
    v = reinterpret_cast<const float2*>(x + static_cast<int64_t>(g) * T)[j];
  }
  if (FROM_SPECTRA) {
    if (in) {
      float sum = v.x + v.y;
#pragma unroll
      for (int off = 32; off > 0; off >>= 1) sum += __shfl_xor(sum, off);
      if (lane == 0) red[wave] = sum;
    }
    __syncthreads();
    float tot = 0.f;
#pragma unroll
    for (int w = 0; w < FW_IN_WAVES; ++w) tot += red[w];  // fixed order
    const float inv = 1.f / (tot / static_cast<float>(T));
    v = make_float2(logf(fmaxf(v.x * inv, 1e-30f)), logf(fmaxf(v.y * inv, 1e-30f)));
  }
  if (in) reinterpret_cast<float2*>(xs)[j] = v;
  __syncthreads();
  // layer 1: one k-step, B[k][t] = bf16(x[t + k - 3]) for k < 7 (lanes h = 1 hold k >= 8: zero)
  {
    const Frag8 a1 = nw->w1[lane];
    float bv[16];
    load_bias(nw->b1, h, bv);
    for (int tile = 0; tile < FW_SPAN / 32; ++tile) {
      const int t = FW_SPAN * wave + 32 * tile + c;
      Frag8 bfr;
#pragma unroll
      for (int i = 0; i < 8; i += 2) {
        uint32_t lo = 0, hi = 0;
        if (h == 0) {
          lo = to_bf16(xs[(t + i - PAD) & (T - 1)]);
          if (i + 1 < TAPS) hi = to_bf16(xs[(t + i + 1 - PAD) & (T - 1)]);
        }
        bfr.w[i / 2] = lo | (hi << 16);
      }
      nf32x16 acc;
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[r] = 0.f;
      acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(nbf16x8, a1),
                                                    __builtin_bit_cast(nbf16x8, bfr), acc, 0, 0, 0);
      store_tile(acc, bv, h, t, act0);
    }
  }
  __syncthreads();
  mfma_layer(act0, act1, nw->w2, nw->b2, wave, lane);
  __syncthreads();
  mfma_layer(act1, act0, nw->w3, nw->b3, wave, lane);
  __syncthreads();
  // layer 4: thread j computes positions t = j + FW_THREADS m (consecutive lanes
  // read consecutive rows: conflict-free 16-byte LDS reads)
  float* out = logits + static_cast<int64_t>(g) * T;
  float acc[FW_PER_THREAD];
#pragma unroll
  for (int m = 0; m < FW_PER_THREAD; ++m) acc[m] = nw->b4;
#pragma unroll 1
  for (int q = 0; q < 4; ++q) {
#pragma unroll
    for (int kk = 0; kk < TAPS; ++kk) {
      float w[8];
#pragma unroll
      for (int i = 0; i < 8; ++i) w[i] = w4s[(8 * q + i) * TAPS + kk];
#pragma unroll
      for (int m = 0; m < FW_PER_THREAD; ++m) {
        const int row = (j + FW_THREADS * m + kk - PAD) & (T - 1);
        const uint4 u4 = *reinterpret_cast<const uint4*>(act0 + act_idx(row, 8 * q));
        const uint32_t u[4] = {u4.x, u4.y, u4.z, u4.w};
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          acc[m] = fmaf(w[2 * i], __uint_as_float(u[i] << 16), acc[m]);
          acc[m] = fmaf(w[2 * i + 1], __uint_as_float(u[i] & 0xffff0000u), acc[m]);
        }
      }
    }
  }
#pragma unroll
  for (int m = 0; m < FW_PER_THREAD; ++m) out[j + FW_THREADS * m] = acc[m];
}

// Forward split over S workgroups per gate, for batches too small to fill the
// chip with one workgroup per gate.  Part q owns the W = T / S output
// positions [a, a + W), a = q W, and computes layers 1..3 on the 32-aligned
// range [a - 32, a + W + 32) (W / 32 + 2 tiles, two per wave), enough for the
// 3-position halo that each later 7-tap layer consumes; the edge tiles read
// zero margin rows and are not used.  Every output takes the same operations
// in the same order as in net_forward_bf16 (the input stage reproduces its
// reduction tree over the whole row), so the logits are bit-identical.
template <int S>
struct SplitGeo {
  static constexpr int W = T / S;            // output positions per part
  static constexpr int NL = W + 64;          // computed positions per layer
  static constexpr int WAVES = NL / 64;      // matrix-layer waves: two 32-position tiles each
  // at least one wave per input-stage wave, so the row sum takes one pass
  static constexpr int THREADS = 64 * (WAVES > FW_IN_WAVES ? WAVES : FW_IN_WAVES);
  static constexpr int ROWS = NL + 2 * PAD;  // local rows: PAD zero margins each side
  static_assert(W % 64 == 0 && THREADS >= W, "split tiling");
};

// One 32-channel layer over the local rows (row u + PAD holds position
// a - 32 + u); same per-output arithmetic as mfma_layer.
template <int S>
__device__ __forceinline__ void mfma_layer_split(const uint16_t* __restrict__ src,
                                                 uint16_t* __restrict__ dst,
                                                 const Frag8 (*__restrict__ wt)[64],
                                                 const float* bias, int wave, int lane) {
  const int h = lane >> 5, c = lane & 31;
  Frag8 afr[14];
#pragma unroll
  for (int ks = 0; ks < 14; ++ks) afr[ks] = wt[ks][lane];
  float bv[16];
  load_bias(bias, h, bv);
  // all weight loads in flight before the first multiply (left to itself the
  // scheduler spreads them between the multiplies, one latency each)
  __builtin_amdgcn_sched_barrier(0);
  auto bfrag = [&](int u, int ks) {
    const int kk = ks >> 1, ci0 = 16 * (ks & 1) + 8 * h;
    return *reinterpret_cast<const Frag8*>(src + act_idx(u + kk, ci0));  // row (u + PAD) + kk - PAD
  };
  const int u0 = 64 * wave + c, u1 = u0 + 32;
  nf32x16 acc0, acc1;
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    acc0[r] = 0.f;
    acc1[r] = 0.f;
  }
  Frag8 b0 = bfrag(u0, 0), b1 = bfrag(u1, 0);
#pragma unroll
  for (int ks = 0; ks < 14; ++ks) {
    Frag8 n0 = b0, n1 = b1;
    if (ks + 1 < 14) {
      n0 = bfrag(u0, ks + 1);
      n1 = bfrag(u1, ks + 1);
    }
    acc0 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(nbf16x8, afr[ks]),
                                                   __builtin_bit_cast(nbf16x8, b0), acc0, 0, 0, 0);
    acc1 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(nbf16x8, afr[ks]),
                                                   __builtin_bit_cast(nbf16x8, b1), acc1, 0, 0, 0);
    b0 = n0;
    b1 = n1;
  }
  store_tile(acc0, bv, h, u0 + PAD, dst);
  store_tile(acc1, bv, h, u1 + PAD, dst);
}

template <bool FROM_SPECTRA, int S>
__global__ void __launch_bounds__(SplitGeo<S>::THREADS)
net_forward_split(const float* __restrict__ x, const NetBf16* __restrict__ nw,
                  float* __restrict__ logits, const float* __restrict__ partial, int32_t chunks,
                  float* __restrict__ x_out, int32_t batch) {
  using Geo = SplitGeo<S>;
  constexpr int W = Geo::W, NL = Geo::NL, ROWS = Geo::ROWS;
  __shared__ __attribute__((aligned(16))) float row_s[T];  // the gate's whole input row
  __shared__ __attribute__((aligned(16))) float xs[ROWS];  // local features
  __shared__ __attribute__((aligned(16))) uint16_t act0[ROWS * 32];
  __shared__ __attribute__((aligned(16))) uint16_t act1[ROWS * 32];
  __shared__ float red[FW_IN_WAVES];
  __shared__ float w4s[32 * TAPS];
  const int b = blockIdx.x, q = b / batch, g = b - q * batch;
  const int a = q * W;
  const int j = threadIdx.x, lane = j & 63;
  const int wave = __builtin_amdgcn_readfirstlane(j >> 6);
  const int h = lane >> 5, c = lane & 31;
  if (j < 32 * TAPS) w4s[j] = nw->w4[j];
  // zero margin rows of both activation buffers
  for (int e = j; e < 2 * PAD * 32; e += Geo::THREADS) {
    const int r = e / 32 < PAD ? e / 32 : NL + e / 32;  // rows 0..PAD-1 and NL+PAD..NL+2PAD-1
    act0[r * 32 + e % 32] = 0;
    act1[r * 32 + e % 32] = 0;
  }
  // input stage over the whole row: thread j < FW_IN_THREADS holds positions
  // 2 j, 2 j + 1 and wave w its share of the total, exactly as the
  // one-workgroup forward does, so the row total is the same float
  if (wave < FW_IN_WAVES) {
    const int jj = j;
    const int vw = wave;
    float2 v;
    if (FROM_SPECTRA && chunks > 1) {
      const int64_t cs = static_cast<int64_t>(batch) * T;
      const float2* pr =
          reinterpret_cast<const float2*>(partial + static_cast<int64_t>(g) * T) + jj;
      v = make_float2(0.f, 0.f);
      // sixteen loads in flight, then the sums in ascending chunk order
      for (int c0 = 0; c0 < chunks; c0 += 16) {
        float2 qv[16];
#pragma unroll
        for (int u = 0; u < 16; ++u)
          qv[u] = c0 + u < chunks ? pr[(c0 + u) * (cs / 2)] : make_float2(0.f, 0.f);
#pragma unroll
        for (int u = 0; u < 16; ++u)
          if (c0 + u < chunks) {
            v.x += qv[u].x;
            v.y += qv[u].y;
          }
      }
    } else {
      v = reinterpret_cast<const float2*>(x + static_cast<int64_t>(g) * T)[jj];
    }
    reinterpret_cast<float2*>(row_s)[jj] = v;
    if (FROM_SPECTRA) {
      float sum = v.x + v.y;
#pragma unroll
      for (int off = 32; off > 0; off >>= 1) sum += __shfl_xor(sum, off);
      if (lane == 0) red[vw] = sum;
    }
  }
  __syncthreads();
  float inv = 1.f;
  if (FROM_SPECTRA) {
    float tot = 0.f;
#pragma unroll
    for (int w = 0; w < FW_IN_WAVES; ++w) tot += red[w];  // fixed order
    inv = 1.f / (tot / static_cast<float>(T));
    if (chunks > 1 && j < W) x_out[static_cast<int64_t>(g) * T + a + j] = row_s[a + j];
  }
  // features of the local rows: row u + PAD holds position a - 32 + u (mod T)
  for (int u = j - PAD; u < NL + PAD; u += Geo::THREADS) {
    const float sv = row_s[(a - 32 + u) & (T - 1)];
    xs[u + PAD] = FROM_SPECTRA ? logf(fmaxf(sv * inv, 1e-30f)) : sv;
  }
  __syncthreads();
  // layer 1: one k-step, B[k][u] = bf16(x[u + k - 3]) for k < 7
  const bool mat = wave < Geo::WAVES;  // whole waves
  if (mat) {
    const Frag8 a1 = nw->w1[lane];
    float bv[16];
    load_bias(nw->b1, h, bv);
#pragma unroll
    for (int tile = 0; tile < 2; ++tile) {
      const int u = 64 * wave + 32 * tile + c;
      Frag8 bfr;
#pragma unroll
      for (int i = 0; i < 8; i += 2) {
        uint32_t lo = 0, hi = 0;
        if (h == 0) {
          lo = to_bf16(xs[u + i]);  // local row u + PAD + i - PAD
          if (i + 1 < TAPS) hi = to_bf16(xs[u + i + 1]);
        }
        bfr.w[i / 2] = lo | (hi << 16);
      }
      nf32x16 acc;
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[r] = 0.f;
      acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(nbf16x8, a1),
                                                    __builtin_bit_cast(nbf16x8, bfr), acc, 0, 0, 0);
      store_tile(acc, bv, h, u + PAD, act0);
    }
  }
  __syncthreads();
  if (mat) mfma_layer_split<S>(act0, act1, nw->w2, nw->b2, wave, lane);
  __syncthreads();
  if (mat) mfma_layer_split<S>(act1, act0, nw->w3, nw->b3, wave, lane);
  __syncthreads();
  // layer 4 on the part's W positions: thread j < W takes position a + j
  // (local u = 32 + j), in the one-workgroup forward's order
  if (j < W) {
    const int u = 32 + j;
    float acc = nw->b4;
#pragma unroll 1
    for (int qq = 0; qq < 4; ++qq) {
#pragma unroll
      for (int kk = 0; kk < TAPS; ++kk) {
        float w[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) w[i] = w4s[(8 * qq + i) * TAPS + kk];
        const uint4 u4 = *reinterpret_cast<const uint4*>(act0 + act_idx(u + kk, 8 * qq));
        const uint32_t uu[4] = {u4.x, u4.y, u4.z, u4.w};
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          acc = fmaf(w[2 * i], __uint_as_float(uu[i] << 16), acc);
          acc = fmaf(w[2 * i + 1], __uint_as_float(uu[i] & 0xffff0000u), acc);
        }
      }
    }
    logits[static_cast<int64_t>(g) * T + a + j] = acc;
  }
}

}  // namespace

size_t net_bf16_bytes() { return sizeof(NetBf16); }

constexpr int kSplitFourMax = 128;  // batches up to this many gates: four parts per gate
constexpr int kSplitTwoMax = 256;   // up to this many: two parts

hipError_t launch_net_prep_bf16(const float* params, void* table, hipStream_t s) {
  hipLaunchKernelGGL(prep_bf16, dim3(1), dim3(256), 0, s, params, static_cast<NetBf16*>(table));
  return hipGetLastError();
}

template <int S>
hipError_t launch_split(const void* table, const float* x, int batch, float* logits, hipStream_t s,
                        bool from_spectra, const float* partial, int32_t chunks, float* x_out) {
  const dim3 grid(static_cast<unsigned>(batch) * S), block(SplitGeo<S>::THREADS);
  const NetBf16* nw = static_cast<const NetBf16*>(table);
  if (from_spectra)
    hipLaunchKernelGGL((net_forward_split<true, S>), grid, block, 0, s, x, nw, logits, partial,
                       chunks, x_out, batch);
  else
    hipLaunchKernelGGL((net_forward_split<false, S>), grid, block, 0, s, x, nw, logits, nullptr, 1,
                       nullptr, batch);
  return hipGetLastError();
}

hipError_t launch_net_forward_bf16(const void* table, const float* x, int batch, float* logits,
                                   hipStream_t s, bool from_spectra, const float* partial,
                                   int32_t chunks, float* x_out) {
  // fewer gates than compute units: several workgroups per gate
  if (batch <= kSplitFourMax)
    return launch_split<4>(table, x, batch, logits, s, from_spectra, partial, chunks, x_out);
  if (batch <= kSplitTwoMax)
    return launch_split<2>(table, x, batch, logits, s, from_spectra, partial, chunks, x_out);
  if (from_spectra)
    hipLaunchKernelGGL(net_forward_bf16<true>, dim3(batch), dim3(FW_THREADS), 0, s, x,
                       static_cast<const NetBf16*>(table), logits, partial, chunks, x_out);
  else
    hipLaunchKernelGGL(net_forward_bf16<false>, dim3(batch), dim3(FW_THREADS), 0, s, x,
                       static_cast<const NetBf16*>(table), logits, nullptr, 1, nullptr);
  return hipGetLastError();
}

}  // namespace ispl
