// Normalisation, convolution and rotary kernels of the drafting step, plus small helpers.
// Each writes its result as bf16 planes ready to be MFMA operands (hi, and lo = rounding
// residual where the next contraction needs fp32-level accuracy).
#include <cmath>

#include "common.h"
#include "kernels.h"
#include "worklist.h"

namespace hspec {

namespace {

__device__ __forceinline__ void put_planes(bf16* hi, bf16* lo, size_t i, float v) {
  const bf16 h = f2bf(v);
  hi[i] = h;
  if (lo) lo[i] = f2bf(v - bf2f(h));
}

__device__ __forceinline__ float silu(float v) { return v / (1.f + __expf(-v)); }
__device__ __forceinline__ float softplus(float v) {
  return fmaxf(v, 0.f) + log1pf(__expf(-fabsf(v)));
}

// Block-wide sum (red: one entry per wave).
__device__ __forceinline__ float block_sum(float v, float* red) {
  v = wave_sum(v);
  const int w = threadIdx.x >> 6;
  if ((threadIdx.x & 63) == 0) red[w] = v;
  __syncthreads();
  float t = 0.f;
  for (int i = 0; i < (int)(blockDim.x >> 6); ++i) t += red[i];
  __syncthreads();
  return t;
}

// Rotation per position of RoPE pair p: theta^(-2p/D).  Pair 0 turns by 1 whatever the base (0 x log2(inf) is NaN).
__device__ __forceinline__ double inv_freq(int p, int D, double log2_theta) {
  return p ? exp2(-2.0 * (double)p / (double)D * log2_theta) : 1.0;
}

// 8 consecutive elements as fp32 (one 16-byte bf16 load or two 16-byte fp32 loads).
__device__ __forceinline__ void load8(const bf16* p, float (&v)[8]) {
  const bf16x8 x = ld8(p);
#pragma unroll
  for (int e = 0; e < 8; ++e) v[e] = bf2f(x[e]);
}
__device__ __forceinline__ void load8(const float* p, float (&v)[8]) {
  const f32x4 a = *reinterpret_cast<const f32x4*>(p), b = *reinterpret_cast<const f32x4*>(p + 4);
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    v[e] = a[e];
    v[4 + e] = b[e];
  }
}
__device__ __forceinline__ void put8(bf16* hi, bf16* lo, size_t i, const float (&v)[8]) {
  bf16x8 h, l;
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    h[e] = f2bf(v[e]);
    l[e] = f2bf(v[e] - bf2f(h[e]));
  }
  *reinterpret_cast<bf16x8*>(hi + i) = h;
  if (lo) *reinterpret_cast<bf16x8*>(lo + i) = l;
}

// One workgroup per row, 8 elements per thread and step (n % 8 == 0).  NR > 0: the row fits in
// NR chunks of 8 per thread (n <= 2048 NR); every chunk is loaded before the sum of squares and
// kept in registers for the scaling pass (chunks past the row end load the row's first chunk and
// count as zero).  NR == 0: any n, the second pass re-reads the row from cache.
// HEAD: the draft head's first kernel, which also clears the call's status words and keys.
struct HeadClear {
  int* status = nullptr;
  int words = 0;
  unsigned long long* keys = nullptr;   // kHeadSlots per row
};
template <typename T, int NR, bool HEAD = false>
__global__ void __launch_bounds__(256) rmsnorm_kernel(const T* x, const float* w, int n, float eps,
                                                      bf16* hi, bf16* lo, HeadClear clr) {
  if constexpr (HEAD) {
    if (threadIdx.x < kHeadSlots) clr.keys[(size_t)blockIdx.x * kHeadSlots + threadIdx.x] = 0;
    if (blockIdx.x == 0 && threadIdx.x < clr.words) clr.status[threadIdx.x] = 0;
  }
  __shared__ float red[4];
  const size_t row = blockIdx.x;
  const T* xr = x + row * n;
  if constexpr (NR > 0) {
    float v[NR][8];
    float ss = 0.f;
#pragma unroll
    for (int c = 0; c < NR; ++c) {
      const int i = (threadIdx.x + c * 256) * 8;
      load8(xr + (i < n ? i : 0), v[c]);
    }
#pragma unroll
    for (int c = 0; c < NR; ++c)
      if ((threadIdx.x + c * 256) * 8 < n)
#pragma unroll
        for (int e = 0; e < 8; ++e) ss += v[c][e] * v[c][e];
    ss = block_sum(ss, red);
    const float r = rsqrtf(ss / n + eps);
#pragma unroll
    for (int c = 0; c < NR; ++c) {
      const int i = (threadIdx.x + c * 256) * 8;
      if (i >= n) break;
      float g[8];
      load8(w + i, g);
#pragma unroll
      for (int e = 0; e < 8; ++e) v[c][e] = v[c][e] * r * g[e];
      put8(hi, lo, row * n + i, v[c]);
    }
    return;
  }
  float ss = 0.f;
  for (int i = threadIdx.x * 8; i < n; i += blockDim.x * 8) {
    float v[8];
    load8(xr + i, v);
#pragma unroll
    for (int e = 0; e < 8; ++e) ss += v[e] * v[e];
  }
  ss = block_sum(ss, red);
  const float r = rsqrtf(ss / n + eps);
  for (int i = threadIdx.x * 8; i < n; i += blockDim.x * 8) {
    float v[8], g[8];
    load8(xr + i, v);
    load8(w + i, g);
#pragma unroll
    for (int e = 0; e < 8; ++e) v[e] = v[e] * r * g[e];
    put8(hi, lo, row * n + i, v);
  }
}

// x = (planes of a product) + residual, written as fp32, and RMSNorm(x) w as bf16 planes: one
// workgroup of 1024 threads per row, 4 consecutive elements per thread and step, every plane's
// load in flight together (a row is a chain of latencies: 256 threads took 8 us at 128 rows of 4096 in
// 8 planes, 1024 take 6.4).  NR > 0: the row fits in NR steps and stays in registers; NR == 0:
// any n, the second pass re-reads the x it wrote.
template <int NR>
__global__ void __launch_bounds__(1024) sum_rmsnorm_kernel(Parts sum, const void* r, int r_bf16, float* x,
                                                           const float* w, int n, float eps, bf16* hi, bf16* lo) {
  __shared__ float red[16];
  const size_t row = (size_t)blockIdx.x * n;
  auto load_x = [&](int i) {
    const size_t at[1] = {row + i};
    f32x4 v[1], q;
    if (r_bf16) {
      const bf16x4 b = *reinterpret_cast<const bf16x4*>(reinterpret_cast<const bf16*>(r) + row + i);
      q = f32x4{bf2f(b[0]), bf2f(b[1]), bf2f(b[2]), bf2f(b[3])};
    } else {
      q = *reinterpret_cast<const f32x4*>(reinterpret_cast<const float*>(r) + row + i);
    }
    ld4_parts<1, 8>(sum.p, sum.np, sum.plane, at, v);
    return v[0] + q;
  };
  auto scale = [&](int i, f32x4 v, float rs) {
    const f32x4 g = *reinterpret_cast<const f32x4*>(w + i);
    bf16x4 h, l;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const float u = v[e] * rs * g[e];
      h[e] = f2bf(u);
      l[e] = f2bf(u - bf2f(h[e]));
    }
    *reinterpret_cast<bf16x4*>(hi + row + i) = h;
    if (lo) *reinterpret_cast<bf16x4*>(lo + row + i) = l;
  };
  f32x4 v[NR > 0 ? NR : 1];
  float ss = 0.f;
  if constexpr (NR > 0) {
#pragma unroll
    for (int c = 0; c < NR; ++c) {
      const int i = (threadIdx.x + c * 1024) * 4;
      v[c] = load_x(i < n ? i : 0);
      if (i >= n) continue;
      *reinterpret_cast<f32x4*>(x + row + i) = v[c];
#pragma unroll
      for (int e = 0; e < 4; ++e) ss += v[c][e] * v[c][e];
    }
  } else {
    for (int i = threadIdx.x * 4; i < n; i += 4096) {
      v[0] = load_x(i);
      *reinterpret_cast<f32x4*>(x + row + i) = v[0];
#pragma unroll
      for (int e = 0; e < 4; ++e) ss += v[0][e] * v[0][e];
    }
  }
  ss = block_sum(ss, red);
  const float rs = rsqrtf(ss / n + eps);
  if constexpr (NR > 0) {
#pragma unroll
    for (int c = 0; c < NR; ++c) {
      const int i = (threadIdx.x + c * 1024) * 4;
      if (i < n) scale(i, v[c], rs);
    }
  } else {
    for (int i = threadIdx.x * 4; i < n; i += 4096)   // (each thread its own elements)
      scale(i, *reinterpret_cast<const f32x4*>(x + row + i), rs);
  }
}

template <typename T>
__global__ void __launch_bounds__(256) conv_split_kernel(ConvArgs a) {
  if (a.clear && blockIdx.x == 0 && blockIdx.y == 0 && threadIdx.x < kStatusClear) a.clear[threadIdx.x] = 0;
  const int di = a.H * a.P, gn = a.G * a.N, cdim = di + 2 * gn;
  const int dproj = 2 * di + 2 * gn + a.H;
  const int tok = blockIdx.y;                        // b*T + t
  const int t = tok % a.T;
  const T* cw = reinterpret_cast<const T*>(a.conv_w);
  const T* cb = reinterpret_cast<const T*>(a.conv_b);
  for (int c = blockIdx.x * blockDim.x + threadIdx.x; c < cdim + a.H; c += gridDim.x * blockDim.x) {
    if (c < cdim) {
      float v = to_f32(cb[c]);
      for (int j = 0; j < a.K; ++j) {
        const int tau = t - (a.K - 1) + j;
        if (tau >= 0) v += to_f32(cw[(size_t)c * a.K + j]) * ld1_parts(a.zxbcdt.p, a.zxbcdt.np, a.zxbcdt.plane, (size_t)(tok - t + tau) * dproj + di + c);
      }
      v = silu(v);
      if (c < di) put_planes(a.x_hi, a.x_lo, (size_t)tok * di + c, v);
      else if (c < di + gn) put_planes(a.B_hi, a.B_lo, (size_t)tok * gn + (c - di), v);
      else put_planes(a.C_hi, a.C_lo, (size_t)tok * gn + (c - di - gn), v);
    } else {
      const int hh = c - cdim;
      a.dt[(size_t)tok * a.H + hh] =
          softplus(ld1_parts(a.zxbcdt.p, a.zxbcdt.np, a.zxbcdt.plane, (size_t)tok * dproj + 2 * di + 2 * gn + hh) + a.dt_bias[hh]);
    }
  }
}

// Causal conv with the paper's width of 4 taps: a thread owns 4 consecutive channels of
// CONV_TT consecutive tokens of one request and reads the CONV_TT + 3 inputs they need (tokens
// before the block's first are zero) straight from zx, all loads in flight together.  Weights of
// the 4 channels are 16 consecutive values, read as vectors.  Same alignment needs as the serial
// kernel below.
//
// CONV_TT = 4 reads each input 1.75 times, CONV_TT = 1 four times: with few tokens the launch is
// a chain of latencies on a handful of workgroups, and one token per thread shortens the chain and
// makes four times the workgroups (128 tokens of 3200 channels in 5 partial planes: 13.8 -> 6.5 us;
// 161 tokens in one plane 9.7 -> 5.0).
template <typename T, int CONV_TT, bool ONE>
__global__ void __launch_bounds__(256) conv4_tok_kernel(ConvArgs a) {
  if (a.clear && blockIdx.x == 0 && blockIdx.y == 0 && threadIdx.x < kStatusClear) a.clear[threadIdx.x] = 0;
  const int di = a.H * a.P, gn = a.G * a.N, cdim = di + 2 * gn;
  const int dproj = 2 * di + 2 * gn + a.H;
  const int nq = (a.T + CONV_TT - 1) / CONV_TT;
  const int b = blockIdx.y / nq, t0 = (blockIdx.y % nq) * CONV_TT;
  const int c = (blockIdx.x * blockDim.x + threadIdx.x) * 4;
  if (c >= cdim + a.H) return;
  const size_t zb = (size_t)b * a.T * dproj;
  if (c >= cdim) {                                   // dt = softplus(dt_raw + dt_bias), 4 heads
    const int hh = c - cdim;
    f32x4 v[CONV_TT];
    size_t at[CONV_TT];
#pragma unroll
    for (int u = 0; u < CONV_TT; ++u) at[u] = zb + (size_t)min(t0 + u, a.T - 1) * dproj + 2 * di + 2 * gn + hh;
    ld4_parts<CONV_TT, ONE ? 0 : 2>(a.zxbcdt.p, a.zxbcdt.np, a.zxbcdt.plane, at, v);
#pragma unroll
    for (int u = 0; u < CONV_TT; ++u) {
      if (t0 + u >= a.T) break;
      f32x4 o;
#pragma unroll
      for (int e = 0; e < 4; ++e) o[e] = softplus(v[u][e] + a.dt_bias[hh + e]);
      *reinterpret_cast<f32x4*>(a.dt + ((size_t)b * a.T + t0 + u) * a.H + hh) = o;
    }
    return;
  }
  // in[j] is token t0 - 3 + j
  f32x4 in[CONV_TT + 3];
  size_t at[CONV_TT + 3];
#pragma unroll
  for (int j = 0; j < CONV_TT + 3; ++j) at[j] = zb + (size_t)max(0, min(t0 - 3 + j, a.T - 1)) * dproj + di + c;
  ld4_parts<CONV_TT + 3, ONE ? 0 : CONV_TT == 1 ? 4 : 2>(a.zxbcdt.p, a.zxbcdt.np, a.zxbcdt.plane, at, in);
#pragma unroll
  for (int j = 0; j < 3; ++j)   // (tokens past the last feed no output that is stored)
    if (t0 - 3 + j < 0) in[j] = f32x4{0.f, 0.f, 0.f, 0.f};
  float w[16], bias[4];
  if constexpr (sizeof(T) == 2) {
    const bf16x8 w0 = ld8(reinterpret_cast<const bf16*>(a.conv_w) + (size_t)c * 4);
    const bf16x8 w1 = ld8(reinterpret_cast<const bf16*>(a.conv_w) + (size_t)c * 4 + 8);
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      w[e] = bf2f(w0[e]);
      w[8 + e] = bf2f(w1[e]);
    }
  } else {
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const f32x4 v = *reinterpret_cast<const f32x4*>(reinterpret_cast<const float*>(a.conv_w) + (size_t)c * 4 + 4 * q);
#pragma unroll
      for (int e = 0; e < 4; ++e) w[4 * q + e] = v[e];
    }
  }
  const T* cb = reinterpret_cast<const T*>(a.conv_b);
#pragma unroll
  for (int e = 0; e < 4; ++e) bias[e] = to_f32(cb[c + e]);
  bf16* ohi;
  bf16* olo;
  int ld, col;
  if (c < di) { ohi = a.x_hi; olo = a.x_lo; ld = di; col = c; }
  else if (c < di + gn) { ohi = a.B_hi; olo = a.B_lo; ld = gn; col = c - di; }
  else { ohi = a.C_hi; olo = a.C_lo; ld = gn; col = c - di - gn; }
#pragma unroll
  for (int u = 0; u < CONV_TT; ++u) {
    if (t0 + u >= a.T) break;
    bf16x4 h, l;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      float v = bias[e];
#pragma unroll
      for (int j = 0; j < 4; ++j) v += w[4 * e + j] * in[u + j][e];
      v = silu(v);
      h[e] = f2bf(v);
      l[e] = f2bf(v - bf2f(h[e]));
    }
    const size_t o = ((size_t)b * a.T + t0 + u) * ld + col;
    *reinterpret_cast<bf16x4*>(ohi + o) = h;
    if (olo) *reinterpret_cast<bf16x4*>(olo + o) = l;
  }
}

// Vectorised causal conv: a thread owns 4 consecutive channels of one request and walks its
// T tokens in order with the last 8 inputs in registers, so zx is read once.  Needs the xBC and
// dt parts of a zx row 16-byte aligned (checked by the launcher).
template <typename T>
__global__ void __launch_bounds__(256) conv_split4_kernel(ConvArgs a) {
  if (a.clear && blockIdx.x == 0 && blockIdx.y == 0 && threadIdx.x < kStatusClear) a.clear[threadIdx.x] = 0;
  const int di = a.H * a.P, gn = a.G * a.N, cdim = di + 2 * gn;
  const int dproj = 2 * di + 2 * gn + a.H;
  const int b = blockIdx.y;
  const int c = (blockIdx.x * blockDim.x + threadIdx.x) * 4;
  if (c >= cdim + a.H) return;
  const size_t zrow = (size_t)b * a.T * dproj;
  auto in4 = [&](size_t i) {
    const size_t at[1] = {i};
    f32x4 v[1];
    ld4_parts<1, 4>(a.zxbcdt.p, a.zxbcdt.np, a.zxbcdt.plane, at, v);
    return v[0];
  };
  if (c >= cdim) {                                   // dt = softplus(dt_raw + dt_bias), 4 heads
    const int hh = c - cdim;
    for (int t = 0; t < a.T; ++t) {
      const f32x4 v = in4(zrow + (size_t)t * dproj + 2 * di + 2 * gn + hh);
      f32x4 o;
#pragma unroll
      for (int e = 0; e < 4; ++e) o[e] = softplus(v[e] + a.dt_bias[hh + e]);
      *reinterpret_cast<f32x4*>(a.dt + ((size_t)b * a.T + t) * a.H + hh) = o;
    }
    return;
  }
  const T* cw = reinterpret_cast<const T*>(a.conv_w);
  const T* cb = reinterpret_cast<const T*>(a.conv_b);
  // taps right-aligned in an 8-wide window: wp[j] multiplies the input 7 - j tokens back
  float wp[8][4], bias[4];
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    bias[e] = to_f32(cb[c + e]);
#pragma unroll
    for (int j = 0; j < 8; ++j) wp[j][e] = j >= 8 - a.K ? to_f32(cw[(size_t)(c + e) * a.K + j - (8 - a.K)]) : 0.f;
  }
  f32x4 hist[8];
#pragma unroll
  for (int j = 0; j < 8; ++j) hist[j] = f32x4{0.f, 0.f, 0.f, 0.f};
  bf16* ohi;
  bf16* olo;
  int ld, col;
  if (c < di) { ohi = a.x_hi; olo = a.x_lo; ld = di; col = c; }
  else if (c < di + gn) { ohi = a.B_hi; olo = a.B_lo; ld = gn; col = c - di; }
  else { ohi = a.C_hi; olo = a.C_lo; ld = gn; col = c - di - gn; }
  for (int t = 0; t < a.T; ++t) {
#pragma unroll
    for (int j = 0; j < 7; ++j) hist[j] = hist[j + 1];
    hist[7] = in4(zrow + (size_t)t * dproj + di + c);
    bf16x4 h, l;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      float v = bias[e];
#pragma unroll
      for (int j = 0; j < 8; ++j) v += wp[j][e] * hist[j][e];
      v = silu(v);
      h[e] = f2bf(v);
      l[e] = f2bf(v - bf2f(h[e]));
    }
    const size_t o = ((size_t)b * a.T + t) * ld + col;
    *reinterpret_cast<bf16x4*>(ohi + o) = h;
    if (olo) *reinterpret_cast<bf16x4*>(olo + o) = l;
  }
}

// One workgroup per (row, group); 8 elements per thread and step.  VEC: y and z rows can be
// read as 16-byte vectors.  NR > 0 (with VEC): the group fits in NR chunks of 8 per thread and is
// gated once, kept in registers between the sum of squares and the scaling pass (chunks past the
// group's end load its first chunk and count as zero); NR == 0: the second pass re-reads y and z.
template <bool VEC, int NR, bool ONE = false>
__global__ void __launch_bounds__(256) gated_rmsnorm_kernel(const float* y, Parts z, int z_ld,
                                                            const float* w, int n, int G, float eps,
                                                            bf16* hi, bf16* lo) {
  __shared__ float red[4];
  const size_t row = blockIdx.x / G;
  const int gi = blockIdx.x % G, gs = n / G;
  const float* yr = y + row * n + (size_t)gi * gs;
  const size_t zr = row * z_ld + (size_t)gi * gs;
  auto load8z = [&](int i, float (&v)[8]) {
    const size_t at[2] = {zr + i, zr + i + 4};
    f32x4 q[2];
    ld4_parts(z.p, z.np, z.plane, at, q);
#pragma unroll
    for (int e = 0; e < 8; ++e) v[e] = q[e / 4][e % 4];
  };
  auto gated8 = [&](int i, float (&v)[8]) {
    float zz[8];
    if constexpr (VEC) {
      load8(yr + i, v);
      load8z(i, zz);
    } else {
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        v[e] = yr[i + e];
        zz[e] = ld1_parts(z.p, z.np, z.plane, zr + i + e);
      }
    }
#pragma unroll
    for (int e = 0; e < 8; ++e) v[e] *= silu(zz[e]);
  };
  if constexpr (NR > 0) {
    float v[NR][8], zz[NR][8];
    size_t at[2 * NR];
    f32x4 zq[2 * NR];
#pragma unroll
    for (int c = 0; c < NR; ++c) {
      const int i = (threadIdx.x + c * 256) * 8, ic = i < gs ? i : 0;
      load8(yr + ic, v[c]);
      at[2 * c] = zr + ic;
      at[2 * c + 1] = zr + ic + 4;
    }
    ld4_parts<2 * NR, ONE ? 0 : 2>(z.p, z.np, z.plane, at, zq);
#pragma unroll
    for (int c = 0; c < NR; ++c)
#pragma unroll
      for (int e = 0; e < 8; ++e) zz[c][e] = zq[2 * c + e / 4][e % 4];
    float ss = 0.f;
#pragma unroll
    for (int c = 0; c < NR; ++c) {
      const bool in = (threadIdx.x + c * 256) * 8 < gs;
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        v[c][e] *= silu(zz[c][e]);
        ss += in ? v[c][e] * v[c][e] : 0.f;
      }
    }
    ss = block_sum(ss, red);
    const float r = rsqrtf(ss / gs + eps);
#pragma unroll
    for (int c = 0; c < NR; ++c) {
      const int i = (threadIdx.x + c * 256) * 8;
      if (i >= gs) break;
      float g[8];
      load8(w + (size_t)gi * gs + i, g);
#pragma unroll
      for (int e = 0; e < 8; ++e) v[c][e] = v[c][e] * r * g[e];
      put8(hi, lo, row * n + (size_t)gi * gs + i, v[c]);
    }
    return;
  }
  float ss = 0.f;
  for (int i = threadIdx.x * 8; i < gs; i += blockDim.x * 8) {
    float v[8];
    gated8(i, v);
#pragma unroll
    for (int e = 0; e < 8; ++e) ss += v[e] * v[e];
  }
  ss = block_sum(ss, red);
  const float r = rsqrtf(ss / gs + eps);
  for (int i = threadIdx.x * 8; i < gs; i += blockDim.x * 8) {
    float v[8], g[8];
    gated8(i, v);
    load8(w + (size_t)gi * gs + i, g);
#pragma unroll
    for (int e = 0; e < 8; ++e) v[e] = v[e] * r * g[e];
    put8(hi, lo, row * n + (size_t)gi * gs + i, v);
  }
}

// Per-head RMSNorm of q and k, then rotate-half RoPE at position ctx_len + j; v heads are copied.
// One workgroup (4 waves) per token, for D a multiple of 8 with D/8 dividing 64 (D = 8 .. 512):
// a lane owns elements i0..i0+3 and i0 + D/2 .. i0 + D/2 + 3 of a head (16-byte loads, 8-byte
// plane stores), D/8 lanes per head.  The D/2 rotation angles of the token are computed once
// (in fp64, reduced modulo 2 pi, then fp32 sin/cos) by the first D/2 threads into LDS while the
// first heads load.
constexpr int QKR4_U = 4;

template <bool PLAN, bool ONE>
__global__ void __launch_bounds__(256) qk_norm_rope4_kernel(Parts qkv, const float* qw, const float* kw,
                                                            const int32_t* ctx_lens, int T, int Hq, int Hkv,
                                                            int D, float eps, double log2_theta, bf16* q_hi,
                                                            bf16* q_lo, bf16* k_hi, bf16* k_lo, bf16* v_hi,
                                                            bf16* v_lo, AttnArgs plan, int plan_clear) {
  touch_args<128 + (PLAN ? sizeof(AttnArgs) : 0)>();
  if constexpr (PLAN) {   // the first workgroup (dispatched first) builds the KV sweep's work list
    __shared__ WorklistLds<kWorklistFusedMax> wl;
    if (blockIdx.x == 0) {
      build_worklist<kWorklistFusedMax>(plan, plan_clear, wl);
      return;
    }
  }
  __shared__ float s_cs[256], s_sn[256];
  const int nh = Hq + 2 * Hkv;
  const int tok = PLAN ? blockIdx.x - 1 : blockIdx.x;
  const int b = tok / T, j = tok % T;
  const int half = D / 2, lph = D / 8, hpw = 64 / lph;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int i0 = 4 * (lane % lph), hsub = lane / lph;
  const int hstep = 4 * hpw;                 // heads per workgroup pass
  const size_t src_tok = (size_t)tok * nh * D;
  f32x4 x1[QKR4_U], x2[QKR4_U];
  auto load_heads = [&](int h0) {
    size_t at[2 * QKR4_U];
    f32x4 v[2 * QKR4_U];
#pragma unroll
    for (int u = 0; u < QKR4_U; ++u) {
      const int head = h0 + u * hstep + wave * hpw + hsub;
      at[2 * u] = src_tok + (size_t)(head < nh ? head : 0) * D + i0;
      at[2 * u + 1] = at[2 * u] + half;
    }
    ld4_parts<2 * QKR4_U, ONE ? 0 : 4>(qkv.p, qkv.np, qkv.plane, at, v);
#pragma unroll
    for (int u = 0; u < QKR4_U; ++u) {
      x1[u] = v[2 * u];
      x2[u] = v[2 * u + 1];
    }
  };
  load_heads(0);
  for (int p = threadIdx.x; p < half; p += blockDim.x) {
    double phi = ((double)ctx_lens[b] + j) * inv_freq(p, D, log2_theta);
    const double two_pi = 6.283185307179586476925286766559;
    phi -= two_pi * rint(phi / two_pi);
    float sn, cs;
    sincosf((float)phi, &sn, &cs);
    s_cs[p] = cs;
    s_sn[p] = sn;
  }
  const f32x4 gq1 = *reinterpret_cast<const f32x4*>(qw + i0), gq2 = *reinterpret_cast<const f32x4*>(qw + half + i0);
  const f32x4 gk1 = *reinterpret_cast<const f32x4*>(kw + i0), gk2 = *reinterpret_cast<const f32x4*>(kw + half + i0);
  __syncthreads();
  float cs[4], sn[4];
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    cs[e] = s_cs[i0 + e];
    sn[e] = s_sn[i0 + e];
  }
  for (int h0 = 0; h0 < nh; h0 += QKR4_U * hstep) {
    if (h0) load_heads(h0);
#pragma unroll
    for (int u = 0; u < QKR4_U; ++u) {
      const int head = h0 + u * hstep + wave * hpw + hsub;
      // sum of squares over the head's D/8 lanes (every lane takes part in the exchange)
      float ss = 0.f;
#pragma unroll
      for (int e = 0; e < 4; ++e) ss += x1[u][e] * x1[u][e] + x2[u][e] * x2[u][e];
      for (int off = lph / 2; off > 0; off >>= 1) ss += __shfl_xor(ss, off);
      if (head >= nh) continue;
      float o1[4], o2[4];
      bf16 *hi, *lo;
      size_t o;
      if (head >= Hq + Hkv) {                  // v heads: copy
        o = ((size_t)tok * Hkv + (head - Hq - Hkv)) * D;
        hi = v_hi;
        lo = v_lo;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          o1[e] = x1[u][e];
          o2[e] = x2[u][e];
        }
      } else {
        const bool isq = head < Hq;
        const float r = rsqrtf(ss / D + eps);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const float a1 = x1[u][e] * r * (isq ? gq1[e] : gk1[e]), a2 = x2[u][e] * r * (isq ? gq2[e] : gk2[e]);
          o1[e] = a1 * cs[e] - a2 * sn[e];
          o2[e] = a2 * cs[e] + a1 * sn[e];
        }
        hi = isq ? q_hi : k_hi;
        lo = isq ? q_lo : k_lo;
        o = isq ? ((size_t)tok * Hq + head) * D : ((size_t)tok * Hkv + (head - Hq)) * D;
      }
      bf16x4 h1, l1, h2, l2;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        h1[e] = f2bf(o1[e]);
        l1[e] = f2bf(o1[e] - bf2f(h1[e]));
        h2[e] = f2bf(o2[e]);
        l2[e] = f2bf(o2[e] - bf2f(h2[e]));
      }
      *reinterpret_cast<bf16x4*>(hi + o + i0) = h1;
      *reinterpret_cast<bf16x4*>(hi + o + half + i0) = h2;
      if (lo) {
        *reinterpret_cast<bf16x4*>(lo + o + i0) = l1;
        *reinterpret_cast<bf16x4*>(lo + o + half + i0) = l2;
      }
    }
  }
}

// blockIdx.y: tensor.  Four elements per thread and step; the tail one by one.
__global__ void __launch_bounds__(256) split_kernel(SplitArgs a) {
  const float* x = a.x[0];
  bf16 *hi = a.hi[0], *lo = a.lo[0];
  size_t n = a.len[0];
#pragma unroll
  for (int k = 1; k < SplitArgs::kMax; ++k)   // (no indexed copy of the arguments)
    if (blockIdx.y == k) {
      x = a.x[k];
      hi = a.hi[k];
      lo = a.lo[k];
      n = a.len[k];
    }
  const size_t i0 = blockIdx.x * 256 + threadIdx.x, step = (size_t)gridDim.x * 256;
  const size_t quads = reinterpret_cast<uintptr_t>(x) % 16 ? 0 : n / 4;
  for (size_t q = i0; q < quads; q += step) {
    const f32x4 v = *reinterpret_cast<const f32x4*>(x + 4 * q);
    bf16x4 h, l;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      h[e] = f2bf(v[e]);
      l[e] = f2bf(v[e] - bf2f(h[e]));
    }
    *reinterpret_cast<bf16x4*>(hi + 4 * q) = h;
    *reinterpret_cast<bf16x4*>(lo + 4 * q) = l;
  }
  for (size_t i = 4 * quads + i0; i < n; i += step) put_planes(hi, lo, i, x[i]);
}

// h = SiLU(gate) * up for rows [gate | up] of width 2 ff, as bf16 hi/lo planes [rows, ff]; four
// columns per thread (ff % 8 == 0).
__global__ void __launch_bounds__(256) silu_mul_kernel(Parts gu, int ff, bf16* hi, bf16* lo) {
  const size_t row = blockIdx.y;
  const int i = (blockIdx.x * 256 + threadIdx.x) * 4;
  if (i >= ff) return;
  const size_t at[2] = {row * 2 * ff + i, row * 2 * ff + ff + i};
  f32x4 x[2];
  ld4_parts<2, 4>(gu.p, gu.np, gu.plane, at, x);
  bf16x4 h, l;
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    const float v = silu(x[0][e]) * x[1][e];
    h[e] = f2bf(v);
    l[e] = f2bf(v - bf2f(h[e]));
  }
  *reinterpret_cast<bf16x4*>(hi + row * ff + i) = h;
  if (lo) *reinterpret_cast<bf16x4*>(lo + row * ff + i) = l;
}

// The new rows of every layer's K and V into its paged cache: one workgroup per token, which computes the
// token's slot and rotation angles once and then walks the heads of all layers as qk_norm_rope4_kernel
// does (k: RMSNorm, RoPE; v: copied), D/8 lanes per head.  Positions the table does not map, or page ids
// outside the pool, set a status bit and are skipped.
template <typename T>
__global__ void __launch_bounds__(256) kv_append_kernel(AppendArgs a, double log2_theta) {
  __shared__ float s_cs[256], s_sn[256];
  const int tok = blockIdx.x, b = tok / a.n, i = tok % a.n;
  const int L = a.ctx_lens[b];
  const unsigned pos = (unsigned)L + i, pg = pos / (unsigned)a.ps;   // (no sum that wraps below zero at lengths near 2^31)
  if (L < 0 || pg >= (unsigned)a.max_pages) {
    if (threadIdx.x == 0 && a.status) atomicOr(a.status, 2);
    return;
  }
  const int pid = a.page_table[(size_t)b * a.max_pages + pg];
  if (pid < 0 || pid >= a.num_pages) {
    if (threadIdx.x == 0 && a.status) atomicOr(a.status, 1);
    return;
  }
  const int D = a.D, half = D / 2, lph = D / 8, hpp = 256 / lph;   // heads per pass
  const size_t dst0 = ((size_t)pid * a.ps + pos % (unsigned)a.ps) * a.Hkv * D;
  for (int p = threadIdx.x; p < half; p += 256) {
    double phi = (double)pos * inv_freq(p, D, log2_theta);
    const double two_pi = 6.283185307179586476925286766559;
    phi -= two_pi * rint(phi / two_pi);
    float sn, cs;
    sincosf((float)phi, &sn, &cs);
    s_cs[p] = cs;
    s_sn[p] = sn;
  }
  __syncthreads();
  const int i0 = 4 * (threadIdx.x % lph), nh = a.n_layers * 2 * a.Hkv;
  f32x4 cs, sn;
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    cs[e] = s_cs[i0 + e];
    sn[e] = s_sn[i0 + e];
  }
  constexpr int U = 4;
  for (int h0 = a.head0; h0 < a.head1; h0 += U * hpp) {
    size_t at[2 * U];
    f32x4 x[2 * U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int head = h0 + u * hpp + threadIdx.x / lph;
      at[2 * u] = ((size_t)tok * nh + (head < a.head1 ? head : a.head0)) * D + i0;
      at[2 * u + 1] = at[2 * u] + half;
    }
    ld4_parts<2 * U, 2>(a.kv.p, a.kv.np, a.kv.plane, at, x);
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int head = h0 + u * hpp + threadIdx.x / lph;
      f32x4 x1 = x[2 * u], x2 = x[2 * u + 1];
      // sum of squares over the head's D/8 lanes (every lane takes part in the exchange)
      float ss = 0.f;
#pragma unroll
      for (int e = 0; e < 4; ++e) ss += x1[e] * x1[e] + x2[e] * x2[e];
      for (int off = lph / 2; off > 0; off >>= 1) ss += __shfl_xor(ss, off);
      if (head >= a.head1) continue;
      const int l = head / (2 * a.Hkv), hh = head % (2 * a.Hkv);
      const float* kw = a.kw[0];
      void* dst = hh < a.Hkv ? a.k_cache[0] : a.v_cache[0];
#pragma unroll
      for (int k = 1; k < AppendArgs::kMaxLayers; ++k)   // (no indexed copy of the arguments)
        if (l == k) {
          kw = a.kw[k];
          dst = hh < a.Hkv ? a.k_cache[k] : a.v_cache[k];
        }
      if (hh < a.Hkv) {
        const float r = rsqrtf(ss / D + a.eps);
        const f32x4 g1 = *reinterpret_cast<const f32x4*>(kw + i0), g2 = *reinterpret_cast<const f32x4*>(kw + half + i0);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const float a1 = x1[e] * r * g1[e], a2 = x2[e] * r * g2[e];
          x1[e] = a1 * cs[e] - a2 * sn[e];
          x2[e] = a2 * cs[e] + a1 * sn[e];
        }
      }
      T* o = reinterpret_cast<T*>(dst) + dst0 + (size_t)(hh % a.Hkv) * D + i0;
      if constexpr (sizeof(T) == 2) {
        *reinterpret_cast<bf16x4*>(o) = bf16x4{f2bf(x1[0]), f2bf(x1[1]), f2bf(x1[2]), f2bf(x1[3])};
        *reinterpret_cast<bf16x4*>(o + half) = bf16x4{f2bf(x2[0]), f2bf(x2[1]), f2bf(x2[2]), f2bf(x2[3])};
      } else {
        *reinterpret_cast<f32x4*>(o) = x1;
        *reinterpret_cast<f32x4*>(o + half) = x2;
      }
    }
  }
}

__global__ void zero_kernel(int* p, int n) {
  for (int i = threadIdx.x; i < n; i += blockDim.x) p[i] = 0;
}

__global__ void __launch_bounds__(256) copy_kernel(const float* x, size_t n, float* y) {
  for (size_t i = blockIdx.x * (size_t)256 + threadIdx.x; i < n; i += (size_t)gridDim.x * 256) y[i] = x[i];
}

}  // namespace

namespace {
// f(chunks of 8 per thread when a row of n is held in registers; 0: two passes over the row).
template <class F>
void with_row_chunks(int n, F f) {
  if (n <= 2048) f(Int<1>{});
  else if (n <= 4096) f(Int<2>{});
  else if (n <= 8192) f(Int<4>{});
  else f(Int<0>{});
}
}  // namespace

hipError_t launch_rmsnorm_planes(const void* x, int x_bf16, const float* w, int rows, int n, float eps,
                                 bf16* out_hi, bf16* out_lo, hipStream_t s) {
  if (rows <= 0) return hipSuccess;
  with_row_chunks(n, [&](auto nr) {
    constexpr int NR = decltype(nr)::value;
    if (x_bf16)
      hipLaunchKernelGGL((rmsnorm_kernel<bf16, NR>), dim3(rows), dim3(256), 0, s, (const bf16*)x, w, n, eps, out_hi,
                         out_lo, HeadClear{});
    else
      hipLaunchKernelGGL((rmsnorm_kernel<float, NR>), dim3(rows), dim3(256), 0, s, (const float*)x, w, n, eps, out_hi,
                         out_lo, HeadClear{});
  });
  return hipGetLastError();
}

hipError_t launch_head_norm(const HeadArgs& a, int status_words, const float* x, const float* w, int n, float eps,
                            bf16* out, hipStream_t s) {
  const int rows = a.B * a.k;
  if (rows <= 0) return hipSuccess;
  HeadClear clr;
  clr.status = a.status;
  clr.words = status_words;
  clr.keys = a.keys;
  with_row_chunks(n, [&](auto nr) {
    hipLaunchKernelGGL((rmsnorm_kernel<float, decltype(nr)::value, true>), dim3(rows), dim3(256), 0, s, x, w, n, eps, out,
                       (bf16*)nullptr, clr);
  });
  return hipGetLastError();
}

hipError_t launch_sum_rmsnorm_planes(Parts sum, const void* r, int r_bf16, float* x_out, const float* w, int rows,
                                     int n, float eps, bf16* out_hi, bf16* out_lo, hipStream_t s) {
  if (rows <= 0) return hipSuccess;
  if (n % 8 || !r) return hipErrorInvalidValue;
  auto launch = [&](auto nrc) {
    hipLaunchKernelGGL((sum_rmsnorm_kernel<decltype(nrc)::value>), dim3(rows), dim3(1024), 0, s, sum, r, r_bf16, x_out, w,
                       n, eps, out_hi, out_lo);
  };
  if (n <= 4096) launch(Int<1>{});
  else if (n <= 8192) launch(Int<2>{});
  else launch(Int<0>{});
  return hipGetLastError();
}

hipError_t launch_conv_split(const ConvArgs& a, hipStream_t s) {
  const int di = a.H * a.P, gn = a.G * a.N;
  const int dproj = 2 * di + 2 * gn + a.H;
  const int total = di + 2 * gn + a.H;
  if (dproj % 4 == 0 && di % 4 == 0 && gn % 4 == 0 && a.H % 4 == 0 && a.K == 4) {
    const int gx = (total / 4 + 255) / 256;
    const bool few = (long long)gx * a.B * ((a.T + 3) / 4) < 512;   // fewer than two workgroups per CU
    const dim3 grid(gx, few ? a.B * a.T : a.B * ((a.T + 3) / 4));
    if (few) {
      if (a.w_bf16) hipLaunchKernelGGL((conv4_tok_kernel<bf16, 1, false>), grid, dim3(256), 0, s, a);
      else hipLaunchKernelGGL((conv4_tok_kernel<float, 1, false>), grid, dim3(256), 0, s, a);
    } else if (a.zxbcdt.np == 1) {   // (64 registers against 86: 1024 tokens of 8448 channels 22.1 -> 19.7 us)
      if (a.w_bf16) hipLaunchKernelGGL((conv4_tok_kernel<bf16, 4, true>), grid, dim3(256), 0, s, a);
      else hipLaunchKernelGGL((conv4_tok_kernel<float, 4, true>), grid, dim3(256), 0, s, a);
    } else {
      if (a.w_bf16) hipLaunchKernelGGL((conv4_tok_kernel<bf16, 4, false>), grid, dim3(256), 0, s, a);
      else hipLaunchKernelGGL((conv4_tok_kernel<float, 4, false>), grid, dim3(256), 0, s, a);
    }
    return hipGetLastError();
  }
  if (dproj % 4 == 0 && di % 4 == 0 && gn % 4 == 0 && a.H % 4 == 0 && a.K <= 8) {
    dim3 grid((total / 4 + 255) / 256, a.B);
    if (a.w_bf16) hipLaunchKernelGGL(conv_split4_kernel<bf16>, grid, dim3(256), 0, s, a);
    else hipLaunchKernelGGL(conv_split4_kernel<float>, grid, dim3(256), 0, s, a);
    return hipGetLastError();
  }
  dim3 grid((total + 255) / 256, a.B * a.T);
  if (a.w_bf16) hipLaunchKernelGGL(conv_split_kernel<bf16>, grid, dim3(256), 0, s, a);
  else hipLaunchKernelGGL(conv_split_kernel<float>, grid, dim3(256), 0, s, a);
  return hipGetLastError();
}

hipError_t launch_gated_rmsnorm(const float* y, Parts z, int z_ld, const float* w, int rows, int n, int G,
                                float eps, bf16* out_hi, bf16* out_lo, hipStream_t s) {
  if (rows <= 0) return hipSuccess;
  const int gs = n / G;
  if (z_ld % 4 == 0 && gs % 4 == 0 && gs % 8 == 0 && gs <= 4096)
    hipLaunchKernelGGL((gated_rmsnorm_kernel<true, 2>), dim3(rows * G), dim3(256), 0, s, y, z, z_ld, w, n, G, eps, out_hi, out_lo);
  else if (z_ld % 4 == 0 && gs % 4 == 0 && gs % 8 == 0 && gs <= 8192 && z.np == 1)   // (59 registers against 124)
    hipLaunchKernelGGL((gated_rmsnorm_kernel<true, 4, true>), dim3(rows * G), dim3(256), 0, s, y, z, z_ld, w, n, G, eps, out_hi, out_lo);
  else if (z_ld % 4 == 0 && gs % 4 == 0 && gs % 8 == 0 && gs <= 8192)
    hipLaunchKernelGGL((gated_rmsnorm_kernel<true, 4>), dim3(rows * G), dim3(256), 0, s, y, z, z_ld, w, n, G, eps, out_hi, out_lo);
  else if (z_ld % 4 == 0 && gs % 4 == 0)
    hipLaunchKernelGGL((gated_rmsnorm_kernel<true, 0>), dim3(rows * G), dim3(256), 0, s, y, z, z_ld, w, n, G, eps, out_hi, out_lo);
  else
    hipLaunchKernelGGL((gated_rmsnorm_kernel<false, 0>), dim3(rows * G), dim3(256), 0, s, y, z, z_ld, w, n, G, eps, out_hi, out_lo);
  return hipGetLastError();
}

hipError_t launch_qk_norm_rope(Parts qkv, const float* qw, const float* kw, const int32_t* ctx_lens, int B,
                               int T, int Hq, int Hkv, int D, float eps, double theta, bf16* q_hi, bf16* q_lo,
                               bf16* k_hi, bf16* k_lo, bf16* v_hi, bf16* v_lo, hipStream_t s, const AttnArgs* plan,
                               int plan_clear) {
  if (B * T <= 0) return hipSuccess;
  if (D < 8 || D % 8 || D > 512 || 64 % (D / 8)) return hipErrorInvalidValue;
  if (plan && plan->B > kWorklistFusedMax) return hipErrorInvalidValue;
  // Products of many tokens come whole (np = 1); their instances do without the registers of the other planes,
  // which leave two waves per SIMD instead of five (188 registers against 90): 1024 tokens of 48 heads
  // 15.8 -> 10.8 us, 2048 of 80 heads 40.4 -> 27.3.
  auto launch = [&](auto with_plan, auto one) {
    constexpr bool PLAN = decltype(with_plan)::value != 0, ONE = decltype(one)::value != 0;
    hipLaunchKernelGGL((qk_norm_rope4_kernel<PLAN, ONE>), dim3(B * T + (PLAN ? 1 : 0)), dim3(256), 0, s, qkv, qw, kw,
                       ctx_lens, T, Hq, Hkv, D, eps, log2(theta), q_hi, q_lo, k_hi, k_lo, v_hi, v_lo,
                       PLAN ? *plan : AttnArgs{}, plan_clear);
  };
  if (plan) {
    if (qkv.np == 1) launch(Int<1>{}, Int<1>{});
    else launch(Int<1>{}, Int<0>{});
  } else {
    if (qkv.np == 1) launch(Int<0>{}, Int<1>{});
    else launch(Int<0>{}, Int<0>{});
  }
  return hipGetLastError();
}

hipError_t launch_split_planes(const SplitArgs& a, hipStream_t s) {
  size_t most = 0;
  for (int i = 0; i < a.n; ++i) most = a.len[i] > most ? a.len[i] : most;
  if (most == 0) return hipSuccess;
  size_t blocks = (most / 4 + 255) / 256;
  blocks = blocks < 1 ? 1 : blocks > 16384 ? 16384 : blocks;
  hipLaunchKernelGGL(split_kernel, dim3((unsigned)blocks, a.n), dim3(256), 0, s, a);
  return hipGetLastError();
}

hipError_t launch_silu_mul(Parts gu, int rows, int ff, bf16* hi, bf16* lo, hipStream_t s) {
  if (rows <= 0 || ff <= 0) return hipSuccess;
  if (ff % 4) return hipErrorInvalidValue;
  hipLaunchKernelGGL(silu_mul_kernel, dim3((ff / 4 + 255) / 256, rows), dim3(256), 0, s, gu, ff, hi, lo);
  return hipGetLastError();
}

hipError_t launch_kv_append(const AppendArgs& a, hipStream_t s) {
  if (a.B * a.n <= 0 || a.n_layers <= 0) return hipSuccess;
  if (a.head0 < 0 || a.head1 <= a.head0 || a.head1 > a.n_layers * 2 * a.Hkv) return hipErrorInvalidValue;
  if (a.D < 8 || a.D % 8 || a.D > 512 || 64 % (a.D / 8) || a.n_layers > AppendArgs::kMaxLayers) return hipErrorInvalidValue;
  if (a.cache_bf16) hipLaunchKernelGGL(kv_append_kernel<bf16>, dim3(a.B * a.n), dim3(256), 0, s, a, log2(a.rope_theta));
  else hipLaunchKernelGGL(kv_append_kernel<float>, dim3(a.B * a.n), dim3(256), 0, s, a, log2(a.rope_theta));
  return hipGetLastError();
}

hipError_t launch_zero_words(int* p, int n, hipStream_t s) {
  hipLaunchKernelGGL(zero_kernel, dim3(1), dim3(64), 0, s, p, n);
  return hipGetLastError();
}

hipError_t launch_copy_f32(const float* x, size_t n, float* y, hipStream_t s) {
  if (n == 0) return hipSuccess;
  const size_t blocks = (n + 255) / 256;
  hipLaunchKernelGGL(copy_kernel, dim3((unsigned)(blocks < 4096 ? blocks : 4096)), dim3(256), 0, s, x, n, y);
  return hipGetLastError();
}

}  // namespace hspec
