// Chunked SSD scan of the Mamba-2 selective recurrence from an injected initial state
// (H-Spec Sec. 3.3.1: the Mamba kernel starts from the projected last-token state and
// evaluates every draft position in one pass).
//
// Per head (scalar decay a_t = exp(dt_t A)), within a chunk with l_t = sum_{u<=t} dt_u A:
//   y_t = exp(l_t) C_t S_in^T + sum_{s<=t} exp(l_t - l_s) dt_s (C_t . B_s) x_s + D x_t
//   S_out = exp(l_end) S_in + sum_s exp(l_end - l_s) dt_s x_s (outer) B_s
// One wave owns one (request, head).  C S_in^T (16 x N x 64), C B^T (16 x N x 16) and the
// intra-chunk product of the 16 x 16 decay-weighted mixing matrix M with x (M as hi/lo planes) run on
// v_mfma_f32_16x16x32_bf16; operands given as bf16 hi/lo planes use three products so fp32
// values survive.  The chunk-local cumulative sum of dt*A is a 16-lane shuffle scan.
//   * One chunk and no final state (ssd_scan_one): the initial state is read straight from global
//     memory into MFMA fragments (as bf16 hi/lo planes, or as one fp16 plane multiplied with C
//     rounded to fp16 on v_mfma_f32_16x16x32_f16); M and the x tile go through LDS in fp32.
//   * With the fp16 plane and heads in groups of 4 that share B and C (the drafting step),
//     ssd_scan_grp runs those 4 heads in one workgroup, one wave each, and shares the C and C B^T
//     work through LDS.
//   * Otherwise (ssd_scan_state) the fp32 state stays in the accumulators of its own update from S0
//     to S_final; x and B lie in LDS as they are, M never leaves its registers.
#include "common.h"
#include "kernels.h"

namespace hspec {

namespace {

constexpr int P = 64;
constexpr int QMAX = 16;

__device__ __forceinline__ bf16x8 ld8_or0(const bf16* p, bool ok) { return ok ? ld8(p) : zero8(); }

__device__ __forceinline__ void split8(const float* v, bf16x8& hi, bf16x8& lo) {
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    const bf16 h = f2bf(v[e]);
    hi[e] = h;
    lo[e] = f2bf(v[e] - bf2f(h));
  }
}

// Intra-chunk term M x on v_mfma_f32_16x16x32_bf16: A = M (row t = lane % 16, k = s), B = x^T
// (k = s, column p = 16 pb + lane % 16); k = 16..31 are zero.  Both fp32 tiles enter as bf16
// hi/lo planes (three products).  Lane gets rows t = 4 (lane / 16) + i of column p, the layout
// of the state term.  M is zero for s > t and outside the chunk, x^T for s outside it.
__device__ __forceinline__ void mix_mfma(const float* Mm, const float* xT, int lane, f32x4 (&mx)[4]) {
  const int g4 = lane >> 4, l16 = lane & 15;
  float v[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) v[e] = g4 < 2 ? Mm[l16 * (QMAX + 1) + 8 * g4 + e] : 0.f;
  bf16x8 mh, ml;
  split8(v, mh, ml);
#pragma unroll
  for (int pb = 0; pb < 4; ++pb) {
#pragma unroll
    for (int e = 0; e < 8; ++e) v[e] = g4 < 2 ? xT[(16 * pb + l16) * (QMAX + 1) + 8 * g4 + e] : 0.f;
    bf16x8 xh, xl;
    split8(v, xh, xl);
    mx[pb] = mma16(mh, xh, f32x4{0.f, 0.f, 0.f, 0.f});
    mx[pb] = mma16(ml, xh, mx[pb]);
    mx[pb] = mma16(mh, xl, mx[pb]);
  }
}

typedef short s16x4 __attribute__((ext_vector_type(4)));
#define LDS_AS __attribute__((address_space(3)))

// Orders a wave's LDS writes before its own later reads (a wave's LDS accesses execute in order;
// this keeps the compiler from exchanging them).
__device__ __forceinline__ void wave_lds_fence() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Elements (row 4 g4 + i, column of this lane) of a 16 x 16 piece of a row-major bf16 tile in LDS,
// i = 0..3: the transposing read takes four columns at a time, piece q = lane % 4 of each row.
__device__ __forceinline__ bf16x4 ld_tr(const bf16* p) {
  return __builtin_bit_cast(bf16x4, __builtin_amdgcn_ds_read_tr16_b64_v4i16((LDS_AS s16x4*)p));
}
__device__ __forceinline__ bf16x8 cat4(bf16x4 a, bf16x4 b) {
  return __builtin_shufflevector(a, b, 0, 1, 2, 3, 4, 5, 6, 7);
}
__device__ __forceinline__ void split4(const float* v, bf16x4& hi, bf16x4& lo) {
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    hi[e] = f2bf(v[e]);
    lo[e] = f2bf(v[e] - bf2f(hi[e]));
  }
}

// Several chunks, or a final state: one wave per (request, head), four to a workgroup, each on its
// own.  Bound by HBM (the fp32 final state is two thirds of the bytes at one to three chunks), so
// the state stays in registers from S0 to S_final, as the accumulators of its own update:
//   * S^T in 16 x 16 blocks, columns p.  The rows of a block pair are ordered so that lane group
//     g4 holds n = 32 j + 8 g4 .. + 7: S0 and S_final move in 16-byte pieces, and the pair is, as
//     it stands, the k operand of C S^T (split into bf16 hi/lo planes).
//   * B C^T comes out with a lane's four rows s = 4 g4 + i of column t, which is the A operand of
//     M x; x and B are staged in LDS as they are and read transposed (ds_read_b64_tr_b16).
//   * k = 16 tokens fill half of v_mfma_f32_16x16x32_bf16: the other half takes the lo plane of M
//     and of W X against the same x and B, so a hi/lo product costs one instruction.
// Measured at B = 64, H = 128, N = 128, bf16 (was: state in LDS, one wave of 47 KB per workgroup,
// three per CU): T = 40 with S_final 500 -> 136 us (3.9 TB/s).
template <int N, bool LO>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(LO ? 1 : 2))) ssd_scan_state(ScanArgs a) {
  if (a.clear && blockIdx.x == 0 && threadIdx.x < kStatusClear) a.clear[threadIdx.x] = 0;
  constexpr int NJ = (N + 31) / 32;
  constexpr int XP = P + 16, BP = (N < 32 ? 32 : N) + 16;   // LDS row pitches, elements
  constexpr int NPL = LO ? 2 : 1;
  __shared__ __align__(16) bf16 xs_all[4][NPL][QMAX * XP];
  __shared__ __align__(16) bf16 bs_all[4][NPL][QMAX * BP];
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lane = threadIdx.x & 63, g4 = lane >> 4, l16 = lane & 15;
  const int H = a.H, T = a.T, G = a.G;
  const long long unit = (long long)blockIdx.x * 4 + wave;
  if (unit >= (long long)a.B * H) return;
  const int b = (int)(unit / H), h = (int)(unit % H), grp = h / (H / G);
  bf16* xs = xs_all[wave][0];
  bf16* bs = bs_all[wave][0];
  constexpr int XLO = QMAX * XP, BLO = QMAX * BP;   // the lo planes' offsets
  const size_t s0_off = (size_t)unit * P * N;

  // ---- S0: lane holds n = 32 j + 8 g4 .. + 7 of rows p = 16 pb + l16; every load of a plane is
  // issued before the first is used
  f32x4 st[2 * NJ][4];
  auto s0_plane = [&](const void* base, bool f16, bool add) __attribute__((always_inline)) {
    u32x4 raw[NJ][4];
#pragma unroll
    for (int j = 0; j < NJ; ++j)
#pragma unroll
      for (int pb = 0; pb < 4; ++pb) {
        const int n = 32 * j + 8 * g4;
        raw[j][pb] = *reinterpret_cast<const u32x4*>(reinterpret_cast<const uint16_t*>(base) + s0_off +
                                                     (size_t)(16 * pb + l16) * N + (n < N ? n : 0));
      }
#pragma unroll
    for (int j = 0; j < NJ; ++j)
#pragma unroll
      for (int pb = 0; pb < 4; ++pb) {
        const bool in = 32 * j + 8 * g4 < N;
        const bf16x8 bv = __builtin_bit_cast(bf16x8, raw[j][pb]);
        const f16x8 hv = __builtin_bit_cast(f16x8, raw[j][pb]);
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          const float v = in ? (f16 ? (float)hv[e] : bf2f(bv[e])) : 0.f;
          f32x4& d = st[2 * j + e / 4][pb];
          d[e % 4] = add ? d[e % 4] + v : v;
        }
      }
  };
  if (a.S0_h16) {
    s0_plane(a.S0_h16, true, false);
  } else if (a.S0_hi) {
    s0_plane(a.S0_hi, false, false);
    if (LO && a.S0_lo) s0_plane(a.S0_lo, false, true);
  } else {
#pragma unroll
    for (int nb = 0; nb < 2 * NJ; ++nb)
#pragma unroll
      for (int pb = 0; pb < 4; ++pb) st[nb][pb] = f32x4{0.f, 0.f, 0.f, 0.f};
  }
  const float Ah = a.A_is_log ? -__expf(a.A[h]) : a.A[h], Dh = a.Dskip[h];

  // ---- a chunk's inputs, loaded while the chunk before updates the state: buffer loads from the
  // chunk's first token, whose ranges end with the chunk (later tokens and absent planes read zero)
  constexpr int NB = N >= 32 ? N / 32 : 1;   // 16-byte pieces of a B row per lane (4 lanes a row; N = 16: 2)
  struct ChunkIn {
    float dtv;
    u32x4 x[NPL][2], bt[NPL][NB], c[NPL][NJ];
  };
  const int rt = lane >> 2, rq = lane & 3;   // this lane's row and quarter of the x and B tiles
  const bool bq = N >= 32 || rq < 2;
  const int x_vo = (rt * a.x_ld + 16 * rq) * 2, b_vo = bq ? (rt * a.bc_ld + 8 * NB * rq) * 2 : BUF_OOB;
  const int c_vo = 8 * g4 < N ? (l16 * a.bc_ld + 8 * g4) * 2 : BUF_OOB, dt_vo = l16 * a.dt_ld * 4;
  auto load_chunk = [&](int c0, ChunkIn& r) __attribute__((always_inline)) {
    const int Qc = min(a.chunk, T - c0);
    const size_t tok0 = (size_t)b * T + c0;
    r.dtv = __uint_as_float(
        __builtin_amdgcn_raw_buffer_load_b32(rsrc(a.dt + tok0 * a.dt_ld + h, (Qc * a.dt_ld - h) * 4), dt_vo, 0, 0));
    const size_t xo = tok0 * a.x_ld + (size_t)h * P, bo = tok0 * a.bc_ld + (size_t)grp * N;
    const int xr = (Qc * a.x_ld - h * P) * 2, br = (Qc * a.bc_ld - grp * N) * 2;
#pragma unroll
    for (int pl = 0; pl < NPL; ++pl) {
      const bf16 *xp = pl ? a.x_lo : a.x_hi, *bp = pl ? a.B_lo : a.B_hi, *cp = pl ? a.C_lo : a.C_hi;
      const __amdgpu_buffer_rsrc_t xs_r = rsrc(xp + xo, xp ? xr : 0), bs_r = rsrc(bp + bo, bp ? br : 0),
                                   cs_r = rsrc(cp + bo, cp ? br : 0);
#pragma unroll
      for (int i = 0; i < 2; ++i) r.x[pl][i] = __builtin_amdgcn_raw_buffer_load_b128(xs_r, x_vo + 16 * i, 0, 0);
#pragma unroll
      for (int i = 0; i < NB; ++i) r.bt[pl][i] = __builtin_amdgcn_raw_buffer_load_b128(bs_r, b_vo + 16 * i, 0, 0);
#pragma unroll
      for (int j = 0; j < NJ; ++j) r.c[pl][j] = __builtin_amdgcn_raw_buffer_load_b128(cs_r, c_vo + 64 * j, 0, 0);
    }
  };
  const int y_vo = (4 * g4 * H * P + l16) * 4;
  if (N < 32) {   // columns 16..31 of the B tile are zero throughout
#pragma unroll
    for (int pl = 0; pl < NPL; ++pl)
      if (rq < 2) *reinterpret_cast<bf16x8*>(bs + pl * BLO + rt * BP + 16 + 8 * rq) = zero8();
  }
  ChunkIn nx;
  load_chunk(0, nx);

  for (int c0 = 0; c0 < T; c0 += a.chunk) {
    const int Qc = min(a.chunk, T - c0);
    const ChunkIn cur = nx;
    wave_lds_fence();   // the previous chunk's tiles have been read
#pragma unroll
    for (int pl = 0; pl < NPL; ++pl) {
#pragma unroll
      for (int i = 0; i < 2; ++i) *reinterpret_cast<u32x4*>(xs + (pl * XLO + rt * XP + 16 * rq + 8 * i)) = cur.x[pl][i];
      if (bq) {
#pragma unroll
        for (int i = 0; i < NB; ++i) *reinterpret_cast<u32x4*>(bs + (pl * BLO + rt * BP + 8 * (rq * NB + i))) = cur.bt[pl][i];
      }
    }
    bf16x8 cf[NPL][NJ];
#pragma unroll
    for (int pl = 0; pl < NPL; ++pl)
#pragma unroll
      for (int j = 0; j < NJ; ++j) cf[pl][j] = __builtin_bit_cast(bf16x8, cur.c[pl][j]);
    wave_lds_fence();

    // ---- l_t, the inclusive cumulative sum of dt A (lane l16 of every group holds token l16)
    const float dtv = cur.dtv;
    float cum = dtv * Ah;
#pragma unroll
    for (int off = 1; off < 16; off <<= 1) {
      const float v = __shfl_up(cum, off, 16);
      if (l16 >= off) cum += v;
    }
    const float ell_end = __shfl(cum, 15);   // (dt is zero past the chunk)
    float ell[4], dts[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      ell[i] = __shfl(cum, 4 * g4 + i);
      dts[i] = __shfl(dtv, 4 * g4 + i);
    }

    // ---- B C^T: rows s = 4 g4 + i, column t = l16; then M[t][s] as the A operand of M x
    f32x4 cb = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int j = 0; j < NJ; ++j) {
      const bf16x8 bf = *reinterpret_cast<const bf16x8*>(bs + l16 * BP + 32 * j + 8 * g4);
      cb = mma16(bf, cf[0][j], cb);
      if constexpr (LO) {
        cb = mma16(bf, cf[NPL - 1][j], cb);
        cb = mma16(*reinterpret_cast<const bf16x8*>(bs + BLO + l16 * BP + 32 * j + 8 * g4), cf[0][j], cb);
      }
    }
    float mv[4], wv[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const bool ok = 4 * g4 + i <= l16 && l16 < Qc;
      mv[i] = ok ? cb[i] * __expf(cum - ell[i]) * dts[i] : 0.f;
      wv[i] = __expf(ell_end - ell[i]) * dts[i];
    }
    const bf16x4 z4 = {(bf16)0.f, (bf16)0.f, (bf16)0.f, (bf16)0.f};
    bf16x4 mh, ml;
    split4(mv, mh, ml);

    // ---- per 16 columns p: C S^T from the state before this chunk, then with x of tokens
    // 4 g4 + i the output y = exp(l_t) C S^T + M x + D x (rows t = 4 g4 + i) and W X
    float dec[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) dec[i] = __expf(ell[i]);
    // (the buffer's range ends with the chunk: rows past it are dropped)
    const __amdgpu_buffer_rsrc_t yr = rsrc(a.y + ((size_t)b * T + c0) * H * P + (size_t)h * P, (Qc * H - h) * P * 4);
    bf16x8 wx[4];
#pragma unroll
    for (int pb = 0; pb < 4; ++pb) {
      f32x4 ys = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int j = 0; j < NJ; ++j) {
        float v[8];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          v[e] = st[2 * j][pb][e];
          v[4 + e] = st[2 * j + 1][pb][e];
        }
        bf16x8 sh, sl;
        split8(v, sh, sl);
        ys = mma16(cf[0][j], sh, ys);
        if constexpr (LO) ys = mma16(cf[NPL - 1][j], sh, ys);
        ys = mma16(cf[0][j], sl, ys);
      }
      const int o = (4 * g4 + (l16 >> 2)) * XP + 16 * pb + 4 * (l16 & 3);
      const bf16x4 xh = ld_tr(xs + o);
      f32x4 y = mma16(cat4(mh, ml), cat4(xh, xh), f32x4{0.f, 0.f, 0.f, 0.f});
      float xv[4], w[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) xv[i] = bf2f(xh[i]);
      if constexpr (LO) {
        const bf16x4 xl = ld_tr(xs + XLO + o);
        y = mma16(cat4(mh, z4), cat4(xl, z4), y);
#pragma unroll
        for (int i = 0; i < 4; ++i) xv[i] += bf2f(xl[i]);
      }
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const float out = dec[i] * ys[i] + Dh * xv[i] + y[i];
        __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(out), yr, y_vo + i * H * P * 4 + 64 * pb, 0, 0);
        w[i] = wv[i] * xv[i];
      }
      bf16x4 wh, wl;
      split4(w, wh, wl);
      wx[pb] = cat4(wh, wl);
      __builtin_amdgcn_sched_barrier(0);   // (one column block's planes of S at a time: registers)
    }
    __builtin_amdgcn_sched_barrier(0);
    if (c0 + a.chunk < T) load_chunk(c0 + a.chunk, nx);   // (here: C's registers are free)
    // ---- S^T <- exp(l_end) S^T + B^T (W X)
    const float de = __expf(ell_end);
#pragma unroll
    for (int nb = 0; nb < 2 * NJ; ++nb) {
      // rows of block nb: position 4 q + i is n = 32 (nb / 2) + 8 q + 4 (nb % 2) + i
      const int o = (4 * g4 + (l16 >> 2)) * BP + 32 * (nb / 2) + 4 * (nb & 1) + 8 * (l16 & 3);
      const bf16x4 bh = ld_tr(bs + o);
      const bf16x8 bb = cat4(bh, bh);
      bf16x8 bl = zero8();
      if constexpr (LO) bl = cat4(ld_tr(bs + BLO + o), z4);
#pragma unroll
      for (int pb = 0; pb < 4; ++pb) {
        st[nb][pb] = mma16(bb, wx[pb], st[nb][pb] * de);
        if constexpr (LO) st[nb][pb] = mma16(bl, wx[pb], st[nb][pb]);
      }
    }
  }

  if (a.S_final) {
    // 16-byte stores where the caller's buffer allows them
    const bool vec = (reinterpret_cast<uintptr_t>(a.S_final) & 15) == 0;
#pragma unroll
    for (int pb = 0; pb < 4; ++pb)
#pragma unroll
      for (int nb = 0; nb < 2 * NJ; ++nb) {
        const int n = 32 * (nb / 2) + 8 * g4 + 4 * (nb & 1);
        if (n >= N) continue;
        float* dst = a.S_final + s0_off + (size_t)(16 * pb + l16) * N + n;
        if (vec) {
          *reinterpret_cast<f32x4*>(dst) = st[nb][pb];
        } else {
#pragma unroll
          for (int e = 0; e < 4; ++e) dst[e] = st[nb][pb][e];
        }
      }
  }
}

// The block in one chunk and no final state (every drafting step): the same arithmetic as
// ssd_scan_state, with every global load of the wave (dt, the x tile, the B and C
// fragments, all initial-state fragments) issued before the first is used, so that a wave
// waits for memory once instead of once per state fragment.
template <int N, bool H16>
__global__ void __launch_bounds__(64) ssd_scan_one(ScanArgs a) {
  if (a.clear && blockIdx.x == 0 && threadIdx.x < kStatusClear) a.clear[threadIdx.x] = 0;
  constexpr int NS = (N + 31) / 32;
  __shared__ float xT[P * (QMAX + 1)];   // x^T tile, fp32, padded rows
  __shared__ float Mm[QMAX * (QMAX + 1)];

  const int H = a.H, T = a.T, G = a.G;
  const int b = blockIdx.x / H, h = blockIdx.x % H;
  const int grp = h / (H / G);
  const int lane = threadIdx.x, g4 = lane >> 4, l16 = lane & 15;
  const size_t s0_off = ((size_t)b * H + h) * P * N;

  // ---- loads, in order of use
  const float dtv = l16 < T ? a.dt[(size_t)(b * T + l16) * a.dt_ld + h] : 0.f;
  // x tile: lane holds x[t = lane / 4][p = 16 (lane % 4) .. + 15]
  const int xt = lane >> 2, xp = 16 * (lane & 3);
  const bool xok = xt < T;
  const size_t xoff = (size_t)(b * T + xt) * a.x_ld + (size_t)h * P + xp;
  const bf16x8 xh0 = ld8_or0(a.x_hi + xoff, xok), xh1 = ld8_or0(a.x_hi + xoff + 8, xok);
  const bf16x8 xl0 = a.x_lo ? ld8_or0(a.x_lo + xoff, xok) : zero8();
  const bf16x8 xl1 = a.x_lo ? ld8_or0(a.x_lo + xoff + 8, xok) : zero8();
  // C (A operand, rows t) and B (B operand, columns s) fragments over n
  bf16x8 cf[NS], cfl[NS], bfr[NS], bfl[NS];
  const size_t tok_t = (size_t)(b * T + l16) * a.bc_ld + (size_t)grp * N;
#pragma unroll
  for (int ns = 0; ns < NS; ++ns) {
    const int n = 32 * ns + 8 * g4;
    const bool ok = l16 < T && n < N;
    cf[ns] = ld8_or0(a.C_hi + tok_t + n, ok);
    cfl[ns] = a.C_lo ? ld8_or0(a.C_lo + tok_t + n, ok) : zero8();
    bfr[ns] = ld8_or0(a.B_hi + tok_t + n, ok);
    bfl[ns] = a.B_lo ? ld8_or0(a.B_lo + tok_t + n, ok) : zero8();
  }
  // initial state as B operand of C S^T: column p = 16 pb + l16, n = 32 ns + 8 g4 ..  (H16: one
  // fp16 plane, multiplied with C rounded to fp16; otherwise bf16 hi/lo planes)
  bf16x8 sh[4][H16 ? 1 : NS], sl[4][H16 ? 1 : NS];
  f16x8 s16[4][H16 ? NS : 1];
#pragma unroll
  for (int pb = 0; pb < 4; ++pb)
#pragma unroll
    for (int ns = 0; ns < NS; ++ns) {
      const int n = 32 * ns + 8 * g4;
      const size_t off = s0_off + (size_t)(16 * pb + l16) * N + n;
      if constexpr (H16) {
        s16[pb][ns] = n < N ? *reinterpret_cast<const f16x8*>(a.S0_h16 + off) : f16x8{};
      } else {
        const bool ok = a.S0_hi != nullptr && n < N;
        sh[pb][ns] = ld8_or0(a.S0_hi + off, ok);
        sl[pb][ns] = a.S0_lo != nullptr ? ld8_or0(a.S0_lo + off, ok) : zero8();
      }
    }
  const float Ah = a.A_is_log ? -__expf(a.A[h]) : a.A[h], Dh = a.Dskip[h];

  // ---- inclusive cumulative sum of dt*A over the chunk (lanes 0..15)
  float cum = dtv * Ah;
#pragma unroll
  for (int off = 1; off < 16; off <<= 1) {
    const float v = __shfl_up(cum, off, 16);
    if (l16 >= off) cum += v;
  }
  // ---- x^T tile in LDS
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    xT[(xp + e) * (QMAX + 1) + xt] = bf2f(xh0[e]) + bf2f(xl0[e]);
    xT[(xp + 8 + e) * (QMAX + 1) + xt] = bf2f(xh1[e]) + bf2f(xl1[e]);
  }
  // ---- C B^T: lane gets rows t = 4 g4 + i, column s = l16
  f32x4 cb = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int ns = 0; ns < NS; ++ns) {
    cb = mma16(cf[ns], bfr[ns], cb);
    if (a.C_lo) cb = mma16(cfl[ns], bfr[ns], cb);
    if (a.B_lo) cb = mma16(cf[ns], bfl[ns], cb);
  }
  // ---- state term C S^T: lane gets rows t = 4 g4 + i, column p = 16 pb + l16
  f32x4 ys[4];
  if constexpr (H16) {
    f16x8 c16[NS];   // C (hi + lo) rounded once to fp16
#pragma unroll
    for (int ns = 0; ns < NS; ++ns)
#pragma unroll
      for (int e = 0; e < 8; ++e) c16[ns][e] = (_Float16)(bf2f(cf[ns][e]) + bf2f(cfl[ns][e]));
#pragma unroll
    for (int pb = 0; pb < 4; ++pb) {
      ys[pb] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int ns = 0; ns < NS; ++ns) ys[pb] = mma16h(c16[ns], s16[pb][ns], ys[pb]);
    }
  } else {
#pragma unroll
    for (int pb = 0; pb < 4; ++pb) {
      ys[pb] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int ns = 0; ns < NS; ++ns) {
        ys[pb] = mma16(cf[ns], sh[pb][ns], ys[pb]);
        if (a.C_lo) ys[pb] = mma16(cfl[ns], sh[pb][ns], ys[pb]);
        if (a.S0_lo) ys[pb] = mma16(cf[ns], sl[pb][ns], ys[pb]);
      }
    }
  }
  // ---- decay-weighted mixing matrix M[t][s] = (C_t . B_s) exp(l_t - l_s) dt_s for s <= t
  const float ell_s = __shfl(cum, l16);
  const float dt_s = __shfl(dtv, l16);
  float ell_t[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int t = 4 * g4 + i;
    ell_t[i] = __shfl(cum, t);
    const bool ok = l16 <= t && t < T;
    Mm[t * (QMAX + 1) + l16] = ok ? cb[i] * __expf(ell_t[i] - ell_s) * dt_s : 0.f;
  }
  __syncthreads();
  // ---- y = exp(l_t) (C S^T) + M x + D x, M x on MFMA (every entry of both tiles is written
  // above: M is zero for s > t and past the block, x^T for s past it)
  f32x4 mx[4];
  mix_mfma(Mm, xT, lane, mx);
#pragma unroll
  for (int pb = 0; pb < 4; ++pb) {
    const int p = 16 * pb + l16;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int t = 4 * g4 + i;
      const float acc = __expf(ell_t[i]) * ys[pb][i] + Dh * xT[p * (QMAX + 1) + t] + mx[pb][i];
      if (t < T) a.y[(size_t)(b * T + t) * H * P + (size_t)h * P + p] = acc;
    }
  }
}

// The drafting step's case (one chunk, no final state, S0 as one fp16 plane) with HW waves per
// workgroup, one per head, for HW heads of one request that read the same B and C.  Each wave
// loads only its own head's S0, dt and x, so it holds a third fewer registers than
// ssd_scan_one and more waves stay resident; wave w loads the w-th (mod HW) 32-wide slices of
// C and B, rounds its C slice to fp16 into LDS and leaves its part of C B^T there, and every
// wave adds the parts in slice order.  The arithmetic is ssd_scan_one<N, true>'s: C S0^T as
// sum over slices of fp16 products, C B^T from the hi/lo planes, the rest unchanged.
constexpr int SCAN_HW = 4;
template <int N>
__global__ void __launch_bounds__(64 * SCAN_HW) __attribute__((amdgpu_waves_per_eu(4))) ssd_scan_grp(ScanArgs a) {
  if (a.clear && blockIdx.x == 0 && threadIdx.x < kStatusClear) a.clear[threadIdx.x] = 0;
  constexpr int NS = (N + 31) / 32;
  constexpr int CP = N + 8;   // fp16 C row pitch (16 bytes of padding)
  __shared__ float xT_all[SCAN_HW][P * (QMAX + 1)];
  __shared__ float Mm_all[SCAN_HW][QMAX * (QMAX + 1)];
  __shared__ __align__(16) _Float16 c16s[QMAX * CP];   // C rounded to fp16, rows t
  __shared__ f32x4 cbp[NS][64];                         // parts of C B^T, one per slice

  const int H = a.H, T = a.T, G = a.G;
  // (the wave index made visibly uniform: the head's A, D and offsets become scalar values)
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lane = threadIdx.x & 63, g4 = lane >> 4, l16 = lane & 15;
  const int hpb = H / SCAN_HW;                          // workgroups per request
  const int b = blockIdx.x / hpb, h = (blockIdx.x % hpb) * SCAN_HW + wave;
  const int grp = h / (H / G);                          // the same for the workgroup's heads
  const size_t s0_off = ((size_t)b * H + h) * P * N;
  float* xT = xT_all[wave];
  float* Mm = Mm_all[wave];

  // ---- loads, in order of use: dt and x of this head, this wave's slices of C and B, S0.
  // Lanes past the block read token 0 (no branch around a load, whose merged value would
  // have to arrive before the next load is issued) and drop the value where it is used.
  const bool tok_ok = l16 < T;
  const float dt_raw = a.dt[(size_t)(b * T + (tok_ok ? l16 : 0)) * a.dt_ld + h];
  const int xt = lane >> 2, xp = 16 * (lane & 3);
  const bool xok = xt < T;
  const size_t xoff = (size_t)(b * T + (xok ? xt : 0)) * a.x_ld + (size_t)h * P + xp;
  const bf16x8 xh0 = ld8(a.x_hi + xoff), xh1 = ld8(a.x_hi + xoff + 8);
  // (lo planes: the hi plane is read in their place when there is none, and dropped)
  const bf16* x_lo = a.x_lo ? a.x_lo : a.x_hi;
  const bf16x8 xl0 = ld8(x_lo + xoff), xl1 = ld8(x_lo + xoff + 8);
  const size_t tok_t = (size_t)(b * T + (tok_ok ? l16 : 0)) * a.bc_ld + (size_t)grp * N;
  constexpr int NSW = (NS + SCAN_HW - 1) / SCAN_HW;    // slices per wave
  bf16x8 cf[NSW], cfl[NSW], bfr[NSW], bfl[NSW];
#pragma unroll
  for (int kk = 0; kk < NSW; ++kk) {
    const int ns = wave + SCAN_HW * kk;
    const int n = 32 * ns + 8 * g4;
    const int nc = ns < NS && n < N ? n : 0;   // (in range; the value is dropped below)
    cf[kk] = ld8(a.C_hi + tok_t + nc);
    cfl[kk] = ld8((a.C_lo ? a.C_lo : a.C_hi) + tok_t + nc);
    bfr[kk] = ld8(a.B_hi + tok_t + nc);
    bfl[kk] = ld8((a.B_lo ? a.B_lo : a.B_hi) + tok_t + nc);
  }
  f16x8 s16[4][NS];
#pragma unroll
  for (int pb = 0; pb < 4; ++pb)
#pragma unroll
    for (int ns = 0; ns < NS; ++ns) {
      const int n = 32 * ns + 8 * g4;
      s16[pb][ns] = n < N ? *reinterpret_cast<const f16x8*>(a.S0_h16 + s0_off + (size_t)(16 * pb + l16) * N + n)
                          : f16x8{};
    }
  const float Ah = a.A_is_log ? -__expf(a.A[h]) : a.A[h], Dh = a.Dskip[h];

  // ---- this wave's C slices (fp16, rows t = l16) and parts of C B^T into LDS
#pragma unroll
  for (int kk = 0; kk < NSW; ++kk) {
    const int ns = wave + SCAN_HW * kk;
    if (ns < NS) {   // (uniform: ns depends on the wave only)
      // the C and B rows of tokens past the block, and columns past N, are zero
      const bool ok = tok_ok && 32 * ns + 8 * g4 < N;
      const bf16x8 cv = ok ? cf[kk] : zero8(), cvl = ok && a.C_lo ? cfl[kk] : zero8();
      const bf16x8 bv = ok ? bfr[kk] : zero8(), bvl = ok && a.B_lo ? bfl[kk] : zero8();
      f32x4 part = {0.f, 0.f, 0.f, 0.f};
      part = mma16(cv, bv, part);
      if (a.C_lo) part = mma16(cvl, bv, part);
      if (a.B_lo) part = mma16(cv, bvl, part);
      cbp[ns][lane] = part;
      f16x8 c;
#pragma unroll
      for (int e = 0; e < 8; ++e) c[e] = (_Float16)(bf2f(cv[e]) + bf2f(cvl[e]));
      if (32 * ns + 8 * g4 < N) *reinterpret_cast<f16x8*>(c16s + l16 * CP + 32 * ns + 8 * g4) = c;
    }
  }
  // ---- inclusive cumulative sum of dt*A over the chunk (lanes 0..15)
  const float dtv = tok_ok ? dt_raw : 0.f;
  float cum = dtv * Ah;
#pragma unroll
  for (int off = 1; off < 16; off <<= 1) {
    const float v = __shfl_up(cum, off, 16);
    if (l16 >= off) cum += v;
  }
  // ---- x^T tile of this head in LDS (zero past the block)
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    xT[(xp + e) * (QMAX + 1) + xt] = xok ? bf2f(xh0[e]) + (a.x_lo ? bf2f(xl0[e]) : 0.f) : 0.f;
    xT[(xp + 8 + e) * (QMAX + 1) + xt] = xok ? bf2f(xh1[e]) + (a.x_lo ? bf2f(xl1[e]) : 0.f) : 0.f;
  }
  __syncthreads();   // C slices and parts of C B^T from every wave
  // ---- C B^T: lane gets rows t = 4 g4 + i, column s = l16 (parts added in slice order)
  f32x4 cb = cbp[0][lane];
#pragma unroll
  for (int ns = 1; ns < NS; ++ns) cb += cbp[ns][lane];
  // ---- state term C S^T: lane gets rows t = 4 g4 + i, column p = 16 pb + l16
  f32x4 ys[4];
#pragma unroll
  for (int pb = 0; pb < 4; ++pb) ys[pb] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int ns = 0; ns < NS; ++ns) {
    const int n = 32 * ns + 8 * g4;   // (columns past N, N = 16: zero, as S0 is there)
    const f16x8 c = n < N ? *reinterpret_cast<const f16x8*>(c16s + l16 * CP + n) : f16x8{};
#pragma unroll
    for (int pb = 0; pb < 4; ++pb) ys[pb] = mma16h(c, s16[pb][ns], ys[pb]);
  }
  // ---- decay-weighted mixing matrix M[t][s] = (C_t . B_s) exp(l_t - l_s) dt_s for s <= t
  const float ell_s = __shfl(cum, l16);
  const float dt_s = __shfl(dtv, l16);
  float ell_t[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int t = 4 * g4 + i;
    ell_t[i] = __shfl(cum, t);
    const bool ok = l16 <= t && t < T;
    Mm[t * (QMAX + 1) + l16] = ok ? cb[i] * __expf(ell_t[i] - ell_s) * dt_s : 0.f;
  }
  __syncthreads();   // (each wave reads only its own tiles; one barrier for the LDS writes)
  // ---- y = exp(l_t) (C S^T) + M x + D x
  f32x4 mx[4];
  mix_mfma(Mm, xT, lane, mx);
#pragma unroll
  for (int pb = 0; pb < 4; ++pb) {
    const int p = 16 * pb + l16;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int t = 4 * g4 + i;
      const float acc = __expf(ell_t[i]) * ys[pb][i] + Dh * xT[p * (QMAX + 1) + t] + mx[pb][i];
      if (t < T) a.y[(size_t)(b * T + t) * H * P + (size_t)h * P + p] = acc;
    }
  }
}

template <int N>
hipError_t launch_n(const ScanArgs& a, hipStream_t s) {
  const bool multi = a.S_final != nullptr || a.T > a.chunk;
  if (multi) {
    const unsigned grid = (unsigned)(((long long)a.B * a.H + 3) / 4);
    if (a.x_lo || a.B_lo || a.C_lo || a.S0_lo) hipLaunchKernelGGL((ssd_scan_state<N, true>), dim3(grid), dim3(256), 0, s, a);
    else hipLaunchKernelGGL((ssd_scan_state<N, false>), dim3(grid), dim3(256), 0, s, a);
  } else {
    // heads in groups of SCAN_HW that share B and C: one workgroup per group of heads
    const bool grouped = a.S0_h16 && a.H % SCAN_HW == 0 && (a.H / a.G) % SCAN_HW == 0;
    if (grouped) hipLaunchKernelGGL(ssd_scan_grp<N>, dim3(a.B * (a.H / SCAN_HW)), dim3(64 * SCAN_HW), 0, s, a);
    else if (a.S0_h16) hipLaunchKernelGGL((ssd_scan_one<N, true>), dim3(a.B * a.H), dim3(64), 0, s, a);
    else hipLaunchKernelGGL((ssd_scan_one<N, false>), dim3(a.B * a.H), dim3(64), 0, s, a);
  }
  return hipGetLastError();
}

}  // namespace

hipError_t launch_ssd_scan(const ScanArgs& a, hipStream_t s) {
  if (a.B <= 0 || a.T <= 0 || a.H <= 0) return hipSuccess;
  if (a.P != P || a.chunk < 1 || a.chunk > QMAX) return hipErrorInvalidValue;
  switch (a.N) {
    case 16: return launch_n<16>(a, s);
    case 32: return launch_n<32>(a, s);
    case 64: return launch_n<64>(a, s);
    case 128: return launch_n<128>(a, s);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace hspec
