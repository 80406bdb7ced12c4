// Draft head: the Markov correction of the block's logits and the choice of draft tokens
// (Sec. 3.3.3 causal correction; App. B.1 "Markov rank"; App. B.2 "Pruned drafter vocabulary").
//
// Position j of request b gets the logits of the LM head plus a rank-R term picked by the token
// chosen at position j - 1:
//   l'[b, j, v] = base[b, j, v] + sum_r E[t_{b, j-1}, r] U[v, r],   t_{b, -1} = prev[b],
// and its token is the argmax over v of l' (greedy) or of l' / T + G (Gumbel-max sampling with
// the caller's noise G).  The chain is sequential in j, so each position is one launch, unless the
// caller forces the tokens (then all positions are one):
//   * a workgroup owns 128 vocabulary columns and all requests (in tiles of 64);
//   * the rank-R product is one MFMA tile per (16 requests, 16 columns); the E rows of the
//     previous tokens are gathered into LDS once per workgroup, the U rows of a wave's columns
//     read from L2;
//   * the argmax across workgroups is a 64-bit atomicMax on (orderable score << 32 | ~column),
//     which picks the largest score and, among equal scores, the lowest column; a position has
//     kHeadSlots keys, so that at most 1 / kHeadSlots of the workgroups meet on one address;
//   * the next launch decodes the previous position's token from those keys.
#include "common.h"
#include "kernels.h"

namespace hspec {
namespace {

constexpr int MK_COLS = 128;   // vocabulary columns per workgroup (rank 256: 8 waves x 16; others: 4 waves x 2 x 16)
constexpr int MK_ROWS = 64;    // requests per tile (4 MFMA row blocks)
constexpr int ST_BAD_TOKEN = 4;
constexpr int ST_NONFINITE = 8;

// Order-preserving map of a float that is no NaN to uint32 (larger float, larger key, never 0).
__device__ __forceinline__ unsigned score_ord(float s) {
  const unsigned u = __float_as_uint(s);
  return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}
__device__ __forceinline__ int key_token(unsigned long long key) {
  return (int)~(unsigned)(key & 0xffffffffu);
}
// Best key of a position over its slots.
__device__ __forceinline__ unsigned long long best_key(const unsigned long long* keys) {
  unsigned long long m = keys[0];
#pragma unroll
  for (int i = 1; i < kHeadSlots; ++i) m = keys[i] > m ? keys[i] : m;
  return m;
}
// Maximum over the 16 lanes of a DPP row, in every lane.
__device__ __forceinline__ unsigned row_max(unsigned v) {
  v = max(v, (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, 0x128, 0xf, 0xf, true));   // row_ror:8, 4, 2, 1
  v = max(v, (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, 0x124, 0xf, 0xf, true));
  v = max(v, (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, 0x122, 0xf, 0xf, true));
  return max(v, (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, 0x121, 0xf, 0xf, true));
}
__device__ __forceinline__ unsigned long long shfl_xor_u64(unsigned long long v, int m) {
  const unsigned lo = __shfl_xor((unsigned)(v & 0xffffffffu), m);
  const unsigned hi = __shfl_xor((unsigned)(v >> 32), m);
  return ((unsigned long long)hi << 32) | lo;
}

// Corrected logits and scores of a wave's 32 columns x 64 requests, and each request's best
// (score, column) among them.
__device__ __forceinline__ void score_tile(const HeadArgs& a, int j, int b0, int vw, int lane, const float (&base)[4][4][2],
                                           const f32x4 (&acc)[4][2], unsigned long long* best) {
  const int l16 = lane & 15, g4 = lane >> 4;
  bool bad = false;
#pragma unroll
  for (int rb = 0; rb < 4; ++rb)
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int r = rb * 16 + 4 * g4 + i, b = b0 + r;
      unsigned ord[2];
#pragma unroll
      for (int cb = 0; cb < 2; ++cb) {
        const int col = vw + cb * 16 + l16;
        ord[cb] = 0;   // (below every score's key)
        if (b < a.B && col < a.V) {
          const size_t off = ((size_t)b * a.k + j) * a.V + col;
          const float l = base[rb][i][cb] + acc[rb][cb][i];
          if (a.logits) a.logits[off] = l;
          float sc = a.gumbel ? l * a.inv_temp + a.gumbel[off] : l;
          if (!(sc == sc)) {
            bad = true;
            sc = -INFINITY;
          }
          ord[cb] = score_ord(sc);
        }
      }
      // the largest score of the 32 columns, and among its columns the lowest
      const unsigned o = max(ord[0], ord[1]);
      const unsigned col = vw + (ord[0] >= ord[1] ? 0 : 16) + l16;
      const unsigned top = row_max(o), low = row_max(o == top && o ? ~col : 0u);
      if (l16 == 0) best[r] = ((unsigned long long)top << 32) | low;
    }
  if (bad) set_status(a.status, ST_NONFINITE);
}

// The workgroup's best of each request of the tile into this workgroup's slot of the position's keys.
template <int NW>
__device__ __forceinline__ void merge_best(const HeadArgs& a, int j, int b0, const unsigned long long (&s_best)[NW][MK_ROWS]) {
  const int tid = threadIdx.x;
  if (tid < MK_ROWS && b0 + tid < a.B) {
    unsigned long long best = s_best[0][tid];
#pragma unroll
    for (int w = 1; w < NW; ++w) best = s_best[w][tid] > best ? s_best[w][tid] : best;
    if (best) atomicMax(a.keys + ((size_t)(b0 + tid) * a.k + j) * kHeadSlots + blockIdx.x % kHeadSlots, best);
  }
}

// Any rank that is a multiple of 32: E and U fragments read from L2, one round of loads per 32.
__global__ void __launch_bounds__(256) markov_step_any(HeadArgs a, int j0) {
  __shared__ int s_prev[MK_ROWS];
  __shared__ unsigned long long s_best[4][MK_ROWS];
  const int j = j0 + blockIdx.y;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int vw = blockIdx.x * MK_COLS + wave * 32;   // first column of this wave
  const int l16 = lane & 15, g4 = lane >> 4;

  for (int b0 = 0; b0 < a.B; b0 += MK_ROWS) {
    if (tid < MK_ROWS) {
      const int b = b0 + tid;
      int t = 0;
      if (b < a.B) {
        if (j == 0) t = a.prev[b];
        else if (a.forced) t = a.forced[(size_t)b * a.k + j - 1];
        else t = key_token(best_key(a.keys + ((size_t)b * a.k + j - 1) * kHeadSlots));
        if (t < 0 || t >= a.V) {
          if (blockIdx.x == 0) set_status(a.status, ST_BAD_TOKEN);
          t = 0;
        }
      }
      s_prev[tid] = t;
    }
    __syncthreads();

    // this tile's LM-head logits, loaded while the rank product runs
    float base[4][4][2];
#pragma unroll
    for (int rb = 0; rb < 4; ++rb)
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int cb = 0; cb < 2; ++cb) {
          const int b = b0 + rb * 16 + 4 * g4 + i, col = vw + cb * 16 + l16;
          base[rb][i][cb] = (b < a.B && col < a.V) ? a.base[((size_t)b * a.k + j) * a.V + col] : 0.f;
        }

    // adj[b][v] = E[prev_b] . U[v] over the rank
    f32x4 acc[4][2];
#pragma unroll
    for (int rb = 0; rb < 4; ++rb)
#pragma unroll
      for (int cb = 0; cb < 2; ++cb) acc[rb][cb] = f32x4{0.f, 0.f, 0.f, 0.f};
    const bf16* urow[2];
    bool ucol[2];
#pragma unroll
    for (int cb = 0; cb < 2; ++cb) {
      const int col = vw + cb * 16 + l16;
      ucol[cb] = col < a.V;
      urow[cb] = a.U + (size_t)(ucol[cb] ? col : 0) * a.R + 8 * g4;
    }
    const bf16* erow[4];
#pragma unroll
    for (int rb = 0; rb < 4; ++rb) erow[rb] = a.E + (size_t)s_prev[rb * 16 + l16] * a.R + 8 * g4;
    for (int ks = 0; ks < a.R; ks += 32) {
      bf16x8 ef[4], uf[2];
#pragma unroll
      for (int rb = 0; rb < 4; ++rb) ef[rb] = ld8(erow[rb] + ks);
#pragma unroll
      for (int cb = 0; cb < 2; ++cb) uf[cb] = ucol[cb] ? ld8(urow[cb] + ks) : zero8();
#pragma unroll
      for (int rb = 0; rb < 4; ++rb)
#pragma unroll
        for (int cb = 0; cb < 2; ++cb) acc[rb][cb] = mma16(ef[rb], uf[cb], acc[rb][cb]);
    }
    score_tile(a, j, b0, vw, lane, base, acc, s_best[wave]);
    __syncthreads();
    merge_best<4>(a, j, b0, s_best);
    __syncthreads();   // s_prev and s_best are reused by the next request tile
  }
}

// Rank 256.  A position is one round of workgroups, so its time is one workgroup's: eight waves of
// 16 columns, every load that depends on nothing (keys, U fragments, LM-head logits) issued before the keys
// are waited for, then the E rows gathered into LDS; range-checked buffer accesses instead of branches
// around each logit, maxima over 16 lanes by DPP, row blocks without requests skipped.
// At 64 requests, V = 32000: 17.2 -> 13.4 us a position; 7 forced positions of 3 requests 93 -> 24 us.
// (Half the waves gathering E while the other half loaded U and the logits: 15.8 and 58 us; the time went
// into 32 branches around the logits of each lane.)
template <bool GUM, bool LOGITS>
__global__ void __launch_bounds__(512) markov_step_256(HeadArgs a, int j0) {
  constexpr int R = 256, RK = R / 32, LDE = R + 8;   // E rows in LDS, padded by 16 bytes
  constexpr int NW = 8;
  __shared__ unsigned long long s_best[NW][MK_ROWS];
  __shared__ __align__(16) bf16 s_e[MK_ROWS * LDE];
  const int j = j0 + blockIdx.y;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l16 = lane & 15, g4 = lane >> 4;
  const int col = blockIdx.x * MK_COLS + wave * 16 + l16;
  const int row = tid >> 3, q = tid & 7;   // gather: eight lanes per request
  const int kV = a.k * a.V;                // elements between a position's logits of two requests
  bf16x8 uf[RK];
  for (int b0 = 0; b0 < a.B; b0 += MK_ROWS) {
    const int rows = min(MK_ROWS, a.B - b0), b = b0 + row;
    // ---- the preceding token: given, or one of the position's keys per lane
    static_assert(kHeadSlots == 8, "one key per gathering lane");
    const bool chain = j > 0 && !a.forced;
    unsigned long long key = 0;
    int t = 0;
    if (row < rows) {
      if (chain) key = a.keys[((size_t)b * a.k + j - 1) * kHeadSlots + q];
      else t = j == 0 ? a.prev[b] : a.forced[(size_t)b * a.k + j - 1];
    }
    __builtin_amdgcn_sched_barrier(0);
    // ---- U fragments of this wave's columns (once), this tile's logits and noise
    if (b0 == 0) {
      const bf16* urow = a.U + (size_t)min(col, a.V - 1) * R + 8 * g4;   // (columns past V are never scored)
#pragma unroll
      for (int s = 0; s < RK; ++s) uf[s] = ld8(urow + 32 * s);
    }
    const size_t t0 = ((size_t)b0 * a.k + j) * a.V;
    const int span = ((rows - 1) * kV + a.V) * 4;
    const int vo = col < a.V ? (4 * g4 * kV + col) * 4 : BUF_OOB;   // row 4 g4 + i + 16 rb: + (i + 16 rb) kV
    const __amdgpu_buffer_rsrc_t r_base = rsrc(a.base + t0, span);
    float base[4][4], gum[4][4];
#pragma unroll
    for (int rb = 0; rb < 4; ++rb)
#pragma unroll
      for (int i = 0; i < 4; ++i)
        base[rb][i] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(r_base, vo + (16 * rb + i) * kV * 4, 0, 0));
    if constexpr (GUM) {
      const __amdgpu_buffer_rsrc_t r_gum = rsrc(a.gumbel + t0, span);
#pragma unroll
      for (int rb = 0; rb < 4; ++rb)
#pragma unroll
        for (int i = 0; i < 4; ++i)
          gum[rb][i] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(r_gum, vo + (16 * rb + i) * kV * 4, 0, 0));
    }
    __builtin_amdgcn_sched_barrier(0);
    // ---- E rows of the preceding tokens into LDS
    if (chain) {
#pragma unroll
      for (int x = 1; x < 8; x <<= 1) {
        const unsigned long long o = shfl_xor_u64(key, x);
        key = o > key ? o : key;
      }
      t = key_token(key);
    }
    if (row < rows) {
      if (t < 0 || t >= a.V) {
        if (blockIdx.x == 0 && q == 0) set_status(a.status, ST_BAD_TOKEN);
        t = 0;
      }
      const bf16* src = a.E + (size_t)t * R + q * (R / 8);
      bf16x8 e[R / 64];
#pragma unroll
      for (int i = 0; i < R / 64; ++i) e[i] = ld8(src + 8 * i);
#pragma unroll
      for (int i = 0; i < R / 64; ++i) *reinterpret_cast<bf16x8*>(s_e + (row * LDE + q * (R / 8) + 8 * i)) = e[i];
    }
    __syncthreads();
    // ---- product, corrected logits, and each request's best (score, column) of the wave
    const __amdgpu_buffer_rsrc_t r_log = rsrc(LOGITS ? a.logits + t0 : nullptr, LOGITS ? span : 0);
    bool bad = false;
#pragma unroll
    for (int rb = 0; rb < 4; ++rb) {
      if (16 * rb >= rows) continue;   // (uniform)
      f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int s = 0; s < RK; ++s)
        acc = mma16(*reinterpret_cast<const bf16x8*>(s_e + ((rb * 16 + l16) * LDE + 32 * s + 8 * g4)), uf[s], acc);
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int r = rb * 16 + 4 * g4 + i;
        const bool in = r < rows && col < a.V;
        const float l = base[rb][i] + acc[i];
        if constexpr (LOGITS)
          __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(l), r_log, vo + (16 * rb + i) * kV * 4, 0, 0);
        float sc = l;
        if constexpr (GUM) sc = l * a.inv_temp + gum[rb][i];
        const bool nan = !(sc == sc);
        bad |= in && nan;
        const unsigned o = in ? score_ord(nan ? -INFINITY : sc) : 0u;   // (0: below every score's key)
        // the largest score of the 16 columns, and among its columns the lowest
        const unsigned top = row_max(o), low = row_max(o == top && o ? ~(unsigned)col : 0u);
        if (l16 == 0) s_best[wave][r] = ((unsigned long long)top << 32) | low;
      }
    }
    if (bad) set_status(a.status, ST_NONFINITE);
    __syncthreads();
    merge_best<NW>(a, j, b0, s_best);
    __syncthreads();   // s_e and s_best are reused by the next request tile
  }
}

__global__ void head_tokens_kernel(const unsigned long long* keys, int n, int32_t* tokens) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) tokens[i] = key_token(best_key(keys + (size_t)i * kHeadSlots));
}

}  // namespace

hipError_t launch_markov_head(const HeadArgs& a, hipStream_t s) {
  if (a.B <= 0 || a.k <= 0) return hipSuccess;
  const int n = a.B * a.k;
  const int cols = (a.V + MK_COLS - 1) / MK_COLS;
  // forced tokens: every position is known, one launch takes them all
  const bool all = a.forced != nullptr && a.k <= 65535;
  // rank 256, and a tile's logits within 31-bit byte offsets
  const bool fast = a.R == 256 && (long long)(MK_ROWS + 16) * a.k * a.V * 4 < BUF_OOB;
  for (int j = 0; j < (all ? 1 : a.k); ++j) {
    const dim3 grid(cols, all ? a.k : 1);
    if (fast) {
      auto kern = a.gumbel ? (a.logits ? markov_step_256<true, true> : markov_step_256<true, false>)
                           : (a.logits ? markov_step_256<false, true> : markov_step_256<false, false>);
      hipLaunchKernelGGL(kern, grid, dim3(512), 0, s, a, j);
    } else {
      hipLaunchKernelGGL(markov_step_any, grid, dim3(256), 0, s, a, j);
    }
    if (hipError_t e = hipGetLastError()) return e;
  }
  hipLaunchKernelGGL(head_tokens_kernel, dim3((n + 255) / 256), dim3(256), 0, s, a.keys, n, a.tokens);
  return hipGetLastError();
}

}  // namespace hspec
