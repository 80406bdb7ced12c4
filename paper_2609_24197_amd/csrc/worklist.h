// Work list of the KV sweep, built on the device from the context lengths.  Shared by the
// work-list kernel of the attention calls and by the q/k-norm + RoPE launch, which builds it in
// one extra workgroup so that the list costs no launch of its own inside a drafting step.
#pragma once
#include <climits>

#include "common.h"
#include "kernels.h"

namespace hspec {

constexpr int MAX_SPLIT = kMaxSplit;   // keys per split (host-enforced by the config check)
constexpr int WL_LOG_THREADS = 8, WL_THREADS = 1 << WL_LOG_THREADS;   // threads of a workgroup that builds the list
constexpr int WL_NCAND = 64;      // split sizes tried under automatic splitting (one lane each)
static_assert(WL_NCAND <= 64 && (WL_NCAND & (WL_NCAND - 1)) == 0, "one lane of a wave per candidate size");

__device__ __forceinline__ int clamp_len(const AttnArgs& a, int L) {
  int cap = a.max_pages * a.ps;
  if (cap > a.max_ctx_len) cap = a.max_ctx_len;
  if (L < 0 || L > cap) {
    set_status(a.status, ST_BAD_CTX_LEN);
    L = L < 0 ? 0 : cap;
  }
  return L;
}

// First cache position a sweep reads for a request of length L.  Under a sliding window the
// query at position L + j sees cache positions p >= L + j - window + 1, so no query of the
// block sees p < L - window + 1; those positions are not read at all.
__device__ __forceinline__ int swept_lo(const AttnArgs& a, int L) {
  return a.window > 0 && L - a.window + 1 > 0 ? L - a.window + 1 : 0;
}

// Splits of one request.  The swept range [swept_lo, L) of n positions is cut into ns runs:
// every run but the last holds q positions (a whole number of 32-key tiles, at most MAX_SPLIT),
// the last one the rest, and ns = ceil(n / q), so no run is empty.  n = 0 is one split with no
// cache keys.  The work-list kernel picks (ns, q) per request and stores them; the sweep and
// the reductions read them back, so all three cut a request the same way.
__device__ __forceinline__ int swept_n(const AttnArgs& a, int L) { return L - swept_lo(a, L); }

// ceil(n / s) for 0 <= n < 2^22 and 1 <= s < 2^22, with rs = rcp(s): a float estimate of the quotient,
// off by at most one, then corrected by the exact remainder.  No branch and no integer division.
__device__ __forceinline__ int ceil_div_f(int n, int s, float rs) {
  const float fn = (float)n, fs = (float)s;
  float q = __builtin_floorf(fn * rs);
  const float r = __builtin_fmaf(-q, fs, fn);   // exact: in (-s, 2 s), or -s where s divides n
  q += (r > 0.f ? 1.f : 0.f) + (r > fs ? 1.f : 0.f) - (r <= -fs ? 1.f : 0.f);
  return (int)q;
}

// Splits of a request of n swept positions (at most 256 x MAX_SPLIT: host-enforced) when splits may hold up
// to S positions (rs = rcp(S); S is at most MAX_SPLIT: host-enforced).
__device__ __forceinline__ int plan_pieces(int n, int S, float rs, int cap) {
  return max(1, min(ceil_div_f(n, S, rs), cap));
}

// (split length, splits) of a request: ceil(n / ns) rounded up to a whole tile, and what that leaves.
__device__ __forceinline__ int2 plan_request(int n, int S, float rs, int cap) {
  if (n <= 0) return int2{0, 1};
  const int ns = plan_pieces(n, S, rs, cap);
  const int q = (ceil_div_f(n, ns, __builtin_amdgcn_rcpf((float)ns)) + 31) & ~31;
  return int2{q, ceil_div_f(n, q, __builtin_amdgcn_rcpf((float)q))};
}

// Inclusive prefix sum over the workgroup (WL_THREADS lanes); total in *total.
__device__ __forceinline__ int plan_scan(int v, int* s_wave, int* total) {
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const int u = __shfl_up(v, o);
    if (lane >= o) v += u;
  }
  __syncthreads();   // s_wave free from the previous scan
  if (lane == 63) s_wave[w] = v;
  __syncthreads();
  int before = 0, all = 0;
#pragma unroll
  for (int i = 0; i < WL_THREADS / 64; ++i) {
    before += i < w ? s_wave[i] : 0;
    all += s_wave[i];
  }
  *total = all;
  return v + before;
}

// LDS of the builder: per-request arrays for up to RANK_MAX (a power of two) requests.
template <int RANK_MAX>
struct WorklistLds {
  static_assert(RANK_MAX <= 4096 && RANK_MAX % WL_THREADS == 0, "request index in 12 bits of a rank word");
  int len[RANK_MAX];             // context length of request b
  alignas(16) int n[RANK_MAX];   // its swept positions; later its first item
  // its rank word: split length / 32 (9 bits) | 4095 - b (12 bits) | splits (10 bits).  A larger
  // word goes earlier in the list.
  alignas(16) unsigned word[RANK_MAX];
  int cnt[WL_THREADS / 64][WL_NCAND];
  int sum[WL_THREADS / 64], max[WL_THREADS / 64];
};

// Work list of the sweep: every (request, split) once, as (request << 16 | split, context
// length, split length, splits of the request), requests ordered by decreasing split length (all
// splits of a request together, ties by index), so that the persistent workgroups, taking items
// longest first, finish close together.  One workgroup of WL_THREADS threads, at most RANK_MAX
// requests.  Also resets the item queue and, as the first kernel of a call, its status words.
//
// Split size.  An explicit split size (split_tokens) is used as given.  With the automatic size
// (auto_split) the work list picks it from the actual lengths, among WL_NCAND sizes from twice
// the host's size (at most MAX_SPLIT) down to min_split: the largest size that gives every persistent
// workgroup one item of at most 1/16 above the average work, else the size whose item count
// comes closest below a whole number (two or more) of rounds of the `grid` workgroups, so that
// the last round of the queue is not left half empty.  Every request is then cut into the
// fewest near-equal runs of at most that size (at most max_splits, at most MAX_SPLIT keys).
//
// One workgroup, so a chain of latencies: each length is read once, divisions are float estimates
// with exact corrections, every wave works out the choice by itself from per-wave counts, and a
// request's first item is the sum of the splits of the requests before it, added up in the
// pass that compares their rank words (no scatter by rank, no prefix sum).  As a kernel of its own, back
// to back: 128 requests 15.1 -> 7.0 us, 256 25.5 -> 9.4, 4096 1927 -> 1134; 1 to 8 requests 7 us before and after.
template <int RANK_MAX>
__device__ void build_worklist(const AttnArgs& a, int clear_words, WorklistLds<RANK_MAX>& lds) {
  const int tid = threadIdx.x, wv = tid >> 6, ln = tid & 63;
  const int B = a.B, B4 = (B + 3) & ~3;
  const int cap = max(1, a.max_splits);
  const int auto_split = a.auto_split, min_split = a.min_split, grid = a.grid;
  asm volatile("" ::"s"(auto_split), "s"(min_split), "s"(grid));   // (all arguments read at once, not after a barrier)
  const bool choose = auto_split && grid > 0;
  const int len0 = tid < B ? a.ctx_lens[tid] : 0;   // on its way while the status words are cleared
  if (tid < clear_words) a.status[tid] = 0;
  __syncthreads();
  for (int b = tid; b < B4; b += WL_THREADS) {
    const int L = b < B ? clamp_len(a, b == tid ? len0 : a.ctx_lens[b]) : 0;
    lds.len[b] = L;
    lds.n[b] = swept_n(a, L);   // (0 past B)
    lds.word[b] = 0;            // (past B: below every request's word)
  }
  __syncthreads();
  // candidate split sizes: twice the host's size down to min_split in WL_NCAND near-even steps
  int S = max(1, a.split);
  if (choose) {
    const int hi = min(MAX_SPLIT, 2 * a.split) / 32, lo = max(1, min_split / 32);
    const int Sc = max(1, 32 * (hi - (hi - lo) * ln / (WL_NCAND - 1)));   // lane l: candidate l
    const float rs = __builtin_amdgcn_rcpf((float)Sc);
    // splits at each candidate size: wave w counts over requests 4 w .. 4 w + 3 of every 16
    int cnt = 0, sum = 0, mx = 0;
    for (int b = 4 * wv; b < B4; b += WL_THREADS / 16) {
      const int4 n = *reinterpret_cast<const int4*>(&lds.n[b]);
      cnt += plan_pieces(n.x, Sc, rs, cap) + plan_pieces(n.y, Sc, rs, cap) + plan_pieces(n.z, Sc, rs, cap) +
             plan_pieces(n.w, Sc, rs, cap) - max(0, b + 4 - B);   // (entries past B count 1)
      sum += n.x + n.y + n.z + n.w;
      mx = max(max(mx, max(n.x, n.y)), max(n.z, n.w));
    }
    lds.cnt[wv][ln] = cnt;
    if (ln == 0) {
      lds.sum[wv] = sum;
      lds.max[wv] = mx;
    }
    __syncthreads();
    // Choice, one lane per candidate: the largest size (smallest c) whose items fit one round
    // with the longest split within 1/16 of the average work per workgroup; else the size
    // leaving the fewest idle slots in the last of two or more rounds (larger size on ties).
    // (Item counts fit in 32 bits: the host bounds B x max_splits x Hkv.)
    cnt = sum = mx = 0;
#pragma unroll
    for (int w = 0; w < WL_THREADS / 64; ++w) {
      cnt += lds.cnt[w][ln];
      sum += lds.sum[w];
      mx = max(mx, lds.max[w]);
    }
    const int items = cnt * a.Hkv;
    // positions of all items, per workgroup: / grid
    const bool fits = items <= grid && (long long)min(Sc, mx) * grid * 16 <= (long long)sum * a.Hkv * 17;
    const unsigned long long one = __ballot(fits);
    if (one) {
      S = __shfl(Sc, __builtin_ctzll(one));
    } else {
      int key = INT_MAX;
      if (items > grid) {
        const int rem = (int)((unsigned)items % (unsigned)grid);
        key = (rem ? grid - rem : 0) * WL_NCAND + ln;
      }
#pragma unroll
      for (int o = 32; o > 0; o >>= 1) key = min(key, __shfl_xor(key, o));
      if (key != INT_MAX) S = __shfl(Sc, key & (WL_NCAND - 1));
    }
  }
  const float rs = __builtin_amdgcn_rcpf((float)S);
  for (int b = tid; b < B; b += WL_THREADS) {
    const int2 qn = plan_request(lds.n[b], S, rs, cap);
    lds.word[b] = (unsigned)(qn.x / 32) << 22 | (unsigned)(4095 - b) << 10 | (unsigned)qn.y;
  }
  __syncthreads();
  int total = 0;
  for (int b = tid; b < B; b += WL_THREADS) {
    const unsigned w = lds.word[b];
    int first = 0;
    total = 0;
#pragma unroll 2
    for (int o = 0; o < B4; o += 4) {
      const uint4 v = *reinterpret_cast<const uint4*>(&lds.word[o]);
      const int nx = v.x & 1023, ny = v.y & 1023, nz = v.z & 1023, nw = v.w & 1023;
      first += (v.x > w ? nx : 0) + (v.y > w ? ny : 0) + (v.z > w ? nz : 0) + (v.w > w ? nw : 0);
      total += nx + ny + nz + nw;
    }
    lds.n[b] = first;
  }
  if (tid == 0) {
    a.status[1] = total * a.Hkv;
    a.status[2] = 0;
  }
  __syncthreads();
  // 2^sh lanes write the items of one request (B 2^sh <= WL_THREADS where B is smaller)
  const int sh = B >= WL_THREADS ? 0 : B > 1 ? __builtin_clz(B - 1) - (31 - WL_LOG_THREADS) - 1 : WL_LOG_THREADS;
  for (int i = tid; i < B << sh; i += WL_THREADS) {
    const int b = i >> sh, sp0 = i & ((1 << sh) - 1);
    const unsigned w = lds.word[b];
    const int q = (int)(w >> 22) * 32, ns = (int)(w & 1023);
    int4* u = reinterpret_cast<int4*>(a.units) + lds.n[b];
    for (int sp = sp0; sp < ns; sp += 1 << sh) u[sp] = int4{(b << 16) | sp, lds.len[b], q, ns};
    if (sp0 == 0) *reinterpret_cast<int2*>(a.req + 2 * b) = int2{ns, q};
  }
}

// The same list for any number of requests, in their own order and at the host's split size: prefix
// sum of the split counts, WL_THREADS requests at a time.
__device__ inline void build_worklist_unranked(const AttnArgs& a, int clear_words) {
  __shared__ int s_wave[WL_THREADS / 64];
  const int tid = threadIdx.x;
  if (tid < clear_words) a.status[tid] = 0;
  __syncthreads();
  const int cap = max(1, a.max_splits), S = max(1, a.split);
  const float rs = __builtin_amdgcn_rcpf((float)S);
  int base = 0;
  for (int r0 = 0; r0 < a.B; r0 += WL_THREADS) {
    const int r = r0 + tid;
    int L = 0;
    int2 qn = {0, 0};
    if (r < a.B) {
      L = clamp_len(a, a.ctx_lens[r]);
      qn = plan_request(swept_n(a, L), S, rs, cap);
    }
    int total = 0;
    const int first = base + plan_scan(qn.y, s_wave, &total) - qn.y;
    if (r < a.B) {
      for (int sp = 0; sp < qn.y; ++sp)
        *reinterpret_cast<int4*>(a.units + 4 * (first + sp)) = int4{(r << 16) | sp, L, qn.x, qn.y};
      *reinterpret_cast<int2*>(a.req + 2 * r) = int2{qn.y, qn.x};
    }
    base += total;
  }
  if (tid == 0) {
    a.status[1] = base * a.Hkv;
    a.status[2] = 0;
  }
}

}  // namespace hspec
