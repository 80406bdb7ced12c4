// C ABI of the drafting step: argument validation, workspace layout, and the stream-ordered
// launch sequence of each entry point.  Host code only; every kernel lives in a .hip file.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <array>
#include <climits>
#include <cmath>
#include <cstdarg>
#include <initializer_list>
#include <cstdio>

#include "hspec.h"
#include "kernels.h"

#define HSPEC_API extern "C" __attribute__((visibility("default")))

using hspec::bf16;

namespace {

// Message of the last failing call on this thread.  A plain array: nothing in the library
// runs a destructor at thread or process exit.
thread_local char g_err[512];

void clear_err() { g_err[0] = 0; }

hspec_status fail(hspec_status s, const char* fmt, ...) {
  va_list ap;
  va_start(ap, fmt);
  vsnprintf(g_err, sizeof g_err, fmt, ap);
  va_end(ap);
  return s;
}

#define HIP_TRY(expr)                                                                        \
  do {                                                                                       \
    hipError_t e_ = (expr);                                                                  \
    if (e_ != hipSuccess) return fail(HSPEC_ERR_LAUNCH, "%s: %s", #expr, hipGetErrorString(e_)); \
  } while (0)

constexpr size_t ALIGN = 256;

#ifdef HSPEC_HOST_SANITIZE
}  // namespace
// Host sanitizer build only: told every region cut from a caller's workspace.
void hspec_host_carve(const void* p, size_t bytes);
namespace {
#endif

// Bump allocator over the caller's workspace.  With base == nullptr it only measures.
struct Arena {
  char* base = nullptr;
  size_t off = 0;
  template <class T>
  T* take(size_t count) {
    size_t o = (off + ALIGN - 1) / ALIGN * ALIGN;
    off = o + count * sizeof(T);
#ifdef HSPEC_HOST_SANITIZE
    if (base) hspec_host_carve(base + o, count * sizeof(T));
#endif
    return base ? reinterpret_cast<T*>(base + o) : nullptr;
  }
  size_t size() const { return (off + ALIGN - 1) / ALIGN * ALIGN; }
};

bool is_f32(hspec_dtype d) { return d == HSPEC_F32; }
long long ceil_div(long long a, long long b) { return (a + b - 1) / b; }
bool dtype_ok(hspec_dtype d) { return d == HSPEC_BF16 || d == HSPEC_F32; }

// A storage-dtype matrix as MFMA planes: bf16 storage is its own hi plane.  fp32 storage is split
// into (hi, lo) in the workspace for the kernels that read planes; products read it in place (f32)
// and split it on chip.
struct Planes {
  const bf16* hi = nullptr;
  const bf16* lo = nullptr;
  const float* f32 = nullptr;
};
Planes in_place(const void* src, hspec_dtype d) {
  if (is_f32(d)) return Planes{nullptr, nullptr, static_cast<const float*>(src)};
  return Planes{static_cast<const bf16*>(src), nullptr, nullptr};
}
const bf16* rows_of(const void* w) { return static_cast<const bf16*>(w); }   // (fp32 rows under GemmArgs::w_f32)
void set_a(hspec::GemmArgs& g, const Planes& a, int ld) {
  g.A_hi = a.f32 ? rows_of(a.f32) : a.hi;
  g.A_lo = a.lo;
  g.a_f32 = a.f32 != nullptr;
  g.lda = ld;
}
void set_w(hspec::GemmArgs& g, const void* w, hspec_dtype d, int ld) {
  g.W = rows_of(w);
  g.w_f32 = is_f32(d);
  g.ldw = ld;
}
struct SplitSlot {
  bf16* hi = nullptr;
  bf16* lo = nullptr;
  size_t n = 0;
};
SplitSlot reserve_split(Arena& ar, hspec_dtype d, size_t n) {
  SplitSlot s;
  if (is_f32(d)) {
    s.hi = ar.take<bf16>(n);
    s.lo = ar.take<bf16>(n);
    s.n = n;
  }
  return s;
}
// The tensors of a call that have to be split, in one launch.
struct Splits {
  hspec::SplitArgs a;
  Planes add(const void* src, hspec_dtype d, const SplitSlot& slot) {
    if (!is_f32(d)) return in_place(src, d);
    a.x[a.n] = static_cast<const float*>(src);
    a.hi[a.n] = slot.hi;
    a.lo[a.n] = slot.lo;
    a.len[a.n++] = slot.n;
    return Planes{slot.hi, slot.lo, nullptr};
  }
  hipError_t launch(hipStream_t st) const { return a.n ? hspec::launch_split_planes(a, st) : hipSuccess; }
};

// The planes Splits gave for src on an earlier call with the same workspace, without
// splitting again: src itself for bf16 storage, the workspace slot for fp32.
Planes planes_in_place(const void* src, hspec_dtype d, const SplitSlot& slot) {
  return is_f32(d) ? Planes{slot.hi, slot.lo, nullptr} : in_place(src, d);
}

// Split-K scratch shared by a sequence of GEMMs on one stream, sized for the largest.
struct GemmScratch {
  float* p = nullptr;
  size_t cap = 0;
};
GemmScratch reserve_gemm(Arena& ar, hspec_dtype d, std::initializer_list<std::array<int, 3>> mnk) {
  GemmScratch s;
  for (const auto& x : mnk) s.cap = std::max(s.cap, hspec::gemm_scratch_elems(x[0], x[1], x[2], true, is_f32(d)));
  if (s.cap) s.p = ar.take<float>(s.cap);
  return s;
}
void use_scratch(hspec::GemmArgs& g, const GemmScratch& s) {
  g.part = s.p;
  g.part_cap = s.cap;
}

// ------------------------------------------------------------------------- validation

hspec_status check_mamba(const hspec_mamba_cfg* c, const hspec_mamba_w* w, bool full) {
  if (!c || !w) return fail(HSPEC_ERR_NULL, "mamba config or weights is NULL");
  if (!dtype_ok(c->dtype)) return fail(HSPEC_ERR_DTYPE, "unknown dtype %d", (int)c->dtype);
  if (c->B <= 0 || c->d_h <= 0 || c->r <= 0 || c->H <= 0 || c->P <= 0 || c->N <= 0)
    return fail(HSPEC_ERR_SHAPE, "non-positive mamba dimension");
  if (c->P != 64) return fail(HSPEC_ERR_UNSUPPORTED, "P (head dim) must be 64, got %d", c->P);
  if (c->N != 16 && c->N != 32 && c->N != 64 && c->N != 128)
    return fail(HSPEC_ERR_UNSUPPORTED, "N (d_state) must be 16, 32, 64 or 128, got %d", c->N);
  if (c->d_h % 8 || c->r % 8) return fail(HSPEC_ERR_UNSUPPORTED, "d_h and r must be multiples of 8");
  if (c->flags & ~(unsigned)(HSPEC_W_DS_PACKED | HSPEC_MAMBA_PRECISE_IO))
    return fail(HSPEC_ERR_UNSUPPORTED, "unknown mamba flags 0x%x", c->flags);
  if ((c->flags & HSPEC_W_DS_PACKED) && (is_f32(c->dtype) || c->r % 64 || c->d_h % 32))
    return fail(HSPEC_ERR_UNSUPPORTED, "a packed W_dS needs bf16 storage, r %% 64 == 0 and d_h %% 32 == 0");
  if (!w->W_r || !w->W_dS) return fail(HSPEC_ERR_NULL, "W_r or W_dS is NULL");
  if (!full) return HSPEC_OK;
  if (c->k <= 0 || c->d_model <= 0 || c->G <= 0 || c->chunk <= 0 || c->conv_w <= 0)
    return fail(HSPEC_ERR_SHAPE, "non-positive mamba dimension");
  if (c->H % c->G) return fail(HSPEC_ERR_SHAPE, "H %% G != 0 (H=%d, G=%d)", c->H, c->G);
  if (c->chunk > 16) return fail(HSPEC_ERR_UNSUPPORTED, "chunk must be <= 16, got %d", c->chunk);
  if (c->conv_w > 8) return fail(HSPEC_ERR_UNSUPPORTED, "conv_w must be <= 8, got %d", c->conv_w);
  if (c->d_model % 8) return fail(HSPEC_ERR_UNSUPPORTED, "d_model must be a multiple of 8");
  if ((c->H * c->P) % c->G) return fail(HSPEC_ERR_SHAPE, "d_inner %% G != 0");
  if (!w->W_in || !w->conv_w || !w->conv_b || !w->dt_bias || !w->A_log || !w->D || !w->gnorm_w || !w->W_out)
    return fail(HSPEC_ERR_NULL, "a mamba weight pointer is NULL");
  return HSPEC_OK;
}

// KV heads per slot of the target cache.
int cache_heads(const hspec_attn_cfg& c) { return c.Hkv_cache > 0 ? c.Hkv_cache : c.Hkv; }

hspec_status check_attn_cfg(const hspec_attn_cfg* c, int max_ctx_len) {
  if (!c) return fail(HSPEC_ERR_NULL, "attention config is NULL");
  if (!dtype_ok(c->dtype)) return fail(HSPEC_ERR_DTYPE, "unknown dtype %d", (int)c->dtype);
  if (c->B <= 0 || c->k <= 0 || c->Hq <= 0 || c->Hkv <= 0 || c->D <= 0 || c->page_size <= 0 ||
      c->max_pages <= 0 || c->num_pages <= 0)
    return fail(HSPEC_ERR_SHAPE, "non-positive attention dimension");
  if (c->Hq % c->Hkv) return fail(HSPEC_ERR_SHAPE, "Hq %% Hkv != 0 (Hq=%d, Hkv=%d)", c->Hq, c->Hkv);
  if (c->D != 64 && c->D != 128) return fail(HSPEC_ERR_UNSUPPORTED, "D must be 64 or 128, got %d", c->D);
  if (c->flags & ~(unsigned)(HSPEC_BLOCK_CAUSAL | HSPEC_ATTN_PRECISE_IO))
    return fail(HSPEC_ERR_UNSUPPORTED, "unknown attention flags 0x%x", c->flags);
  if (c->k * (c->Hq / c->Hkv) > 128)
    return fail(HSPEC_ERR_UNSUPPORTED, "k * Hq/Hkv must be <= 128, got %d", c->k * (c->Hq / c->Hkv));
  if (c->Hkv_cache != 0 && (c->Hkv_cache < c->Hkv))
    return fail(HSPEC_ERR_SHAPE, "Hkv_cache (%d) < Hkv (%d)", c->Hkv_cache, c->Hkv);
  if (cache_heads(*c) > 16 && (c->kv_heads || c->Hkv_cache != 0))
    return fail(HSPEC_ERR_UNSUPPORTED, "KV-head reuse supports at most 16 cache heads, got %d", cache_heads(*c));
  if (c->kv_heads)
    for (int i = 0; i < c->Hkv; ++i)
      if (c->kv_heads[i] < 0 || c->kv_heads[i] >= cache_heads(*c))
        return fail(HSPEC_ERR_SHAPE, "kv_heads[%d] = %d outside [0, %d)", i, c->kv_heads[i], cache_heads(*c));
  if (c->window < 0) return fail(HSPEC_ERR_SHAPE, "window < 0");
  if (c->window > 0 && c->k > c->window) return fail(HSPEC_ERR_SHAPE, "k > window");
  if (c->split_tokens < 0 || c->split_tokens % 64)
    return fail(HSPEC_ERR_SHAPE, "split_tokens must be a non-negative multiple of 64");
  if (max_ctx_len < 0) return fail(HSPEC_ERR_SHAPE, "max_ctx_len < 0");
  if (c->B > 32767) return fail(HSPEC_ERR_UNSUPPORTED, "B must be <= 32767");
  if (c->page_size < 16 || (c->page_size & (c->page_size - 1)))
    return fail(HSPEC_ERR_UNSUPPORTED, "page_size must be a power of two >= 16, got %d", c->page_size);
  if (c->split_tokens > hspec::kMaxSplit)
    return fail(HSPEC_ERR_UNSUPPORTED, "split_tokens must be <= %d", hspec::kMaxSplit);
  const int swept = hspec::attention_swept_len(max_ctx_len, c->window);
  const int split = c->split_tokens > 0 ? c->split_tokens : hspec::attention_default_split(c->B, c->Hkv, swept);
  if (swept > 0 && ceil_div(swept, split) > 256)
    return fail(HSPEC_ERR_UNSUPPORTED, "swept context / split_tokens gives more than 256 splits");
  if ((long long)c->B * c->Hkv * (swept > 0 ? ceil_div(swept, 64) : 1) > 0x7fffffffLL)
    return fail(HSPEC_ERR_UNSUPPORTED, "B x Hkv x swept context is too large for the work list");
  if (split > hspec::kMaxSplit)   // the sweep holds one split's page ids in a fixed LDS array
    return fail(HSPEC_ERR_UNSUPPORTED, "swept context of %d keys needs splits above %d keys (at most 256 x %d)",
                swept, hspec::kMaxSplit, hspec::kMaxSplit);
  return HSPEC_OK;
}

hspec_status check_attn_w(const hspec_attn_cfg* c, const hspec_attn_w* w) {
  if (!w) return fail(HSPEC_ERR_NULL, "attention weights is NULL");
  if (!w->W_q || !w->W_k || !w->W_v || !w->W_o || !w->q_norm_w || !w->k_norm_w)
    return fail(HSPEC_ERR_NULL, "an attention weight pointer is NULL");
  if (c->d_model <= 0 || c->d_model % 8) return fail(HSPEC_ERR_UNSUPPORTED, "d_model must be a positive multiple of 8");
  return HSPEC_OK;
}

hspec_status check_ws(void* ws, size_t have, size_t need) {
  if (!ws) return fail(HSPEC_ERR_WORKSPACE, "workspace is NULL");
  if (reinterpret_cast<uintptr_t>(ws) % ALIGN) return fail(HSPEC_ERR_WORKSPACE, "workspace is not 256-byte aligned");
  if (have < need) return fail(HSPEC_ERR_WORKSPACE, "workspace has %zu bytes, needs %zu", have, need);
  return HSPEC_OK;
}

// ---------------------------------------------------------------------- layout + launch

// F enters Proj_dS with the packed (fp16) W_dS as fp16 planes of F x 2^-kFScaleLog2, which
// Proj_r writes directly: finite for |F| < 65504 x 64 (about 4e6), full fp16 precision down to
// |F| = 2^-8, and an absolute error under 2^-19 below that.
constexpr int kFScaleLog2 = 6;

struct StatePlan {
  GemmScratch gs;
  bf16 *F_hi = nullptr, *F_lo = nullptr;        // bf16 planes of F (unpacked W_dS)
  _Float16 *F_h16 = nullptr, *F_l16 = nullptr;  // fp16 planes of F (packed W_dS; l16 only precise)
  bf16 *S0_hi = nullptr, *S0_lo = nullptr;
  _Float16* S0_h16 = nullptr;
};

void plan_state(Arena& ar, const hspec_mamba_cfg& c, bool s0_planes, StatePlan& p) {
  const size_t dS = (size_t)c.H * c.P * c.N;
  if (c.flags & HSPEC_W_DS_PACKED) {
    // one fp16 plane (11 significant bits), or hi/lo fp16 planes with HSPEC_MAMBA_PRECISE_IO
    p.F_h16 = ar.take<_Float16>((size_t)c.B * c.r);
    if (c.flags & HSPEC_MAMBA_PRECISE_IO) p.F_l16 = ar.take<_Float16>((size_t)c.B * c.r);
  } else {
    p.F_hi = ar.take<bf16>((size_t)c.B * c.r);
    p.F_lo = ar.take<bf16>((size_t)c.B * c.r);
  }
  p.gs = reserve_gemm(ar, c.dtype, {{c.B, c.r, c.d_h}, {c.B, (int)dS, c.r}});
  if (s0_planes) {
    // S0 only feeds the scan: one fp16 plane (11 significant bits, half the bytes of hi/lo
    // bf16 planes) where the state projection runs on the weight-streaming path, else hi/lo
    if (!is_f32(c.dtype) && hspec::gemm_f16_out_ok(c.B, (int)dS, c.r)) {
      p.S0_h16 = ar.take<_Float16>((size_t)c.B * dS);
    } else {
      p.S0_hi = ar.take<bf16>((size_t)c.B * dS);
      p.S0_lo = ar.take<bf16>((size_t)c.B * dS);
    }
  }
}

// F = W_r h_last (bf16 planes, or fp16 planes for the packed W_dS), then S0 = W_dS F (fp32,
// bf16 planes and/or one fp16 plane).
hspec_status run_state(const hspec_mamba_cfg& c, const hspec_mamba_w& w, const void* h_last, const StatePlan& p,
                       float* S0_f32, hipStream_t st) {
  hspec::GemmArgs g1;
  set_a(g1, in_place(h_last, c.dtype), c.d_h);
  set_w(g1, w.W_r, c.dtype, c.d_h);
  g1.M = c.B; g1.N = c.r; g1.K = c.d_h;
  g1.C_hi = p.F_hi; g1.C_lo = p.F_lo; g1.ldch = c.r;
  g1.C_h16 = p.F_h16; g1.C_l16 = p.F_l16; g1.h16_scale = 1.f / (1 << kFScaleLog2);
  use_scratch(g1, p.gs);
  HIP_TRY(hspec::launch_gemm(g1, st));
  const int dS = c.H * c.P * c.N;
  hspec::GemmArgs g2;
  g2.A_hi = p.F_hi; g2.A_lo = p.F_lo; g2.lda = c.r;
  if (p.F_h16) {   // fp16 product with the packed W_dS (x 2^kPackScaleLog2), F x 2^-kFScaleLog2
    g2.A_hi = reinterpret_cast<const bf16*>(p.F_h16);
    g2.A_lo = reinterpret_cast<const bf16*>(p.F_l16);
    g2.f16 = 1;
    g2.out_scale = (float)(1 << kFScaleLog2) / (float)(1 << hspec::kPackScaleLog2);
  }
  set_w(g2, w.W_dS, c.dtype, c.r);
  g2.M = c.B; g2.N = dS; g2.K = c.r;
  g2.C = S0_f32; g2.ldc = dS;
  g2.C_hi = p.S0_hi; g2.C_lo = p.S0_lo; g2.C_h16 = p.S0_h16; g2.ldch = dS;
  g2.w_packed = (c.flags & HSPEC_W_DS_PACKED) ? 1 : 0;
  use_scratch(g2, p.gs);
  HIP_TRY(hspec::launch_gemm(g2, st));
  return HSPEC_OK;
}

struct MambaPlan {
  StatePlan st;
  bf16 *u_hi = nullptr, *u_lo = nullptr;      // normalised block input (draft step)
  float* zx = nullptr;
  bf16 *x_hi = nullptr, *x_lo = nullptr, *B_hi = nullptr, *B_lo = nullptr, *C_hi = nullptr, *C_lo = nullptr;
  float* dt = nullptr;
  float* y = nullptr;
  bf16 *yn_hi = nullptr, *yn_lo = nullptr;
  GemmScratch gs;
};

// Whether the Mamba projections take their activations as hi/lo planes (fp32 storage, or
// HSPEC_MAMBA_PRECISE_IO) or as one bf16 plane.
bool mamba_io_lo(const hspec_mamba_cfg& c) { return is_f32(c.dtype) || (c.flags & HSPEC_MAMBA_PRECISE_IO); }

void plan_mamba(Arena& ar, const hspec_mamba_cfg& c, bool u_norm, MambaPlan& p) {
  plan_state(ar, c, true, p.st);
  const size_t M = (size_t)c.B * c.k;
  const size_t di = (size_t)c.H * c.P, gn = (size_t)c.G * c.N;
  const size_t dproj = 2 * di + 2 * gn + c.H;
  const bool io_lo = mamba_io_lo(c);
  if (u_norm) {
    p.u_hi = ar.take<bf16>(M * c.d_model);
    if (io_lo) p.u_lo = ar.take<bf16>(M * c.d_model);
  }
  p.zx = ar.take<float>(M * dproj);
  p.x_hi = ar.take<bf16>(M * di);
  p.x_lo = ar.take<bf16>(M * di);   // x feeds the state update: kept as hi/lo planes
  p.B_hi = ar.take<bf16>(M * gn);
  p.B_lo = ar.take<bf16>(M * gn);
  p.C_hi = ar.take<bf16>(M * gn);
  p.C_lo = ar.take<bf16>(M * gn);
  p.dt = ar.take<float>(M * c.H);
  p.y = ar.take<float>(M * di);
  p.yn_hi = ar.take<bf16>(M * di);
  if (io_lo) p.yn_lo = ar.take<bf16>(M * di);
  p.gs = reserve_gemm(ar, c.dtype, {{(int)M, (int)dproj, c.d_model}, {(int)M, c.d_model, (int)di}});
}

// in_proj -> conv/split -> scan from S0 planes -> gated norm -> out_proj (+ residual R).
// With `sum`, out_proj's product may be left as partial sums for the next kernel, which then adds R
// (the residual) and writes out: see GemmArgs::defer.  `clear`: status words to clear, or null.
hspec_status run_mamba_core(const hspec_mamba_cfg& c, const hspec_mamba_w& w, Planes u, const MambaPlan& p,
                            const void* R, int r_bf16, float* out, float* S_final, int* clear, hspec::Parts* sum,
                            hipStream_t st) {
  const int M = c.B * c.k;
  const int di = c.H * c.P, gn = c.G * c.N;
  const int dproj = 2 * di + 2 * gn + c.H;
  hspec::GemmArgs gi;
  set_a(gi, u, c.d_model);
  set_w(gi, w.W_in, c.dtype, c.d_model);
  gi.M = M; gi.N = dproj; gi.K = c.d_model;
  gi.C = p.zx; gi.ldc = dproj;
  hspec::Parts zx(p.zx);
  gi.defer = &zx;
  use_scratch(gi, p.gs);
  HIP_TRY(hspec::launch_gemm(gi, st));

  hspec::ConvArgs ca;
  ca.clear = clear;
  ca.zxbcdt = zx; ca.conv_w = w.conv_w; ca.conv_b = w.conv_b; ca.w_bf16 = !is_f32(c.dtype);
  ca.dt_bias = w.dt_bias;
  ca.B = c.B; ca.T = c.k; ca.H = c.H; ca.P = c.P; ca.G = c.G; ca.N = c.N; ca.K = c.conv_w;
  ca.x_hi = p.x_hi; ca.x_lo = p.x_lo; ca.B_hi = p.B_hi; ca.B_lo = p.B_lo; ca.C_hi = p.C_hi; ca.C_lo = p.C_lo;
  ca.dt = p.dt;
  HIP_TRY(hspec::launch_conv_split(ca, st));

  hspec::ScanArgs sa;
  sa.x_hi = p.x_hi; sa.x_lo = p.x_lo; sa.dt = p.dt; sa.A = w.A_log; sa.A_is_log = 1;
  sa.B_hi = p.B_hi; sa.B_lo = p.B_lo; sa.C_hi = p.C_hi; sa.C_lo = p.C_lo; sa.Dskip = w.D;
  sa.S0_hi = p.st.S0_hi; sa.S0_lo = p.st.S0_lo; sa.S0_h16 = p.st.S0_h16; sa.y = p.y; sa.S_final = S_final;
  sa.B = c.B; sa.T = c.k; sa.H = c.H; sa.P = c.P; sa.N = c.N; sa.G = c.G; sa.chunk = c.chunk;
  sa.x_ld = di; sa.bc_ld = gn; sa.dt_ld = c.H;
  HIP_TRY(hspec::launch_ssd_scan(sa, st));

  HIP_TRY(hspec::launch_gated_rmsnorm(p.y, zx, dproj, w.gnorm_w, M, di, c.G, c.eps, p.yn_hi, p.yn_lo, st));

  hspec::GemmArgs go;
  go.A_hi = p.yn_hi; go.A_lo = p.yn_lo; go.lda = di;
  set_w(go, w.W_out, c.dtype, di);
  go.M = M; go.N = c.d_model; go.K = di;
  go.C = out; go.ldc = c.d_model;
  go.R = R; go.ldr = c.d_model; go.r_bf16 = r_bf16;
  go.defer = sum;
  use_scratch(go, p.gs);   // (in_proj's partial sums were last read by the gated norm)
  HIP_TRY(hspec::launch_gemm(go, st));
  return HSPEC_OK;
}

struct AttnPlan {
  SplitSlot kc, vc, qin, kbin, vbin;
  bf16 *xn_hi = nullptr, *xn_lo = nullptr;   // normalised input (draft step)
  float* qkv = nullptr;
  bf16 *q_hi = nullptr, *q_lo = nullptr, *k_hi = nullptr, *k_lo = nullptr, *v_hi = nullptr, *v_lo = nullptr;
  float* part_o = nullptr;
  float* part_ml = nullptr;
  int32_t* units = nullptr;
  int32_t* req = nullptr;
  bf16 *o_hi = nullptr, *o_lo = nullptr;
  int split = 0, max_splits = 0, auto_split = 0, min_split = 0;
  GemmScratch gs;
};

void plan_sweep(Arena& ar, const hspec_attn_cfg& c, int max_ctx_len, AttnPlan& p) {
  const int swept = hspec::attention_swept_len(max_ctx_len, c.window);
  p.split = c.split_tokens > 0 ? c.split_tokens : hspec::attention_default_split(c.B, c.Hkv, swept);
  // automatic splitting: the work-list kernel may cut requests finer than p.split (down to
  // attention_min_auto_split), so the buffers are sized for that many splits
  p.auto_split = c.split_tokens > 0 ? 0 : 1;
  p.min_split = p.auto_split ? hspec::attention_min_auto_split(p.split, swept) : p.split;
  // (a validated call has at most 256 splits; a query for any other config stays defined)
  const long long ns = swept > 0 ? ceil_div(swept, p.min_split) : 1;
  p.max_splits = (int)std::min<long long>(ns, INT_MAX);
  const int R = c.k * (c.Hq / c.Hkv);
  const size_t units = (size_t)c.B * c.Hkv * p.max_splits;
  p.units = ar.take<int32_t>((size_t)4 * c.B * p.max_splits);
  p.req = ar.take<int32_t>((size_t)2 * c.B);
  if (p.max_splits > 1 || (c.flags & HSPEC_ATTN_PRECISE_IO)) {   // split partials
    p.part_o = ar.take<float>(units * R * c.D);
    p.part_ml = ar.take<float>(units * R * 2);
  }
  const size_t cache = (size_t)c.num_pages * c.page_size * cache_heads(c) * c.D;
  p.kc = reserve_split(ar, c.dtype, cache);
  p.vc = reserve_split(ar, c.dtype, cache);
}

void plan_attn(Arena& ar, const hspec_attn_cfg& c, int max_ctx_len, bool x_norm, AttnPlan& p) {
  const size_t M = (size_t)c.B * c.k;
  const bool f32 = is_f32(c.dtype);
  const bool io_lo = f32 || (c.flags & HSPEC_ATTN_PRECISE_IO);   // hi/lo planes into W_q/k/v and W_o
  if (x_norm) {
    p.xn_hi = ar.take<bf16>(M * c.d_model);
    if (io_lo) p.xn_lo = ar.take<bf16>(M * c.d_model);
  }
  p.qkv = ar.take<float>(M * (c.Hq + 2 * c.Hkv) * c.D);
  // q, k and v: hi/lo planes for fp32 storage (the sweep's hi/lo products) and for precise
  // attention I/O (the reduction rebuilds the block keys in fp32 from both planes)
  p.q_hi = ar.take<bf16>(M * c.Hq * c.D);
  p.k_hi = ar.take<bf16>(M * c.Hkv * c.D);
  p.v_hi = ar.take<bf16>(M * c.Hkv * c.D);
  if (io_lo) {
    p.q_lo = ar.take<bf16>(M * c.Hq * c.D);
    p.k_lo = ar.take<bf16>(M * c.Hkv * c.D);
    p.v_lo = ar.take<bf16>(M * c.Hkv * c.D);
  }
  plan_sweep(ar, c, max_ctx_len, p);
  p.o_hi = ar.take<bf16>(M * c.Hq * c.D);
  if (io_lo) p.o_lo = ar.take<bf16>(M * c.Hq * c.D);
  // the fused QKV product (one launch over the three weight segments) and the separate ones
  p.gs = reserve_gemm(ar, c.dtype, {{(int)M, (c.Hq + 2 * c.Hkv) * c.D, c.d_model}, {(int)M, c.Hq * c.D, c.d_model},
                                    {(int)M, c.Hkv * c.D, c.d_model}, {(int)M, c.d_model, c.Hq * c.D}});
}

hspec::AttnArgs sweep_args(const hspec_attn_cfg& c, const AttnPlan& p, const int32_t* pt, const int32_t* lens,
                           int max_ctx_len, int* status) {
  hspec::AttnArgs a;
  a.page_table = pt; a.ctx_lens = lens;
  a.B = c.B; a.T = c.k; a.Hq = c.Hq; a.Hkv = c.Hkv; a.D = c.D; a.ps = c.page_size;
  a.Hkv_cache = cache_heads(c);
  a.kv_remap = c.kv_heads ? 1 : 0;   // (at most 16 cache heads then: checked)
  a.kv_map = 0;
  for (int h = 0; c.kv_heads && h < c.Hkv && h < 16; ++h) a.kv_map |= (unsigned long long)(c.kv_heads[h] & 15) << (4 * h);
  a.max_pages = c.max_pages; a.num_pages = c.num_pages; a.window = c.window;
  a.causal = (c.flags & HSPEC_BLOCK_CAUSAL) ? 1 : 0;
  a.block_in_sweep = (c.flags & HSPEC_ATTN_PRECISE_IO) ? 0 : 1;
  a.max_ctx_len = max_ctx_len; a.split = p.split; a.max_splits = p.max_splits;
  const float scale = c.scale > 0.f ? c.scale : 1.f / std::sqrt((float)c.D);
  a.scale_log2 = scale * 1.4426950408889634f;
  a.part_o = p.part_o; a.part_ml = p.part_ml; a.status = status; a.units = p.units; a.req = p.req;
  a.auto_split = p.auto_split; a.min_split = p.min_split;
  a.grid = a.auto_split ? hspec::attention_sweep_grid(c.D, c.k * (c.Hq / c.Hkv), is_f32(c.dtype)) : 0;
  return a;
}

// QKV projections -> q/k norm + RoPE -> sweep + reduce -> O projection (+ residual R).  The
// sweep's work list is built inside the q/k-norm + RoPE launch (its own launch, ahead of the
// projections, past kWorklistFusedMax requests), clearing the first plan_clear status words.
hspec_status run_attn_core(const hspec_attn_cfg& c, const hspec_attn_w& w, Planes xn, const void* k_cache,
                           const void* v_cache, const int32_t* pt, const int32_t* lens, int max_ctx_len,
                           const AttnPlan& p, const void* R, int r_bf16, float* out, int* status, int plan_clear,
                           hspec::Parts* sum, hipStream_t st) {
  const int M = c.B * c.k;
  const hspec::AttnArgs plan = sweep_args(c, p, pt, lens, max_ctx_len, status);
  const bool plan_fused = c.B <= hspec::kWorklistFusedMax;
  if (!plan_fused) HIP_TRY(hspec::launch_attention_plan(plan, plan_clear, st));
  const int ldq = (c.Hq + 2 * c.Hkv) * c.D;
  Splits split;
  const Planes kc = split.add(k_cache, c.dtype, p.kc), vc = split.add(v_cache, c.dtype, p.vc);
  HIP_TRY(split.launch(st));
  hspec::Parts qkv(p.qkv);
  hspec::GemmArgs gq;   // one product over the three row segments [W_q; W_k; W_v]
  set_a(gq, xn, c.d_model);
  set_w(gq, w.W_q, c.dtype, c.d_model);
  gq.W2 = rows_of(w.W_k); gq.W3 = rows_of(w.W_v); gq.N1 = c.Hq * c.D; gq.N2 = c.Hkv * c.D;
  gq.M = M; gq.N = ldq; gq.K = c.d_model;
  gq.C = p.qkv; gq.ldc = ldq;
  gq.defer = &qkv;
  use_scratch(gq, p.gs);
  HIP_TRY(hspec::launch_gemm(gq, st));
  HIP_TRY(hspec::launch_qk_norm_rope(qkv, w.q_norm_w, w.k_norm_w, lens, c.B, c.k, c.Hq, c.Hkv, c.D, c.eps,
                                     c.rope_theta, p.q_hi, p.q_lo, p.k_hi, p.k_lo, p.v_hi, p.v_lo, st,
                                     plan_fused ? &plan : nullptr, plan_clear));
  hspec::AttnArgs a = plan;
  a.q_hi = p.q_hi; a.q_lo = p.q_lo; a.kb_hi = p.k_hi; a.kb_lo = p.k_lo; a.vb_hi = p.v_hi; a.vb_lo = p.v_lo;
  a.kc_hi = kc.hi; a.kc_lo = kc.lo; a.vc_hi = vc.hi; a.vc_lo = vc.lo;
  a.o_bf16 = p.o_hi;
  a.o_bf16_lo = p.o_lo;
  HIP_TRY(hspec::launch_attention(a, st));
  hspec::GemmArgs g;
  g.A_hi = p.o_hi; g.A_lo = p.o_lo; g.lda = c.Hq * c.D;
  set_w(g, w.W_o, c.dtype, c.Hq * c.D);
  g.M = M; g.N = c.d_model; g.K = c.Hq * c.D;
  g.C = out; g.ldc = c.d_model;
  g.R = R; g.ldr = c.d_model; g.r_bf16 = r_bf16;
  g.defer = sum;
  use_scratch(g, p.gs);
  HIP_TRY(hspec::launch_gemm(g, st));
  return HSPEC_OK;
}

// RMSNorm of a sublayer's output: out itself, or the sum of the partial products it was left as
// (GemmArgs::defer) and the residual R, which also writes out.
hipError_t norm_output(const hspec::Parts& sum, const void* R, int r_bf16, float* out, const float* w, int rows, int n,
                       float eps, bf16* hi, bf16* lo, hipStream_t st) {
  if (sum.p == out) return hspec::launch_rmsnorm_planes(out, 0, w, rows, n, eps, hi, lo, st);
  return hspec::launch_sum_rmsnorm_planes(sum, R, r_bf16, out, w, rows, n, eps, hi, lo, st);
}

struct DraftPlan {
  MambaPlan m;
  float* x1 = nullptr;
  AttnPlan at;
};

void plan_draft(Arena& ar, const hspec_mamba_cfg& mc, const hspec_attn_cfg& ac, int max_ctx_len, DraftPlan& p) {
  plan_mamba(ar, mc, true, p.m);
  p.x1 = ar.take<float>((size_t)mc.B * mc.k * mc.d_model);
  plan_attn(ar, ac, max_ctx_len, true, p.at);
}

int* status_word(Arena& ar) { return ar.take<int>(ALIGN / sizeof(int)); }

}  // namespace

// ============================================================================ C ABI

HSPEC_API size_t hspec_state_init_workspace(const hspec_mamba_cfg* cfg) {
  if (!cfg) return 0;
  Arena ar;
  status_word(ar);
  StatePlan p;
  plan_state(ar, *cfg, false, p);
  return ar.size();
}

HSPEC_API hspec_status hspec_state_init(const hspec_mamba_cfg* cfg, const hspec_mamba_w* w, const void* h_last,
                                        float* S0, void* workspace, size_t ws_bytes, void* stream) {
  clear_err();
  if (hspec_status s = check_mamba(cfg, w, false)) return s;
  if (!h_last || !S0) return fail(HSPEC_ERR_NULL, "h_last or S0 is NULL");
  if (hspec_status s = check_ws(workspace, ws_bytes, hspec_state_init_workspace(cfg))) return s;
  hipStream_t st = (hipStream_t)stream;
  Arena ar{(char*)workspace};
  int* status = status_word(ar);
  StatePlan p;
  plan_state(ar, *cfg, false, p);
  HIP_TRY(hspec::launch_zero_words(status, hspec::kStatusClear, st));
  return run_state(*cfg, *w, h_last, p, S0, st);
}

HSPEC_API size_t hspec_mamba_block_scan_workspace(const hspec_mamba_cfg* cfg) {
  if (!cfg) return 0;
  Arena ar;
  status_word(ar);
  MambaPlan p;
  plan_mamba(ar, *cfg, false, p);
  return ar.size();
}

HSPEC_API hspec_status hspec_mamba_block_scan(const hspec_mamba_cfg* cfg, const hspec_mamba_w* w,
                                              const void* h_last, const void* block_hidden, float* out,
                                              float* S_final, void* workspace, size_t ws_bytes, void* stream) {
  clear_err();
  if (hspec_status s = check_mamba(cfg, w, true)) return s;
  if (!h_last || !block_hidden || !out) return fail(HSPEC_ERR_NULL, "h_last, block_hidden or out is NULL");
  if (hspec_status s = check_ws(workspace, ws_bytes, hspec_mamba_block_scan_workspace(cfg))) return s;
  hipStream_t st = (hipStream_t)stream;
  Arena ar{(char*)workspace};
  int* status = status_word(ar);
  MambaPlan p;
  plan_mamba(ar, *cfg, false, p);
  if (hspec_status s = run_state(*cfg, *w, h_last, p.st, nullptr, st)) return s;
  return run_mamba_core(*cfg, *w, in_place(block_hidden, cfg->dtype), p, nullptr, 0, out, S_final, status, nullptr, st);   // (no kernel sets a bit)
}

HSPEC_API size_t hspec_target_kv_block_attn_workspace(const hspec_attn_cfg* cfg, int max_ctx_len) {
  if (!cfg) return 0;
  Arena ar;
  status_word(ar);
  AttnPlan p;
  plan_attn(ar, *cfg, max_ctx_len < 0 ? 0 : max_ctx_len, false, p);
  return ar.size();
}

HSPEC_API hspec_status hspec_target_kv_block_attn(const hspec_attn_cfg* cfg, const hspec_attn_w* w, const void* x,
                                                  const void* k_cache, const void* v_cache,
                                                  const int32_t* page_table, const int32_t* ctx_lens,
                                                  int max_ctx_len, float* out, void* workspace, size_t ws_bytes,
                                                  void* stream) {
  clear_err();
  if (hspec_status s = check_attn_cfg(cfg, max_ctx_len)) return s;
  if (hspec_status s = check_attn_w(cfg, w)) return s;
  if (!x || !k_cache || !v_cache || !page_table || !ctx_lens || !out)
    return fail(HSPEC_ERR_NULL, "an input or output pointer is NULL");
  if (hspec_status s = check_ws(workspace, ws_bytes, hspec_target_kv_block_attn_workspace(cfg, max_ctx_len)))
    return s;
  hipStream_t st = (hipStream_t)stream;
  Arena ar{(char*)workspace};
  int* status = status_word(ar);
  AttnPlan p;
  plan_attn(ar, *cfg, max_ctx_len, false, p);
  // no kernel before the work list sets a status bit: the work list clears the status words
  return run_attn_core(*cfg, *w, in_place(x, cfg->dtype), k_cache, v_cache, page_table, ctx_lens, max_ctx_len, p, nullptr, 0, out, status,
                       hspec::kStatusClear, nullptr, st);
}

HSPEC_API size_t hspec_draft_step_workspace(const hspec_mamba_cfg* mcfg, const hspec_attn_cfg* acfg,
                                            int max_ctx_len) {
  if (!mcfg || !acfg) return 0;
  Arena ar;
  status_word(ar);
  DraftPlan p;
  plan_draft(ar, *mcfg, *acfg, max_ctx_len < 0 ? 0 : max_ctx_len, p);
  return ar.size();
}

HSPEC_API hspec_status hspec_draft_step(const hspec_mamba_cfg* mcfg, const hspec_mamba_w* mw, const float* norm1_w,
                                        const hspec_attn_cfg* acfg, const hspec_attn_w* aw, const float* norm2_w,
                                        const void* h_last, const void* block_emb, const void* k_cache,
                                        const void* v_cache, const int32_t* page_table, const int32_t* ctx_lens,
                                        int max_ctx_len, float* out, void* workspace, size_t ws_bytes, void* stream) {
  clear_err();
  if (hspec_status s = check_mamba(mcfg, mw, true)) return s;
  if (hspec_status s = check_attn_cfg(acfg, max_ctx_len)) return s;
  if (hspec_status s = check_attn_w(acfg, aw)) return s;
  if (mcfg->B != acfg->B || mcfg->k != acfg->k || mcfg->d_model != acfg->d_model)
    return fail(HSPEC_ERR_SHAPE, "mamba and attention configs disagree on B, k or d_model");
  if (mcfg->dtype != acfg->dtype) return fail(HSPEC_ERR_DTYPE, "mamba and attention dtypes differ");
  if (!norm1_w || !norm2_w || !h_last || !block_emb || !k_cache || !v_cache || !page_table || !ctx_lens || !out)
    return fail(HSPEC_ERR_NULL, "an input or output pointer is NULL");
  if (hspec_status s = check_ws(workspace, ws_bytes, hspec_draft_step_workspace(mcfg, acfg, max_ctx_len))) return s;
  hipStream_t st = (hipStream_t)stream;
  Arena ar{(char*)workspace};
  int* status = status_word(ar);
  DraftPlan p;
  plan_draft(ar, *mcfg, *acfg, max_ctx_len, p);
  const int M = mcfg->B * mcfg->k;
  const bool f32 = is_f32(mcfg->dtype);
  // no kernel before the attention's work list sets a status bit: the work list clears them
  if (hspec_status s = run_state(*mcfg, *mw, h_last, p.m.st, nullptr, st)) return s;
  HIP_TRY(hspec::launch_rmsnorm_planes(block_emb, !f32, norm1_w, M, mcfg->d_model, mcfg->eps, p.m.u_hi, p.m.u_lo, st));
  Planes u{p.m.u_hi, p.m.u_lo};
  hspec::Parts x1(p.x1);
  if (hspec_status s = run_mamba_core(*mcfg, *mw, u, p.m, block_emb, !f32, p.x1, nullptr, nullptr, &x1, st)) return s;
  HIP_TRY(norm_output(x1, block_emb, !f32, p.x1, norm2_w, M, acfg->d_model, acfg->eps, p.at.xn_hi, p.at.xn_lo, st));
  Planes xn{p.at.xn_hi, p.at.xn_lo};
  return run_attn_core(*acfg, *aw, xn, k_cache, v_cache, page_table, ctx_lens, max_ctx_len, p.at, p.x1, 0, out, status,
                       hspec::kStatusClear, nullptr, st);
}

HSPEC_API size_t hspec_ssd_scan_workspace(int B, int T, int H, int P, int N, int G, hspec_dtype dtype) {
  Arena ar;
  status_word(ar);
  if (dtype == HSPEC_F32 && B > 0 && T > 0) {
    reserve_split(ar, dtype, (size_t)B * T * H * P);
    reserve_split(ar, dtype, (size_t)B * T * G * N);
    reserve_split(ar, dtype, (size_t)B * T * G * N);
    reserve_split(ar, dtype, (size_t)B * H * P * N);
  }
  return ar.size();
}

HSPEC_API hspec_status hspec_ssd_scan(int B, int T, int H, int P, int N, int G, int chunk, hspec_dtype dtype,
                                      const void* x, const float* dt, const float* A, const void* Bm, const void* Cm,
                                      const float* Dskip, const void* S0, float* y, float* S_final, void* workspace,
                                      size_t ws_bytes, void* stream) {
  clear_err();
  if (!dtype_ok(dtype)) return fail(HSPEC_ERR_DTYPE, "unknown dtype %d", (int)dtype);
  if (B <= 0 || T <= 0 || H <= 0 || P <= 0 || N <= 0 || G <= 0 || chunk <= 0)
    return fail(HSPEC_ERR_SHAPE, "non-positive scan dimension");
  if (H % G) return fail(HSPEC_ERR_SHAPE, "H %% G != 0");
  if (P != 64) return fail(HSPEC_ERR_UNSUPPORTED, "P must be 64, got %d", P);
  if (N != 16 && N != 32 && N != 64 && N != 128) return fail(HSPEC_ERR_UNSUPPORTED, "N must be 16/32/64/128");
  if (chunk > 16) return fail(HSPEC_ERR_UNSUPPORTED, "chunk must be <= 16");
  if (!x || !dt || !A || !Bm || !Cm || !Dskip || !y) return fail(HSPEC_ERR_NULL, "a scan pointer is NULL");
  if (hspec_status s = check_ws(workspace, ws_bytes, hspec_ssd_scan_workspace(B, T, H, P, N, G, dtype))) return s;
  hipStream_t st = (hipStream_t)stream;
  Arena ar{(char*)workspace};
  int* status = status_word(ar);
  SplitSlot sx, sb, sc, ss;
  if (dtype == HSPEC_F32) {
    sx = reserve_split(ar, dtype, (size_t)B * T * H * P);
    sb = reserve_split(ar, dtype, (size_t)B * T * G * N);
    sc = reserve_split(ar, dtype, (size_t)B * T * G * N);
    ss = reserve_split(ar, dtype, (size_t)B * H * P * N);
  }
  Splits split;
  const Planes px = split.add(x, dtype, sx), pb = split.add(Bm, dtype, sb), pc = split.add(Cm, dtype, sc);
  const Planes ps = S0 ? split.add(S0, dtype, ss) : Planes{};
  HIP_TRY(split.launch(st));
  hspec::ScanArgs a;
  a.x_hi = px.hi; a.x_lo = px.lo; a.dt = dt; a.A = A; a.A_is_log = 0;
  a.B_hi = pb.hi; a.B_lo = pb.lo; a.C_hi = pc.hi; a.C_lo = pc.lo; a.Dskip = Dskip;
  a.S0_hi = ps.hi; a.S0_lo = ps.lo;
  a.y = y; a.S_final = S_final;
  a.B = B; a.T = T; a.H = H; a.P = P; a.N = N; a.G = G; a.chunk = chunk;
  a.x_ld = H * P; a.bc_ld = G * N; a.dt_ld = H;
  a.clear = status;
  HIP_TRY(hspec::launch_ssd_scan(a, st));
  return HSPEC_OK;
}

HSPEC_API size_t hspec_paged_attn_workspace(const hspec_attn_cfg* cfg, int max_ctx_len) {
  if (!cfg) return 0;
  Arena ar;
  status_word(ar);
  AttnPlan p;
  const size_t M = (size_t)cfg->B * cfg->k;
  p.qin = reserve_split(ar, cfg->dtype, M * cfg->Hq * cfg->D);
  p.kbin = reserve_split(ar, cfg->dtype, M * cfg->Hkv * cfg->D);
  p.vbin = reserve_split(ar, cfg->dtype, M * cfg->Hkv * cfg->D);
  plan_sweep(ar, *cfg, max_ctx_len < 0 ? 0 : max_ctx_len, p);
  return ar.size();
}

HSPEC_API hspec_status hspec_paged_attn_phase(const hspec_attn_cfg* cfg, const void* q, const void* k_blk,
                                              const void* v_blk, const void* k_cache, const void* v_cache,
                                              const int32_t* page_table, const int32_t* ctx_lens, int max_ctx_len,
                                              float* o, void* workspace, size_t ws_bytes, unsigned phases,
                                              void* stream) {
  clear_err();
  if (hspec_status s = check_attn_cfg(cfg, max_ctx_len)) return s;
  if (!q || !k_blk || !v_blk || !k_cache || !v_cache || !page_table || !ctx_lens || !o)
    return fail(HSPEC_ERR_NULL, "an input or output pointer is NULL");
  if (phases & ~(unsigned)(HSPEC_PHASE_WORKLIST | HSPEC_PHASE_SWEEP | HSPEC_PHASE_REDUCE))
    return fail(HSPEC_ERR_UNSUPPORTED, "unknown phase bits 0x%x", phases);
  if (hspec_status s = check_ws(workspace, ws_bytes, hspec_paged_attn_workspace(cfg, max_ctx_len))) return s;
  hipStream_t st = (hipStream_t)stream;
  Arena ar{(char*)workspace};
  int* status = status_word(ar);
  AttnPlan p;
  const size_t M = (size_t)cfg->B * cfg->k;
  p.qin = reserve_split(ar, cfg->dtype, M * cfg->Hq * cfg->D);
  p.kbin = reserve_split(ar, cfg->dtype, M * cfg->Hkv * cfg->D);
  p.vbin = reserve_split(ar, cfg->dtype, M * cfg->Hkv * cfg->D);
  plan_sweep(ar, *cfg, max_ctx_len, p);
  // the sweep's work list is the call's first kernel and clears the status words
  if (phases & HSPEC_PHASE_WORKLIST)
    HIP_TRY(hspec::launch_attention_plan(sweep_args(*cfg, p, page_table, ctx_lens, max_ctx_len, status),
                                         hspec::kStatusClear, st));
  if (!(phases & (HSPEC_PHASE_SWEEP | HSPEC_PHASE_REDUCE))) return HSPEC_OK;
  Planes pq, pk, pv, kc, vc;
  if (phases & HSPEC_PHASE_SWEEP) {
    Splits split;
    pq = split.add(q, cfg->dtype, p.qin);
    pk = split.add(k_blk, cfg->dtype, p.kbin);
    pv = split.add(v_blk, cfg->dtype, p.vbin);
    kc = split.add(k_cache, cfg->dtype, p.kc);
    vc = split.add(v_cache, cfg->dtype, p.vc);
    HIP_TRY(split.launch(st));
  } else {
    // the reduction alone still reads the block q, k and v: the caller's bf16 tensors, or the
    // planes the sweep phase of this attention wrote into the workspace (fp32 storage)
    pq = planes_in_place(q, cfg->dtype, p.qin);
    pk = planes_in_place(k_blk, cfg->dtype, p.kbin);
    pv = planes_in_place(v_blk, cfg->dtype, p.vbin);
  }
  hspec::AttnArgs a = sweep_args(*cfg, p, page_table, ctx_lens, max_ctx_len, status);
  a.q_hi = pq.hi; a.q_lo = pq.lo; a.kb_hi = pk.hi; a.kb_lo = pk.lo; a.vb_hi = pv.hi; a.vb_lo = pv.lo;
  a.kc_hi = kc.hi; a.kc_lo = kc.lo; a.vc_hi = vc.hi; a.vc_lo = vc.lo;
  a.o_f32 = o;
  const unsigned parts = ((phases & HSPEC_PHASE_SWEEP) ? hspec::ATTN_SWEEP : 0u) |
                         ((phases & HSPEC_PHASE_REDUCE) ? hspec::ATTN_REDUCE : 0u);
  HIP_TRY(hspec::launch_attention(a, st, parts));
  return HSPEC_OK;
}

HSPEC_API hspec_status hspec_paged_attn(const hspec_attn_cfg* cfg, const void* q, const void* k_blk,
                                        const void* v_blk, const void* k_cache, const void* v_cache,
                                        const int32_t* page_table, const int32_t* ctx_lens, int max_ctx_len, float* o,
                                        void* workspace, size_t ws_bytes, void* stream) {
  return hspec_paged_attn_phase(cfg, q, k_blk, v_blk, k_cache, v_cache, page_table, ctx_lens, max_ctx_len, o,
                                workspace, ws_bytes, HSPEC_PHASE_WORKLIST | HSPEC_PHASE_SWEEP | HSPEC_PHASE_REDUCE,
                                stream);
}

HSPEC_API hspec_status hspec_gather_slots(int B, int max_pages, int page_size, int num_pages,
                                          const int32_t* page_table, const int32_t* ctx_lens, int max_ctx_len,
                                          int32_t* slots, int32_t* status, void* stream) {
  clear_err();
  if (B <= 0 || max_pages <= 0 || page_size <= 0 || num_pages <= 0 || max_ctx_len < 0)
    return fail(HSPEC_ERR_SHAPE, "non-positive gather dimension");
  if (!page_table || !ctx_lens || (!slots && max_ctx_len > 0)) return fail(HSPEC_ERR_NULL, "a gather pointer is NULL");
  if (page_size < 16 || (page_size & (page_size - 1)))
    return fail(HSPEC_ERR_UNSUPPORTED, "page_size must be a power of two >= 16, got %d", page_size);
  HIP_TRY(hspec::launch_gather_slots(B, max_pages, page_size, num_pages, page_table, ctx_lens, max_ctx_len, slots,
                                     status, (hipStream_t)stream));
  return HSPEC_OK;
}

// fp32 storage: room for both operands, for calls whose C lies over one of them (see operand_for).
struct LinearPlan {
  int* status = nullptr;
  float *A = nullptr, *W = nullptr;
  GemmScratch gs;
};
void plan_linear(Arena& ar, hspec_dtype dtype, int M, int N, int K, LinearPlan& p) {
  p.status = status_word(ar);
  if (M <= 0 || N <= 0 || K <= 0) return;
  if (is_f32(dtype)) {
    p.A = ar.take<float>((size_t)M * K);
    p.W = ar.take<float>((size_t)N * K);
  }
  p.gs = reserve_gemm(ar, dtype, {{M, N, K}});
}

// The product reads fp32 operands in place while it writes C: an operand that shares memory with C
// is read from a copy in the workspace (K == N and C in place of A, say).
hipError_t operand_for(const void* x, size_t n, hspec_dtype dtype, const float* C, size_t c_n, float* copy,
                       const void*& out, hipStream_t st) {
  out = x;
  if (!is_f32(dtype)) return hipSuccess;
  const uintptr_t x0 = (uintptr_t)x, c0 = (uintptr_t)C;
  if (x0 >= c0 + 4 * c_n || c0 >= x0 + 4 * n) return hipSuccess;
  out = copy;
  return hspec::launch_copy_f32(static_cast<const float*>(x), n, copy, st);
}

HSPEC_API size_t hspec_linear_workspace(hspec_dtype dtype, int M, int N, int K) {
  Arena ar;
  LinearPlan p;
  plan_linear(ar, dtype, M, N, K, p);
  return ar.size();
}

HSPEC_API hspec_status hspec_linear(hspec_dtype dtype, int M, int N, int K, const void* A, const void* W,
                                    const float* R, float* C, void* workspace, size_t ws_bytes, void* stream) {
  clear_err();
  if (!dtype_ok(dtype)) return fail(HSPEC_ERR_DTYPE, "unknown dtype %d", (int)dtype);
  if (M <= 0 || N <= 0 || K <= 0) return fail(HSPEC_ERR_SHAPE, "non-positive GEMM dimension");
  if (K % 8) return fail(HSPEC_ERR_UNSUPPORTED, "K must be a multiple of 8");
  if (!A || !W || !C) return fail(HSPEC_ERR_NULL, "A, W or C is NULL");
  if (hspec_status s = check_ws(workspace, ws_bytes, hspec_linear_workspace(dtype, M, N, K))) return s;
  hipStream_t st = (hipStream_t)stream;
  Arena ar{(char*)workspace};
  LinearPlan p;
  plan_linear(ar, dtype, M, N, K, p);
  HIP_TRY(hspec::launch_zero_words(p.status, hspec::kStatusClear, st));
  HIP_TRY(operand_for(A, (size_t)M * K, dtype, C, (size_t)M * N, p.A, A, st));
  HIP_TRY(operand_for(W, (size_t)N * K, dtype, C, (size_t)M * N, p.W, W, st));
  hspec::GemmArgs g;
  set_a(g, in_place(A, dtype), K);
  set_w(g, W, dtype, K);
  g.M = M; g.N = N; g.K = K;
  g.C = C; g.ldc = N; g.R = R; g.ldr = N; g.r_bf16 = 0;
  use_scratch(g, p.gs);
  HIP_TRY(hspec::launch_gemm(g, st));
  return HSPEC_OK;
}

// ---------------------------------------------------------------- whole drafter forward

struct ForwardPlan {
  MambaPlan m;                              // with the state plan; its u planes also feed the MLP
  AttnPlan at;
  float *xa = nullptr, *xb = nullptr;       // residual stream, alternating
  float* gu = nullptr;                      // [M, 2 ff]: gate | up
  bf16 *h_hi = nullptr, *h_lo = nullptr;    // [M, ff]
  GemmScratch gs;
};

void plan_forward(Arena& ar, const hspec_mamba_cfg& mc, const hspec_attn_cfg& ac, int ff, int max_ctx_len,
                  ForwardPlan& p) {
  plan_mamba(ar, mc, true, p.m);
  plan_attn(ar, ac, max_ctx_len, true, p.at);
  const size_t M = (size_t)mc.B * mc.k;
  p.xa = ar.take<float>(M * mc.d_model);
  p.xb = ar.take<float>(M * mc.d_model);
  p.gu = ar.take<float>(M * 2 * ff);
  p.h_hi = ar.take<bf16>(M * ff);
  p.h_lo = ar.take<bf16>(M * ff);
  p.gs = reserve_gemm(ar, mc.dtype, {{(int)M, 2 * ff, mc.d_model}, {(int)M, ff, mc.d_model}, {(int)M, mc.d_model, ff}});
}

// x_out = x + W_down (SiLU(W_gate u) * (W_up u)), u already normalised (planes).
hspec_status run_mlp(const hspec_mamba_cfg& c, const hspec_layer_w& L, int ff, Planes u, const ForwardPlan& p,
                     const void* x, int x_bf16, float* x_out, hspec::Parts* sum, hipStream_t st) {
  const int M = c.B * c.k;
  hspec::Parts gu(p.gu);
  hspec::GemmArgs gg;   // one product over the two row segments [W_gate; W_up]
  set_a(gg, u, c.d_model);
  set_w(gg, L.W_gate, c.dtype, c.d_model);
  gg.W2 = rows_of(L.W_up); gg.N1 = ff; gg.N2 = ff;
  gg.M = M; gg.N = 2 * ff; gg.K = c.d_model;
  gg.C = p.gu; gg.ldc = 2 * ff;
  gg.defer = &gu;
  use_scratch(gg, p.gs);
  HIP_TRY(hspec::launch_gemm(gg, st));
  HIP_TRY(hspec::launch_silu_mul(gu, M, ff, p.h_hi, p.h_lo, st));
  hspec::GemmArgs g;
  g.A_hi = p.h_hi; g.A_lo = p.h_lo; g.lda = ff;
  set_w(g, L.W_down, c.dtype, ff);
  g.M = M; g.N = c.d_model; g.K = ff;
  g.C = x_out; g.ldc = c.d_model;
  g.R = x; g.ldr = c.d_model; g.r_bf16 = x_bf16;
  g.defer = sum;
  use_scratch(g, p.gs);
  HIP_TRY(hspec::launch_gemm(g, st));
  return HSPEC_OK;
}

HSPEC_API size_t hspec_drafter_forward_workspace(const hspec_mamba_cfg* mcfg, const hspec_attn_cfg* acfg, int ff,
                                                 int max_ctx_len) {
  if (!mcfg || !acfg || ff <= 0) return 0;
  hspec_mamba_cfg mc = *mcfg;
  mc.flags |= HSPEC_MAMBA_PRECISE_IO;
  hspec_attn_cfg ac = *acfg;
  ac.flags |= HSPEC_ATTN_PRECISE_IO;
  Arena ar;
  status_word(ar);
  ForwardPlan p;
  plan_forward(ar, mc, ac, ff, max_ctx_len < 0 ? 0 : max_ctx_len, p);
  return ar.size();
}

HSPEC_API hspec_status hspec_drafter_forward(const hspec_mamba_cfg* mcfg, const hspec_attn_cfg* acfg, int ff,
                                             int n_layers, const void* W_r, const void* W_dS,
                                             const hspec_layer_w* layers, const void* h_last, const void* block_emb,
                                             const int32_t* page_table, const int32_t* ctx_lens, int max_ctx_len,
                                             float* out, void* workspace, size_t ws_bytes, void* stream) {
  clear_err();
  if (!mcfg || !acfg) return fail(HSPEC_ERR_NULL, "mamba or attention config is NULL");
  if (n_layers < 1) return fail(HSPEC_ERR_SHAPE, "n_layers must be >= 1");
  if (!layers) return fail(HSPEC_ERR_NULL, "layers is NULL");
  if (ff <= 0) return fail(HSPEC_ERR_SHAPE, "ff must be positive");
  if (ff % 8) return fail(HSPEC_ERR_UNSUPPORTED, "ff must be a multiple of 8");
  bool any_attn = false, any_mamba = false;
  for (int l = 0; l < n_layers; ++l) {
    const hspec_layer_w& L = layers[l];
    if (L.mamba) {
      any_mamba = true;
      hspec_mamba_w mw = *L.mamba;
      mw.W_r = W_r;
      mw.W_dS = W_dS;
      if (hspec_status s = check_mamba(mcfg, &mw, true)) return s;
      if (!L.norm1_w) return fail(HSPEC_ERR_NULL, "layer %d: norm1_w is NULL", l);
    }
    if (!L.norm3_w || !L.W_gate || !L.W_up || !L.W_down)
      return fail(HSPEC_ERR_NULL, "layer %d: a norm or MLP weight is NULL", l);
    if (L.attn) {
      any_attn = true;
      if (hspec_status s = check_attn_w(acfg, L.attn)) return s;
      if (!L.norm2_w || !L.k_cache || !L.v_cache) return fail(HSPEC_ERR_NULL, "layer %d: attention input is NULL", l);
    }
  }
  if (hspec_status s = check_attn_cfg(acfg, max_ctx_len)) return s;
  if (mcfg->B != acfg->B || mcfg->k != acfg->k || mcfg->d_model != acfg->d_model)
    return fail(HSPEC_ERR_SHAPE, "mamba and attention configs disagree on B, k or d_model");
  if (mcfg->dtype != acfg->dtype) return fail(HSPEC_ERR_DTYPE, "mamba and attention dtypes differ");
  if (!any_mamba && (mcfg->B <= 0 || mcfg->k <= 0 || mcfg->d_model <= 0 || mcfg->d_model % 8 || !dtype_ok(mcfg->dtype)))
    return fail(HSPEC_ERR_SHAPE, "bad B, k, d_model or dtype");
  if (!block_emb || !out || (any_mamba && !h_last) || (any_attn && (!page_table || !ctx_lens)))
    return fail(HSPEC_ERR_NULL, "an input or output pointer is NULL");
  if (hspec_status s = check_ws(workspace, ws_bytes, hspec_drafter_forward_workspace(mcfg, acfg, ff, max_ctx_len)))
    return s;
  hipStream_t st = (hipStream_t)stream;
  // the layers' errors add up over the stack: activations enter every projection as hi/lo planes
  hspec_mamba_cfg mc = *mcfg;
  mc.flags |= HSPEC_MAMBA_PRECISE_IO;
  hspec_attn_cfg ac = *acfg;
  ac.flags |= HSPEC_ATTN_PRECISE_IO;
  Arena ar{(char*)workspace};
  int* status = status_word(ar);
  ForwardPlan p;
  plan_forward(ar, mc, ac, ff, max_ctx_len, p);
  const int M = mc.B * mc.k;
  const bool f32 = is_f32(mc.dtype);
  // the status words: cleared by the first attention's work list (no kernel before it sets a bit),
  // or here when there is no attention
  int plan_clear = hspec::kStatusClear;
  if (!any_attn) HIP_TRY(hspec::launch_zero_words(status, hspec::kStatusClear, st));
  if (any_mamba) {
    hspec_mamba_w sw{};
    sw.W_r = W_r;
    sw.W_dS = W_dS;
    if (hspec_status s = run_state(mc, sw, h_last, p.m.st, nullptr, st)) return s;
  }

  // the residual stream: block_emb (storage dtype), then fp32 buffers; the last sublayer
  // writes straight into out.  Between sublayers it may be (x_sum, x_res): a product's partial
  // sums and the residual to add, which the next norm adds up into x.
  int total = 0;
  for (int l = 0; l < n_layers; ++l) total += 1 + (layers[l].mamba ? 1 : 0) + (layers[l].attn ? 1 : 0);
  int done = 0;
  const void* x = block_emb;
  int x_bf16 = !f32;
  hspec::Parts x_sum;
  const void* x_res = nullptr;
  int res_bf16 = 0;
  float* x_f32 = nullptr;   // x as the fp32 buffer it is (or will be) in, null for block_emb
  // norm of the residual stream, then x becomes the residual of the sublayer that writes y
  auto norm = [&](const float* w, int n, float eps, bf16* hi, bf16* lo) -> hipError_t {
    if (!x_f32) return hspec::launch_rmsnorm_planes(x, x_bf16, w, M, n, eps, hi, lo, st);
    return norm_output(x_sum, x_res, res_bf16, x_f32, w, M, n, eps, hi, lo, st);
  };
  auto next = [&]() -> float* { return ++done == total ? out : (x_f32 == p.xa ? p.xb : p.xa); };
  auto advance = [&](float* y) {
    x_res = x;
    res_bf16 = x_bf16;
    x = x_f32 = y;
    x_bf16 = 0;
  };
  Planes u{p.m.u_hi, p.m.u_lo};
  for (int l = 0; l < n_layers; ++l) {
    const hspec_layer_w& L = layers[l];
    if (L.mamba) {
      HIP_TRY(norm(L.norm1_w, mc.d_model, mc.eps, p.m.u_hi, p.m.u_lo));
      float* y = next();
      x_sum = hspec::Parts(y);
      if (hspec_status s = run_mamba_core(mc, *L.mamba, u, p.m, x, x_bf16, y, nullptr, nullptr, &x_sum, st)) return s;
      advance(y);
    }
    if (L.attn) {
      HIP_TRY(norm(L.norm2_w, ac.d_model, ac.eps, p.at.xn_hi, p.at.xn_lo));
      Planes xn{p.at.xn_hi, p.at.xn_lo};
      float* y = next();
      x_sum = hspec::Parts(y);
      if (hspec_status s = run_attn_core(ac, *L.attn, xn, L.k_cache, L.v_cache, page_table, ctx_lens, max_ctx_len,
                                         p.at, x, x_bf16, y, status, plan_clear, &x_sum, st))   // work list, fresh queue
        return s;
      plan_clear = 0;
      advance(y);
    }
    HIP_TRY(norm(L.norm3_w, mc.d_model, mc.eps, p.m.u_hi, p.m.u_lo));
    float* y = next();
    x_sum = hspec::Parts(y);
    if (hspec_status s = run_mlp(mc, L, ff, u, p, x, x_bf16, y, done == total ? nullptr : &x_sum, st)) return s;
    advance(y);
  }
  return HSPEC_OK;
}

// ------------------------------------------------ drafter-side KV injection (comparison)

// Layers are taken in groups: one product over the K and V weights of a group, one append launch.
constexpr int kInjectGroup = hspec::AppendArgs::kMaxLayers;

struct InjectPlan {
  int* status = nullptr;
  bf16 *f_hi = nullptr, *f_lo = nullptr;     // fused [M, d_model]
  float* kv = nullptr;                       // [M, layers of a group, 2 Hkv D]: k | v of each layer
  GemmScratch gs;
};

void plan_inject(Arena& ar, const hspec_attn_cfg& c, int d_h, InjectPlan& p) {
  p.status = status_word(ar);
  const size_t M = (size_t)c.B * c.k, kvw = (size_t)c.Hkv * c.D;
  p.f_hi = ar.take<bf16>(M * c.d_model);
  p.f_lo = ar.take<bf16>(M * c.d_model);
  p.kv = ar.take<float>(M * 2 * kvw * kInjectGroup);
  // the fusion, and a group of any size (the last may be short)
  p.gs.cap = hspec::gemm_scratch_elems((int)M, c.d_model, d_h, true, is_f32(c.dtype));
  for (int n = 1; n <= 2 * kInjectGroup; ++n)
    p.gs.cap = std::max(p.gs.cap, hspec::gemm_scratch_elems((int)M, n * (int)kvw, c.d_model, true, is_f32(c.dtype)));
  if (p.gs.cap) p.gs.p = ar.take<float>(p.gs.cap);
}

// Whether no two of the layers' caches share memory.
bool caches_apart(const hspec_attn_cfg& c, int n, void* const* k, void* const* v) {
  const uintptr_t bytes = (uintptr_t)c.num_pages * c.page_size * c.Hkv * c.D * (is_f32(c.dtype) ? 4 : 2);
  for (int i = 0; i < 2 * n; ++i)
    for (int j = 0; j < i; ++j) {
      const uintptr_t x = (uintptr_t)(i % 2 ? v : k)[i / 2], y = (uintptr_t)(j % 2 ? v : k)[j / 2];
      if (x < y + bytes && y < x + bytes) return false;
    }
  return true;
}

HSPEC_API size_t hspec_kv_inject_workspace(const hspec_attn_cfg* cfg, int d_h) {
  if (!cfg || d_h <= 0 || cfg->B <= 0 || cfg->k <= 0) return 0;
  Arena ar;
  InjectPlan p;
  plan_inject(ar, *cfg, d_h, p);
  return ar.size();
}

HSPEC_API hspec_status hspec_kv_inject(const hspec_attn_cfg* cfg, int d_h, int n_layers, const void* h_new,
                                       const void* W_fc, const void* const* W_k, const void* const* W_v,
                                       const float* const* k_norm_w, void* const* k_cache, void* const* v_cache,
                                       const int32_t* page_table, const int32_t* ctx_lens, void* workspace,
                                       size_t ws_bytes, void* stream) {
  clear_err();
  if (hspec_status s = check_attn_cfg(cfg, 0)) return s;
  if (cfg->kv_heads || (cfg->Hkv_cache != 0 && cfg->Hkv_cache != cfg->Hkv))
    return fail(HSPEC_ERR_UNSUPPORTED, "KV injection writes the drafter's own caches: no KV-head subset");
  if (d_h <= 0 || n_layers < 1) return fail(HSPEC_ERR_SHAPE, "d_h and n_layers must be positive");
  if (d_h % 8) return fail(HSPEC_ERR_UNSUPPORTED, "d_h must be a multiple of 8");
  if (cfg->d_model <= 0 || cfg->d_model % 8) return fail(HSPEC_ERR_UNSUPPORTED, "d_model must be a positive multiple of 8");
  if (!h_new || !W_fc || !W_k || !W_v || !k_norm_w || !k_cache || !v_cache || !page_table || !ctx_lens)
    return fail(HSPEC_ERR_NULL, "an input or output pointer is NULL");
  for (int l = 0; l < n_layers; ++l)
    if (!W_k[l] || !W_v[l] || !k_norm_w[l] || !k_cache[l] || !v_cache[l])
      return fail(HSPEC_ERR_NULL, "layer %d: a weight or cache pointer is NULL", l);
  if (hspec_status s = check_ws(workspace, ws_bytes, hspec_kv_inject_workspace(cfg, d_h))) return s;
  hipStream_t st = (hipStream_t)stream;
  const hspec_attn_cfg& c = *cfg;
  Arena ar{(char*)workspace};
  InjectPlan p;
  plan_inject(ar, c, d_h, p);
  HIP_TRY(hspec::launch_zero_words(p.status, hspec::kStatusClear, st));
  const int M = c.B * c.k, kvw = c.Hkv * c.D;
  hspec::GemmArgs g;
  set_a(g, in_place(h_new, c.dtype), d_h);
  set_w(g, W_fc, c.dtype, d_h);
  g.M = M; g.N = c.d_model; g.K = d_h;
  g.C_hi = p.f_hi; g.C_lo = p.f_lo; g.ldch = c.d_model;
  use_scratch(g, p.gs);
  HIP_TRY(hspec::launch_gemm(g, st));
  for (int l0 = 0; l0 < n_layers; l0 += kInjectGroup) {
    const int nl = std::min(kInjectGroup, n_layers - l0), ld = nl * 2 * kvw;
    hspec::AppendArgs a;
    a.kv = hspec::Parts(p.kv);
    // one product over the row segments [W_k; W_v] of the group's layers
    hspec::GemmArgs gk;
    gk.A_hi = p.f_hi; gk.A_lo = p.f_lo; gk.lda = c.d_model;
    set_w(gk, nullptr, c.dtype, c.d_model);
    gk.nseg = 2 * nl; gk.seg_rows = kvw;
    for (int i = 0; i < 2 * nl; ++i) gk.seg[i] = rows_of(i % 2 ? W_v[l0 + i / 2] : W_k[l0 + i / 2]);
    gk.M = M; gk.N = ld; gk.K = c.d_model;
    gk.C = p.kv; gk.ldc = ld;
    gk.defer = &a.kv;
    use_scratch(gk, p.gs);
    HIP_TRY(hspec::launch_gemm(gk, st));
    a.n_layers = nl;
    for (int i = 0; i < nl; ++i) {
      a.kw[i] = k_norm_w[l0 + i];
      a.k_cache[i] = k_cache[l0 + i];
      a.v_cache[i] = v_cache[l0 + i];
    }
    a.cache_bf16 = !is_f32(c.dtype);
    a.B = c.B; a.n = c.k; a.Hkv = c.Hkv; a.D = c.D; a.eps = c.eps; a.rope_theta = c.rope_theta;
    a.page_table = page_table; a.max_pages = c.max_pages; a.num_pages = c.num_pages; a.ps = c.page_size;
    a.ctx_lens = ctx_lens; a.status = p.status;
    // the group's caches at once, or one after the other (k, then v of each layer) where two share memory
    const bool apart = caches_apart(c, nl, k_cache + l0, v_cache + l0);
    const int heads = nl * 2 * c.Hkv, step = apart ? heads : c.Hkv;
    for (a.head0 = 0; a.head0 < heads; a.head0 += step) {
      a.head1 = a.head0 + step;
      HIP_TRY(hspec::launch_kv_append(a, st));
    }
  }
  return HSPEC_OK;
}

// ------------------------------------------------------------------------- draft head

hspec_status check_head(const hspec_head_cfg* c) {
  if (!c) return fail(HSPEC_ERR_NULL, "head config is NULL");
  if (c->B <= 0 || c->k <= 0 || c->d_model <= 0 || c->vocab <= 0 || c->rank <= 0)
    return fail(HSPEC_ERR_SHAPE, "non-positive head dimension");
  if (c->d_model % 8) return fail(HSPEC_ERR_UNSUPPORTED, "d_model must be a multiple of 8");
  if (c->rank % 32) return fail(HSPEC_ERR_UNSUPPORTED, "the Markov rank must be a multiple of 32");
  if ((long long)c->B * c->k > (1LL << 30) || (long long)c->vocab * c->rank > (1LL << 40))
    return fail(HSPEC_ERR_UNSUPPORTED, "head too large");
  return HSPEC_OK;
}

struct HeadPlan {
  int* status = nullptr;
  bf16* hn = nullptr;
  float* base = nullptr;
  unsigned long long* keys = nullptr;
  GemmScratch gs;
};

void plan_head(Arena& ar, const hspec_head_cfg& c, HeadPlan& p) {
  p.status = status_word(ar);
  const size_t M = (size_t)c.B * c.k;
  p.hn = ar.take<bf16>(M * c.d_model);
  p.base = ar.take<float>(M * c.vocab);
  p.keys = ar.take<unsigned long long>(M * hspec::kHeadSlots);
  p.gs = reserve_gemm(ar, HSPEC_BF16, {{(int)M, c.vocab, c.d_model}});
}

HSPEC_API size_t hspec_draft_head_workspace(const hspec_head_cfg* cfg) {
  if (!cfg || cfg->B <= 0 || cfg->k <= 0 || cfg->d_model <= 0 || cfg->vocab <= 0) return 0;
  Arena ar;
  HeadPlan p;
  plan_head(ar, *cfg, p);
  return ar.size();
}

HSPEC_API hspec_status hspec_draft_head(const hspec_head_cfg* cfg, const hspec_head_w* w, const float* hidden,
                                        const int32_t* prev_tok, const float* gumbel, const int32_t* forced,
                                        int32_t* tokens, float* logits, void* workspace, size_t ws_bytes,
                                        void* stream) {
  clear_err();
  if (hspec_status s = check_head(cfg)) return s;
  if (!w || !w->norm_f_w || !w->W_lm || !w->E_M || !w->U_M) return fail(HSPEC_ERR_NULL, "head weight is NULL");
  if (!hidden || !prev_tok || !tokens) return fail(HSPEC_ERR_NULL, "hidden, prev_tok or tokens is NULL");
  if (gumbel && !(cfg->temperature > 0.f)) return fail(HSPEC_ERR_SHAPE, "sampling needs temperature > 0");
  if (hspec_status s = check_ws(workspace, ws_bytes, hspec_draft_head_workspace(cfg))) return s;
  hipStream_t st = (hipStream_t)stream;
  const hspec_head_cfg& c = *cfg;
  Arena ar{(char*)workspace};
  HeadPlan p;
  plan_head(ar, c, p);
  hspec::HeadArgs h;
  h.B = c.B; h.k = c.k; h.V = c.vocab; h.R = c.rank;
  h.keys = p.keys; h.status = p.status;
  const int M = c.B * c.k;
  HIP_TRY(hspec::launch_head_norm(h, hspec::kStatusClear, hidden, w->norm_f_w, c.d_model, c.eps, p.hn, st));
  // LM head over the pruned vocabulary; written straight into the caller's logits when given
  float* base = logits ? logits : p.base;
  hspec::GemmArgs g;
  g.A_hi = p.hn; g.lda = c.d_model;
  g.W = static_cast<const bf16*>(w->W_lm); g.ldw = c.d_model;
  g.M = M; g.N = c.vocab; g.K = c.d_model;
  g.C = base; g.ldc = c.vocab;
  use_scratch(g, p.gs);
  HIP_TRY(hspec::launch_gemm(g, st));
  h.E = static_cast<const bf16*>(w->E_M); h.U = static_cast<const bf16*>(w->U_M);
  h.base = base; h.logits = logits; h.gumbel = gumbel;
  h.inv_temp = gumbel ? 1.f / c.temperature : 1.f;
  h.prev = prev_tok; h.forced = forced; h.tokens = tokens;
  HIP_TRY(hspec::launch_markov_head(h, st));
  return HSPEC_OK;
}

HSPEC_API size_t hspec_pack_w_ds_bytes(int d_S, int r) {
  if (d_S <= 0 || r <= 0 || d_S % 16 || r % 64) return 0;
  return (size_t)d_S * r * sizeof(bf16);
}

HSPEC_API hspec_status hspec_pack_w_ds(int d_S, int r, const void* W_dS, void* W_packed, void* stream) {
  clear_err();
  if (d_S <= 0 || r <= 0) return fail(HSPEC_ERR_SHAPE, "non-positive W_dS dimension");
  if (d_S % 16 || r % 64) return fail(HSPEC_ERR_UNSUPPORTED, "packing needs d_S %% 16 == 0 and r %% 64 == 0");
  if (!W_dS || !W_packed) return fail(HSPEC_ERR_NULL, "W_dS or W_packed is NULL");
  HIP_TRY(hspec::launch_pack_w(static_cast<const bf16*>(W_dS), d_S, r, static_cast<_Float16*>(W_packed),
                               (hipStream_t)stream));
  return HSPEC_OK;
}

HSPEC_API hspec_status hspec_read_status(const void* workspace, int32_t* status, void* stream) {
  clear_err();
  if (!workspace || !status) return fail(HSPEC_ERR_NULL, "workspace or status is NULL");
  hipStream_t st = (hipStream_t)stream;
  HIP_TRY(hipMemcpyAsync(status, workspace, sizeof(int32_t), hipMemcpyDeviceToHost, st));
  HIP_TRY(hipStreamSynchronize(st));
  return HSPEC_OK;
}

HSPEC_API const char* hspec_status_string(hspec_status s) {
  switch (s) {
    case HSPEC_OK: return "ok";
    case HSPEC_ERR_NULL: return "null pointer";
    case HSPEC_ERR_SHAPE: return "bad shape";
    case HSPEC_ERR_DTYPE: return "bad dtype";
    case HSPEC_ERR_UNSUPPORTED: return "unsupported dimension";
    case HSPEC_ERR_WORKSPACE: return "workspace too small or misaligned";
    case HSPEC_ERR_LAUNCH: return "kernel launch failed";
  }
  return "unknown status";
}

HSPEC_API const char* hspec_last_error(void) { return g_err; }

namespace hspec {
hspec_status api_fail(hspec_status s, const char* msg) { return fail(s, "%s", msg); }
}  // namespace hspec
