// Device-side building blocks shared by the gfx950 kernels of the drafting step:
// bf16 helpers, MFMA fragment types and wrappers, wave-level reductions.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

namespace hspec {

typedef __bf16 bf16;
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef _Float16 f16x4 __attribute__((ext_vector_type(4)));

constexpr int WAVE = 64;

// Device status word bits (first int32 of every workspace).
enum : int {
  ST_BAD_PAGE = 1,      // a page id outside [0, num_pages)
  ST_BAD_CTX_LEN = 2,   // ctx_len < 0 or beyond the table / max_ctx_len
};

__device__ __forceinline__ float bf2f(bf16 v) { return (float)v; }
__device__ __forceinline__ bf16 f2bf(float v) { return (bf16)v; }   // v_cvt_pk_bf16_f32, RNE

// Widening of storage element types to fp32 for VALU code.
__device__ __forceinline__ float to_f32(float v) { return v; }
__device__ __forceinline__ float to_f32(bf16 v) { return (float)v; }

// 16-byte fragment of 8 bf16 values.
__device__ __forceinline__ bf16x8 ld8(const bf16* p) {
  return *reinterpret_cast<const bf16x8*>(p);
}
__device__ __forceinline__ bf16x8 zero8() {
  u32x4 z = {0u, 0u, 0u, 0u};
  return __builtin_bit_cast(bf16x8, z);
}

// D += A(16x32) * B(32x16); lane l holds A[l%16][8(l/16)..+7], B[8(l/16)..+7][l%16],
// D[4(l/16)+i][l%16].
__device__ __forceinline__ f32x4 mma16(bf16x8 a, bf16x8 b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}
// The same 16x16x32 product on fp16 operands (11 significant bits).
__device__ __forceinline__ f32x4 mma16h(f16x8 a, f16x8 b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_f16(a, b, c, 0, 0, 0);
}
// D += A(32x16) * B(16x32); lane l holds A[l%32][8(l/32)..+7], B[8(l/32)..+7][l%32],
// D[8(i/4)+4(l/32)+i%4][l%32].
__device__ __forceinline__ f32x16 mma32(bf16x8 a, bf16x8 b, f32x16 c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
}

// Reductions over the four lanes l, l^16, l^32, l^48 (one column of a 16-wide MFMA tile),
// with the gfx950 lane-swap instructions: every lane ends with the same, identically ordered
// result.
__device__ __forceinline__ float wave_max16x4(float v) {
  auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  v = fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
  auto q = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return fmaxf(__uint_as_float(q[0]), __uint_as_float(q[1]));
}
__device__ __forceinline__ float wave_sum16x4(float v) {
  auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  v = __uint_as_float(r[0]) + __uint_as_float(r[1]);
  auto q = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return __uint_as_float(q[0]) + __uint_as_float(q[1]);
}
__device__ __forceinline__ float wave_sum(float v) {
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
  return v;
}

// Wait until at most VM vector-memory operations (loads, LDS DMA) of this wave are pending.
template <int VM>
__device__ __forceinline__ void wait_vmcnt() {
  static_assert(VM >= 0 && VM < 64, "vmcnt range");
  // gfx9 s_waitcnt immediate: vmcnt[3:0] and [15:14], expcnt[6:4] = 7, lgkmcnt[11:8] = 15 (no wait)
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_waitcnt((VM & 15) | (7 << 4) | (15 << 8) | ((VM >> 4) << 14));
  asm volatile("" ::: "memory");
}

template <int VM>
__device__ __forceinline__ void wait_vm_lgkm0() {
  // vmcnt <= VM and every LDS access of this wave complete
  static_assert(VM >= 0 && VM < 64, "vmcnt range");
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_waitcnt((VM & 15) | (7 << 4) | (0 << 8) | ((VM >> 4) << 14));
  asm volatile("" ::: "memory");
}

// Workgroup barrier without the memory fence of __syncthreads (which would also wait for
// every outstanding global load); callers order LDS traffic with explicit waits.
__device__ __forceinline__ void wg_barrier() {
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
}

// NV pieces of 4 elements (16-byte aligned, from element i[e]) of a matrix given as np planes,
// added in plane order.  Every load of UP planes is issued before the first is added.  UP = 0: one plane
// (np = 1), without the registers of the others.
template <int NV, int UP = 2>
__device__ __forceinline__ void ld4_parts(const float* p, int np, size_t plane, const size_t (&i)[NV], f32x4 (&v)[NV]) {
#pragma unroll
  for (int e = 0; e < NV; ++e) v[e] = *reinterpret_cast<const f32x4*>(p + i[e]);
  if constexpr (UP > 0) {
    for (int k = 1; k < np; k += UP) {
      f32x4 t[UP][NV];
#pragma unroll
      for (int u = 0; u < UP; ++u) {
        const float* q = p + (size_t)min(k + u, np - 1) * plane;
#pragma unroll
        for (int e = 0; e < NV; ++e) t[u][e] = *reinterpret_cast<const f32x4*>(q + i[e]);
      }
#pragma unroll
      for (int u = 0; u < UP; ++u)
        if (k + u < np) {
#pragma unroll
          for (int e = 0; e < NV; ++e) v[e] += t[u][e];
        }
    }
  }
}
__device__ __forceinline__ float ld1_parts(const float* p, int np, size_t plane, size_t i) {
  float v = p[i];
  for (int k = 1; k < np; ++k) v += p[(size_t)k * plane + i];
  return v;
}

// Buffer resource of `bytes` bytes from base (wave-uniform); accesses past the end read zero and
// write nothing.  BUF_OOB: an offset past every range.
constexpr int BUF_OOB = 0x7fffff00;
__device__ __forceinline__ __amdgpu_buffer_rsrc_t rsrc(const void* base, int bytes) {
  return __builtin_amdgcn_make_buffer_rsrc((void*)base, 0, __builtin_amdgcn_readfirstlane(bytes), 0x00020000);
}

// Reads one word of every 64-byte line of a kernel's first `BYTES` argument bytes, so that arguments first used late
// in the kernel are scalar cache hits by then: the compiler loads them where they are used, and each such
// line is a trip to memory on a launch's critical path.  For kernels with a late argument on that path:
// streamed product of 16 x 4096 x 4096 10.9 -> 10.1 us, of 128 rows 24.0 -> 22.8, RoPE launch with the
// work list of 31 requests 8.7 -> 6.3.  Not for the others, which would wait for lines they need later
// anyway (scan of 6 us + 1.4, no change in the norms).
template <int BYTES>
__device__ __forceinline__ void touch_args() {
  const __attribute__((address_space(4))) int* k =
      (const __attribute__((address_space(4))) int*)__builtin_amdgcn_kernarg_segment_ptr();
  int v[BYTES / 64 + 1];
#pragma unroll
  for (int i = 0; i < BYTES / 64; ++i) v[i] = k[16 * i];
  v[BYTES / 64] = k[BYTES / 4 - 1];
#pragma unroll
  for (int i = 0; i <= BYTES / 64; ++i) asm volatile("" ::"s"(v[i]));
}

template <int V>
using Int = std::integral_constant<int, V>;

__device__ __forceinline__ void set_status(int* st, int bit) {
  if (st) atomicOr(st, bit);
}

}  // namespace hspec
