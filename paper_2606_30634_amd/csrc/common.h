// Internal helpers shared by the gfx950 kernels and the host code of the stage library.
#pragma once
#include <hip/hip_runtime.h>
#include <cstdint>
#include <cstddef>

typedef __bf16 bf16;
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

#define WAVE 64

// fp32 <-> storage conversions; the bf16 cast is round-to-nearest-even on gfx950.
__device__ __forceinline__ float to_f32(float v) { return v; }
__device__ __forceinline__ float to_f32(bf16 v) { return (float)v; }
template <typename T> __device__ __forceinline__ T from_f32(float v);
template <> __device__ __forceinline__ float from_f32<float>(float v) { return v; }
template <> __device__ __forceinline__ bf16 from_f32<bf16>(float v) { return (bf16)v; }

__device__ __forceinline__ float wave_sum(float v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, WAVE);
  return v;
}
__device__ __forceinline__ double wave_sum(double v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, WAVE);
  return v;
}
__device__ __forceinline__ float wave_max(float v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v = fmaxf(v, __shfl_xor(v, o, WAVE));
  return v;
}

// Block-wide sum for blockDim.x a multiple of 64 (<= 1024); result valid in every thread.
template <typename T>
__device__ __forceinline__ T block_sum(T v, T* smem /* >= 16 entries */) {
  v = wave_sum(v);
  const int w = threadIdx.x / WAVE, l = threadIdx.x % WAVE, nw = blockDim.x / WAVE;
  __syncthreads();
  if (l == 0) smem[w] = v;
  __syncthreads();
  T r = 0;
  for (int i = 0; i < nw; ++i) r += smem[i];  // fixed order: deterministic
  return r;
}

static inline int64_t cdiv(int64_t a, int64_t b) { return (a + b - 1) / b; }

// what ds_read_b64_tr_b16 returns: 4 elements of a column of 4 consecutive rows
typedef short v4i16_t __attribute__((ext_vector_type(4)));

// Compile-time loop: f(std::integral_constant<int, 0>) ... f(<N-1>).  Keeps register-array indices
// constant even where a loop body holds a barrier (which can stop the unroller).
#include <utility>
template <typename F, int... Is>
__device__ __forceinline__ void static_for_impl(F&& f, std::integer_sequence<int, Is...>) {
  (f(std::integral_constant<int, Is>{}), ...);
}
template <int N, typename F>
__device__ __forceinline__ void static_for(F&& f) {
  static_for_impl(f, std::make_integer_sequence<int, N>{});
}

// ------------------------------------------------------------------ direct-to-LDS loads (gfx950)
// s_waitcnt: at most N vector-memory operations and no LDS operation outstanding
template <int N>
__device__ __forceinline__ void wait_vm_lds() {
  static_assert(N >= 0 && N < 64, "vmcnt range");
  __builtin_amdgcn_s_waitcnt((N & 15) | ((N >> 4) << 14) | (7 << 4) | (0 << 8));
}

// One 16-byte global -> LDS load per lane from base + voff bytes (base wave-uniform; lane l
// writes lds + 16 l).  Issued as inline assembly so that the compiler neither counts it in its own
// waits nor orders LDS reads after it: a kernel waits for these loads itself (wait_vm_lds)
// before the barrier that publishes the LDS they fill.
__device__ __forceinline__ void dma16(const void* base, uint32_t voff, uint32_t lds) {
  asm volatile("global_load_lds_dwordx4 %0, %1" ::"v"(voff), "s"(base), "{m0}"(lds) : "memory");
}
// The same with 4 bytes per lane (lane l writes lds + 4 l).
__device__ __forceinline__ void dma4(const void* base, uint32_t voff, uint32_t lds) {
  asm volatile("global_load_lds_dword %0, %1" ::"v"(voff), "s"(base), "{m0}"(lds) : "memory");
}

// The same 16-byte load with a range: a raw buffer descriptor over [base, end) (base wave-uniform;
// end - base clamped to 2 GB), and lanes whose 16 bytes start past the range write zeros.  BUFFER_OUT
// is an offset that no range holds.
constexpr uint32_t BUFFER_OUT = 0x80000000u;
__device__ __forceinline__ u32x4 buffer_range(const void* base, const void* end) {
  const uint64_t a = (uint64_t)(uintptr_t)base;
  const int64_t n = (const char*)end - (const char*)base;
  const uint32_t bytes = n <= 0 ? 0u : n > 0x7fffffffll ? 0x7ffffff0u : (uint32_t)n;
  return u32x4{(uint32_t)a, (uint32_t)(a >> 32) & 0xffffu, bytes, 0x00020000u};
}
__device__ __forceinline__ void dma16_range(u32x4 range, uint32_t voff, uint32_t lds) {
  asm volatile("buffer_load_dwordx4 %0, %1, 0 offen lds" ::"v"(voff), "s"(range), "{m0}"(lds) : "memory");
}
__device__ __forceinline__ void dma4_range(u32x4 range, uint32_t voff, uint32_t lds) {
  asm volatile("buffer_load_dword %0, %1, 0 offen lds" ::"v"(voff), "s"(range), "{m0}"(lds) : "memory");
}

__device__ __forceinline__ void block_barrier() {
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
}

// LDS byte address of a pointer into __shared__ memory (the m0 operand of dma16 / dma4)
template <typename T>
__device__ __forceinline__ uint32_t lds_addr(const T* p) {
  typedef __attribute__((address_space(3))) const T lds_t;
  return (uint32_t)(uintptr_t)(lds_t*)p;
}
