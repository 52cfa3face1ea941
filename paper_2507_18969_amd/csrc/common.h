// Shared definitions of the EDPC HIP library (gfx950 only).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace edpc {

typedef uint16_t bf16_t;  // storage type of BF16 values (bit pattern)

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));

__device__ __forceinline__ float bf2f(bf16_t h) { return __uint_as_float(((uint32_t)h) << 16); }

// Round-to-nearest-even FP32 -> BF16 (the gfx950 conversion instruction;
// NaN stays NaN).
__device__ __forceinline__ bf16_t f2bf(float f) { return __builtin_bit_cast(bf16_t, (__bf16)f); }

// Per-step scalars, written on the device by the step-advance kernel so that
// the same launch sequence (or a captured graph of it) serves every step.
struct StepState {
  int32_t step;      // position i in the streams
  int32_t rows;      // active rows (streams) this step
  float inv_rows;    // 1 / rows (the mean of Eq. 2)
  float bc1, bc2;    // Adam bias corrections 1 - beta^tau
  uint32_t tau;      // Adam step number (1 for the first update)
  int32_t model;     // 1 if the model runs this step (step >= context)
  int32_t base;      // step before a captured window; its steps count from it
};

// Adam constants (Kingma & Ba 2015; lr from the configuration).
struct AdamCfg {
  float lr, beta1, beta2, eps;
};

// Adam's bias correction 1 - beta^tau, formed as -expm1(tau log1p(beta - 1))
// so that it keeps full FP32 relative accuracy at small tau (1 - powf loses
// log2(1 / (1 - beta^tau)) bits to cancellation, about 8 bits at beta 0.999
// and tau 3).  beta - 1 is exact in FP32 for beta in [0.5, 1]; beta = 0
// gives 1.  tau = 0 (no update yet) gives 0.
__device__ __forceinline__ float adam_bias_correction(float beta, uint32_t tau) {
  if (tau == 0) return 0.0f;
  if (beta <= 0.0f) return 1.0f;
  return -expm1f((float)tau * log1pf(beta - 1.0f));
}

__device__ __forceinline__ float gelu_f(float x) {
  return 0.5f * x * (1.0f + erff(x * 0.70710678118654752f));
}
// (The rounding of the sum is written out: kernels with the same sums share it.)
__device__ __forceinline__ float gelu_grad_f(float x) {
#pragma clang fp contract(off)
  const float cdf = 0.5f * (1.0f + erff(x * 0.70710678118654752f));
  const float pdf = expf(-0.5f * x * x) * 0.39894228040143268f;
  return fmaf(x, pdf, cdf);
}

// Fixed-order wave reductions: a butterfly over the 64 lanes at distances 32, 16,
// .. 1, all lanes active.  By lane swaps and DPP: a step is one or two instructions
// where a shuffle is a round trip through LDS (the BF16 row-block kernel, 1024 rows:
// 113.8 us with shuffles, 107.4 so).
// Distances 8 and 4 are rotations in a row of 16, whose values repeat by then.
template <int CTRL, class T>
__device__ __forceinline__ T dpp(T v) {
  return __builtin_bit_cast(
      T, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), CTRL, 0xF, 0xF, true));
}
template <class T, class Op>
__device__ __forceinline__ T wave_reduce(T v, Op op) {
  static_assert(sizeof(T) == 4, "one register");
  typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
  const uint32_t x = __builtin_bit_cast(uint32_t, v);
  const u32x2 h = __builtin_bit_cast(u32x2, __builtin_amdgcn_permlane32_swap(x, x, false, false));
  const uint32_t h0 = h[0], h1 = h[1];  // (a bit cast of a vector's element takes its first)
  v = op(__builtin_bit_cast(T, h0), __builtin_bit_cast(T, h1));
  const uint32_t y = __builtin_bit_cast(uint32_t, v);
  const u32x2 r = __builtin_bit_cast(u32x2, __builtin_amdgcn_permlane16_swap(y, y, false, false));
  const uint32_t r0 = r[0], r1 = r[1];
  v = op(__builtin_bit_cast(T, r0), __builtin_bit_cast(T, r1));
  v = op(v, dpp<0x128>(v));  // row_ror:8
  v = op(v, dpp<0x124>(v));  // row_ror:4
  v = op(v, dpp<0x4E>(v));   // quad_perm: 2 3 0 1
  return op(v, dpp<0xB1>(v));  // 1 0 3 2
}
__device__ __forceinline__ float wave_sum(float v) {
  return wave_reduce(v, [](float a, float b) { return a + b; });
}
__device__ __forceinline__ float wave_max(float v) {
  return wave_reduce(v, [](float a, float b) { return fmaxf(a, b); });
}
__device__ __forceinline__ int wave_sum_i(int v) {
  return wave_reduce(v, [](int a, int b) { return a + b; });
}
__device__ __forceinline__ uint32_t wave_max_u(uint32_t v) {
  return wave_reduce(v, [](uint32_t a, uint32_t b) { return a > b ? a : b; });
}
// Over each row of 16 lanes, at distances 8, 4, 2, 1.
__device__ __forceinline__ float row_sum(float v) {
  v += dpp<0x128>(v);
  v += dpp<0x124>(v);
  v += dpp<0x4E>(v);
  return v + dpp<0xB1>(v);
}
// Over the 4 lanes at distances 16 and 32, in this order.
__device__ __forceinline__ float rows_sum(float v) {
  typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
  const uint32_t x = __float_as_uint(v);
  const u32x2 r = __builtin_bit_cast(u32x2, __builtin_amdgcn_permlane16_swap(x, x, false, false));
  const uint32_t y = __float_as_uint(__uint_as_float(r[0]) + __uint_as_float(r[1]));
  const u32x2 h = __builtin_bit_cast(u32x2, __builtin_amdgcn_permlane32_swap(y, y, false, false));
  return __uint_as_float(h[0]) + __uint_as_float(h[1]);
}
// Sum over lanes 0 .. l, in lane l.
__device__ __forceinline__ int wave_scan_i(int v) {
  v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xF, 0xF, true);   // row_shr:1
  v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xF, 0xF, true);   // row_shr:2
  v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xF, 0xF, true);   // row_shr:4
  v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xF, 0xF, true);   // row_shr:8
  v += __builtin_amdgcn_update_dpp(0, v, 0x142, 0xA, 0xF, false);  // row_bcast:15, rows 1 and 3
  v += __builtin_amdgcn_update_dpp(0, v, 0x143, 0xC, 0xF, false);  // row_bcast:31, rows 2 and 3
  return v;
}
// Lane `lane`'s value (the same lane in the whole wave), in every lane.
__device__ __forceinline__ int wave_pick(int v, int lane) { return __builtin_amdgcn_readlane(v, lane); }
__device__ __forceinline__ float wave_pick(float v, int lane) {
  return __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(v), lane));
}

// Global-memory view of a generic pointer.  Pointers read from device memory
// (job tables) are generic to the compiler, which then emits flat accesses;
// flat loads also count against the LDS wait counter, so every LDS access
// after them waits for the loads.  Accessing through this view gives global
// loads and stores.
template <class T>
__device__ __forceinline__ __attribute__((address_space(1))) T* gl(T* p) {
  return (__attribute__((address_space(1))) T*)p;
}

// 16-byte global loads and stores through the global view (HIP's vector
// classes cannot be assigned across address spaces, so the data moves as a
// native 4 x 32-bit vector).
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
__device__ __forceinline__ uint4 ld_global16(const void* p) {
  const u32x4 v = *(const __attribute__((address_space(1))) u32x4*)p;
  return __builtin_bit_cast(uint4, v);
}
__device__ __forceinline__ void st_global16(void* p, uint4 x) {
  *(__attribute__((address_space(1))) u32x4*)p = __builtin_bit_cast(u32x4, x);
}
// Raw buffer view of global memory from `base` on (32-bit byte offsets, no
// swizzle, no index stride; word 3 as gfx9-family GPUs take it).  A load at
// kBufferNone is out of its range: it reads zeros and touches no memory.
constexpr int kBufferWord3 = 0x00020000;
constexpr uint32_t kBufferNone = 0x80000000u;
__device__ __forceinline__ __amdgpu_buffer_rsrc_t raw_buffer(const void* base) {
  return __builtin_amdgcn_make_buffer_rsrc((void*)base, (short)0, 0x7FFFFFFF, kBufferWord3);
}

// A 16-byte load issued unconditionally: where `ok` is false it reads 16
// zero bytes kept in device memory.  With no branch around the load and no
// select after it, the compiler counts outstanding loads exactly and needs
// the data only where it is consumed, so tiles staged ahead stay in flight
// under the matrix products instead of being waited for right away.
__device__ __align__(16) static const uint32_t kZero16[4] = {0u, 0u, 0u, 0u};
__device__ __forceinline__ uint4 ld_global16_or_zero(const void* p, bool ok) {
  return ld_global16(ok ? p : (const void*)kZero16);
}

// Barrier for LDS traffic only: waits for the wave's LDS accesses, not for its
// outstanding global loads and stores.
__device__ __forceinline__ void lds_barrier() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// A 4 x 16 block of 16-bit values in LDS, by 16 lanes: lane i gives the address
// of values 4 (i mod 4) .. of row i / 4 and gets column i.  Two such blocks (k 0
// .. 3 and 4 .. 7 of the lane's group) make a BF16 MFMA operand.
typedef short s16x4 __attribute__((ext_vector_type(4)));
__device__ __forceinline__ s16x4 lds_read_tr(const char* p) {
  return __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4*)p);
}
__device__ __forceinline__ bf16x8 lds_frag_tr(const char* lo, const char* hi) {
  return __builtin_bit_cast(bf16x8, __builtin_shufflevector(lds_read_tr(lo), lds_read_tr(hi), 0, 1, 2, 3,
                                                            4, 5, 6, 7));
}

// Index of the last of n entries with begin <= x (entry 0 begins at 0): one
// round of loads for 64 entries instead of a chain of dependent ones.
template <class Job, class Begin>
__device__ __forceinline__ int find_entry(const Job* jobs, int n, int x, Begin begin) {
  const int lane = threadIdx.x & 63;
  int at = -1;
  for (int b = 0; b < n; b += 64) {
    const bool le = b + lane < n && begin(jobs[b + lane < n ? b + lane : 0]) <= x;
    at += __popcll(__ballot(le));
  }
  return __builtin_amdgcn_readfirstlane(at);
}

// p[0] + p[stride] + ... + p[(n-1) stride], added strictly in index order;
// the loads are issued 32 at a time so their latencies overlap (slots past n
// add an exact zero).
__device__ __forceinline__ float ordered_sum(const float* __restrict__ pg, size_t stride, int n) {
  const auto p = gl(pg);
  float s = 0.f;
  for (int k = 0; k < n; k += 32) {
    float v[32];
#pragma unroll
    for (int q = 0; q < 32; ++q) v[q] = k + q < n ? p[(size_t)(k + q) * stride] : 0.f;
#pragma unroll
    for (int q = 0; q < 32; ++q) s += v[q];
  }
  return s;
}

}  // namespace edpc
