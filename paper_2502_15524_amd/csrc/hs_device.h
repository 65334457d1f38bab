// Device-side helpers shared by the engine's HIP kernels (gfx950, wave64).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

typedef uint16_t bf16_t;  // raw bfloat16 bits
typedef __bf16 bf16x8_v __attribute__((ext_vector_type(8)));
typedef float f32x4_v __attribute__((ext_vector_type(4)));
typedef float f32x16_v __attribute__((ext_vector_type(16)));

// 16 bytes = 8 bf16 values.
struct alignas(16) pack8 {
  uint32_t w[4];
};

__device__ __forceinline__ float bf2f(bf16_t b) {
  return __uint_as_float(static_cast<uint32_t>(b) << 16);
}

// float -> bf16, round to nearest even: one v_cvt_pk_bf16_f32 for two values,
// where integer arithmetic takes about ten VALU instructions (the same bits for
// every finite value; a NaN stays a NaN).
typedef __bf16 bf16x2_v __attribute__((ext_vector_type(2)));
typedef float f32x2_v __attribute__((ext_vector_type(2)));
__device__ __forceinline__ uint32_t pack2bf(float lo, float hi) {
  return __builtin_bit_cast(uint32_t, __builtin_convertvector((f32x2_v{lo, hi}), bf16x2_v));
}

__device__ __forceinline__ bf16_t f2bf(float f) {
  return static_cast<bf16_t>(pack2bf(f, 0.f));
}

__device__ __forceinline__ float lo_bf(uint32_t w) { return __uint_as_float(w << 16); }
__device__ __forceinline__ float hi_bf(uint32_t w) { return __uint_as_float(w & 0xFFFF0000u); }

__device__ __forceinline__ pack8 ld16(const void* p) {
  return *reinterpret_cast<const pack8*>(p);
}
// 16 bytes read once per call (weights, cached keys and values): a
// non-temporal load
__device__ __forceinline__ pack8 ld16_nt(const void* p) {
  typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
  const u32x4 v = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(p));
  pack8 r;
  r.w[0] = v[0];
  r.w[1] = v[1];
  r.w[2] = v[2];
  r.w[3] = v[3];
  return r;
}
__device__ __forceinline__ void st16(void* p, const pack8& v) {
  *reinterpret_cast<pack8*>(p) = v;
}
__device__ __forceinline__ pack8 zero8() {
  pack8 z;
  z.w[0] = z.w[1] = z.w[2] = z.w[3] = 0u;
  return z;
}

__device__ __forceinline__ bf16x8_v as_bf16x8(const pack8& v) {
  return __builtin_bit_cast(bf16x8_v, v);
}

// 2^x on the hardware exp unit.
__device__ __forceinline__ float fast_exp2(float x) { return __builtin_amdgcn_exp2f(x); }

__device__ __forceinline__ float silu_f(float g) {
  // g * sigmoid(g), with e^-g = 2^(-g log2 e)
  return g / (1.0f + fast_exp2(-g * 1.4426950408889634f));
}

// Copies from global memory straight into LDS. The instruction takes its LDS
// address from M0; a scalar write of M0 needs one wait state before a load that
// reads it, and the assembler adds none inside inline assembly: hence the s_nop
// (one issue slot per 1 KiB).
typedef int v4i_t __attribute__((ext_vector_type(4)));

constexpr int kRsrcWord3 = 0x00020000;  // raw buffer, 32-bit data format

__device__ __forceinline__ v4i_t buf_rsrc(const void* p, uint64_t bytes) {
  const uint64_t a = reinterpret_cast<uint64_t>(p);
  const uint32_t n = bytes >= 0xFFFFFFFFull ? 0xFFFFFFFFu : (uint32_t)bytes;
  return v4i_t{(int)(uint32_t)a, (int)(uint32_t)((a >> 32) & 0xFFFFu), (int)n, kRsrcWord3};
}

// 64 lanes x 16 bytes from rsrc + voff + soff into LDS bytes [lds, lds + 1024)
__device__ __forceinline__ void dma16(v4i_t rsrc, int voff, int soff, uint32_t lds) {
  asm volatile("s_mov_b32 m0, %3\n\ts_nop 0\n\tbuffer_load_dwordx4 %0, %1, %2 offen lds"
               :: "v"(voff), "s"(rsrc), "s"(__builtin_amdgcn_readfirstlane(soff)),
                  "s"(__builtin_amdgcn_readfirstlane(lds))
               : "memory", "m0");
}
__device__ __forceinline__ void dma16(v4i_t rsrc, int voff, uint32_t lds) {
  asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tbuffer_load_dwordx4 %0, %1, 0 offen lds"
               :: "v"(voff), "s"(rsrc), "s"(__builtin_amdgcn_readfirstlane(lds))
               : "memory", "m0");
}

// One thread's 16 bytes of a pull from pinned host memory (units i of n16): the
// loads are system-coherent (sc0 sc1), so they see what the host wrote before
// the launch, never a cached copy of an earlier call's values.
__device__ __forceinline__ void pull16(const int32_t* host, int32_t* dev, int n16, int i) {
  if (i >= n16) return;
  typedef unsigned u32x4_v __attribute__((ext_vector_type(4)));
  constexpr int kSystem = 1 | 16;  // sc0 | sc1
  const __amdgpu_buffer_rsrc_t r =
      __builtin_amdgcn_make_buffer_rsrc(const_cast<int32_t*>(host), 0, n16 * 16, 0x00020000);
  const u32x4_v v = __builtin_amdgcn_raw_buffer_load_b128(r, i * 16, 0, kSystem);
  *reinterpret_cast<u32x4_v*>(dev + (int64_t)i * 4) = v;
}

// Rotate-half RoPE of one pair: x1 at index i of a head's first half, x2 at
// i + D/2, angle with cosine c and sine s. Every kernel that rotates uses
// these two (with explicit fused multiply-adds), so they all round alike.
__device__ __forceinline__ float rope_first(float x1, float x2, float c, float s) {
  return fmaf(x1, c, -(x2 * s));
}
__device__ __forceinline__ float rope_second(float x1, float x2, float c, float s) {
  return fmaf(x2, c, x1 * s);
}

template <typename T>
__device__ __forceinline__ T wave_sum(T v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}
