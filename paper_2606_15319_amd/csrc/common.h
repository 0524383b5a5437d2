// Shared device helpers for the gfx950 kernels of libardit.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace ardit {

typedef uint16_t bf16_t;  // storage type of every bf16 tensor
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));  // 16-byte register chunk

constexpr int kWave = 64;
constexpr int kNumXcd = 8;   // MI355X: 8 XCDs; workgroups are dispatched round-robin over them

__device__ __forceinline__ float bf2f(bf16_t b) {
  return __uint_as_float(static_cast<uint32_t>(b) << 16);
}

// fp32 -> bf16, round to nearest even (hardware conversion on gfx950)
__device__ __forceinline__ bf16_t f2bf(float f) {
  return __builtin_bit_cast(bf16_t, static_cast<__bf16>(f));
}

__device__ __forceinline__ uint32_t pack_bf16x2(float lo, float hi) {
  bf16x2 v = {static_cast<__bf16>(lo), static_cast<__bf16>(hi)};
  return __builtin_bit_cast(uint32_t, v);
}

// unpack 8 bf16 held in a uint4 into fp32
__device__ __forceinline__ void unpack8(const uint4& u, float* f) {
  const uint32_t w[4] = {u.x, u.y, u.z, u.w};
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    f[2 * i] = __uint_as_float(w[i] << 16);
    f[2 * i + 1] = __uint_as_float(w[i] & 0xffff0000u);
  }
}

__device__ __forceinline__ uint4 pack8(const float* f) {
  uint4 u;
  u.x = pack_bf16x2(f[0], f[1]);
  u.y = pack_bf16x2(f[2], f[3]);
  u.z = pack_bf16x2(f[4], f[5]);
  u.w = pack_bf16x2(f[6], f[7]);
  return u;
}

// Max / sum of x over the four 16-lane rows of a wave (lanes l, l ^ 16, l ^ 32,
// l ^ 48), the same value in every lane: two row swaps on the VALU
// (v_permlane16_swap, v_permlane32_swap), no LDS traffic and no wait.
// Operands combine in the same pairs as with xor shuffles, so results match
// those bit for bit.
__device__ __forceinline__ float rows4_max(float x) {
  auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  x = fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
  r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
__device__ __forceinline__ float rows4_sum(float x) {
  auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  x = __uint_as_float(r[0]) + __uint_as_float(r[1]);
  r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

__device__ __forceinline__ float wave_sum(float v) {
#pragma unroll
  for (int m = 32; m >= 1; m >>= 1) v += __shfl_xor(v, m, kWave);
  return v;
}

// Division by a runtime-invariant positive divisor via multiply-high
// (round-up method of Granlund and Montgomery); valid for 0 <= n < 2^31.
struct FastDiv {
  uint32_t d;
  uint32_t mul;
  uint32_t shift;
};

__host__ inline FastDiv make_fastdiv(uint32_t d) {
  FastDiv f;
  f.d = d;
  uint32_t l = 0;
  while ((1ull << l) < d) ++l;
  f.shift = l;
  f.mul = static_cast<uint32_t>(((1ull << 32) * ((1ull << l) - d)) / d + 1);
  return f;
}

__device__ __forceinline__ uint32_t fdiv(uint32_t n, const FastDiv& f) {
  uint32_t t = __umulhi(n, f.mul);
  return (t + n) >> f.shift;
}

// 16 bytes per lane from base + off to LDS byte address m0 + 16 * lane.  base
// and m0 are the same for every lane of the wave and live in scalar
// registers, so issuing a load costs no vector instruction.
__device__ __forceinline__ void lds_dma16(const char* base, uint32_t off, uint32_t m0) {
  asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %2"
               :: "v"(off), "s"(m0), "s"(base) : "m0");
}

// A pointer the compiler may hold in vector registers, made scalar (it is the
// same in every lane).  readfirstlane returns int, so each half goes through
// uint32_t before it is widened: a low half with bit 31 set must not be
// sign-extended into the high half.
__device__ __forceinline__ const char* uniform_ptr(const void* p) {
  const uint64_t b = reinterpret_cast<uint64_t>(p);
  const uint32_t hi = static_cast<uint32_t>(__builtin_amdgcn_readfirstlane(static_cast<uint32_t>(b >> 32)));
  const uint32_t lo = static_cast<uint32_t>(__builtin_amdgcn_readfirstlane(static_cast<uint32_t>(b)));
  return reinterpret_cast<const char*>((static_cast<uint64_t>(hi) << 32) | lo);
}
// The same from a 64-bit address per lane.
__device__ __forceinline__ void lds_dma16(const char* addr, uint32_t m0) {
  asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, off"
               :: "v"(addr), "s"(m0) : "m0");
}
// 4 bytes per lane to LDS byte address m0 + 4 * lane.
__device__ __forceinline__ void lds_dma4(const char* base, uint32_t off, uint32_t m0) {
  asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dword %0, %2"
               :: "v"(off), "s"(m0), "s"(base) : "m0");
}
// LDS byte address of a shared array, in a scalar register.
__device__ __forceinline__ uint32_t lds_address(const void* p) {
  return static_cast<uint32_t>(__builtin_amdgcn_readfirstlane(static_cast<uint32_t>(
      reinterpret_cast<uintptr_t>((__attribute__((address_space(3))) const char*)p))));
}

// An attention's running maximum before any key: below every finite scaled score
// (fp32 scores times log2(e) / sqrt(d) stay above -6.2e37 at d = 64).
constexpr float kNoMax = -3.0e38f;

__device__ __forceinline__ float gelu_tanh(float y) {
  // 0.5 y (1 + tanh z) = y * sigmoid(2 z) = y / (1 + 2^(-2 z log2(e))),
  // z = sqrt(2/pi) (y + 0.044715 y^3): one exp2 and one reciprocal; for large
  // |y| the power goes to 0 or +inf and the result to y or -0
  constexpr float c1 = -2.0f * 0.7978845608028654f * 1.4426950408889634f;
  constexpr float c2 = c1 * 0.044715f;
  const float u = y * fmaf(c2, y * y, c1);
  return y * __builtin_amdgcn_rcpf(1.0f + __builtin_amdgcn_exp2f(u));
}

}  // namespace ardit
