// Device helpers shared by the attention kernels.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace ff {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

#define LDS_PTR(T, p) ((__attribute__((address_space(3))) T*)(p))

// N 1 KB copies from global memory straight into LDS: copy i takes 16 bytes
// per lane from base + off[i] + 1024 i into LDS at dst + 1024 i + 16 lane.  The
// instruction's immediate offset moves both addresses, so m0 (the LDS base) is
// written once for all N; callers fold -1024 i into off[i] and lower base by
// 1024 (N - 1) so that every per-lane offset stays non-negative.  Written out so
// that the compiler does not track these copies: their completion is waited
// for explicitly (vmcnt) before the copied bytes are read.
template <int N>
__device__ inline void lds_copy_blocks(uint32_t dst, const char* base, const uint32_t (&off)[N]) {
  static_assert(N == 1 || N == 2 || N == 4, "1 KB copies per wave and tensor");
  if constexpr (N == 1)
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2"
                 :: "s"(dst), "v"(off[0]), "s"(base) : "memory");
  else if constexpr (N == 2)
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\t"
                 "global_load_lds_dwordx4 %1, %3\n\t"
                 "global_load_lds_dwordx4 %2, %3 offset:1024"
                 :: "s"(dst), "v"(off[0]), "v"(off[1]), "s"(base) : "memory");
  else
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\t"
                 "global_load_lds_dwordx4 %1, %5\n\t"
                 "global_load_lds_dwordx4 %2, %5 offset:1024\n\t"
                 "global_load_lds_dwordx4 %3, %5 offset:2048\n\t"
                 "global_load_lds_dwordx4 %4, %5 offset:3072"
                 :: "s"(dst), "v"(off[0]), "v"(off[1]), "v"(off[2]), "v"(off[3]), "s"(base) : "memory");
}

__device__ inline uint32_t pack_bf16(float a, float b) {
  f32x2 f = {a, b};
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(f, bf16x2));
}

// max and sum over the lanes n, n + 16, n + 32, n + 48 (the four lane groups
// holding one query's keys)
__device__ inline float max_across_groups(float x) {
  auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  const float y = fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
  r = __builtin_amdgcn_permlane32_swap(__float_as_uint(y), __float_as_uint(y), false, false);
  return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}

__device__ inline float sum_across_groups(float x) {
  auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  const float y = __uint_as_float(r[0]) + __uint_as_float(r[1]);
  r = __builtin_amdgcn_permlane32_swap(__float_as_uint(y), __float_as_uint(y), false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

// 64-bit value of lane `lane` (wave-uniform index).  The builtin works on
// signed 32-bit words: each half is widened as unsigned, so a low word with
// its top bit set does not sign-extend into the high word.
__device__ inline uint64_t readlane_u64(uint64_t v, int lane) {
  const uint32_t lo = uint32_t(__builtin_amdgcn_readlane(int(uint32_t(v)), lane));
  const uint32_t hi = uint32_t(__builtin_amdgcn_readlane(int(uint32_t(v >> 32)), lane));
  return (uint64_t(hi) << 32) | uint64_t(lo);
}

// s_waitcnt immediate: vmcnt = vm; lgkmcnt and expcnt not waited for
constexpr int waitcnt_vm(int vm) { return (vm & 15) | ((vm >> 4) << 14) | (7 << 4) | (15 << 8); }

}  // namespace ff
