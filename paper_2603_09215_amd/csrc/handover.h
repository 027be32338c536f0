// What the launches that stay (one_row.h, small_steps.h) share: words that carry a value and its number from one workgroup to
// another, sums over a wave in registers, and arguments that are read again where they are used.
#pragma once
#include "device_common.h"

namespace spark {

// A value and the number of what it belongs to (a phase, a layer) in one 64-bit word, through device-scope accesses.  Who needs
// it asks until the number is there: no flush, acknowledgement or flag lies between.  How it asks is each kernel's own: with 256
// workgroups the questions hold up the answers, with 32 they don't.
typedef unsigned long long hand_word;
__device__ __forceinline__ void put_word(hand_word *p, float v, unsigned tag) {
  __hip_atomic_store(p, ((hand_word)tag << 32) | __float_as_uint(v), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ hand_word peek_word(const hand_word *p) { return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }

#define HAND_DPP(v, ctrl, rows) __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), ctrl, rows, 0xf, false))
// sums over the halves of the wave, in the last lane of each
__device__ __forceinline__ float half_totals_last(float v) {
  v += HAND_DPP(v, 0x111, 0xf);   // row_shr 1, 2, 4, 8: the last lane of a row of 16 has the row's sum
  v += HAND_DPP(v, 0x112, 0xf);
  v += HAND_DPP(v, 0x114, 0xf);
  v += HAND_DPP(v, 0x118, 0xf);
  v += HAND_DPP(v, 0x142, 0xa);   // row_bcast 15 into rows 1 and 3
  return v;
}
// sum over the wave, in its last lane
__device__ __forceinline__ float wave_total_last(float v) {
  v = half_totals_last(v);
  v += HAND_DPP(v, 0x143, 0xc);   // row_bcast 31 into rows 2 and 3
  return v;
}
__device__ __forceinline__ float wave_total(float v) {
  return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(wave_total_last(v)), 63));
}
// ... the last addition in 64 bits
__device__ __forceinline__ double wave_total64(float v) {
  const int h = __float_as_int(half_totals_last(v));
  return (double)__int_as_float(__builtin_amdgcn_readlane(h, 31)) + (double)__int_as_float(__builtin_amdgcn_readlane(h, 63));
}
// sum over each 16 lanes, in all of them
__device__ __forceinline__ float row16_total(float v) {
  v += HAND_DPP(v, 0x121, 0xf);   // row_ror 1, 2, 4, 8
  v += HAND_DPP(v, 0x122, 0xf);
  v += HAND_DPP(v, 0x124, 0xf);
  v += HAND_DPP(v, 0x128, 0xf);
  return v;
}
__device__ __forceinline__ float wave_largest(float v) {
  v = fmaxf(v, HAND_DPP(v, 0x121, 0xf));
  v = fmaxf(v, HAND_DPP(v, 0x122, 0xf));
  v = fmaxf(v, HAND_DPP(v, 0x124, 0xf));
  v = fmaxf(v, HAND_DPP(v, 0x128, 0xf));
  const int a = __float_as_int(v);
  const float m0 = fmaxf(__int_as_float(__builtin_amdgcn_readlane(a, 0)), __int_as_float(__builtin_amdgcn_readlane(a, 16)));
  const float m1 = fmaxf(__int_as_float(__builtin_amdgcn_readlane(a, 32)), __int_as_float(__builtin_amdgcn_readlane(a, 48)));
  return fmaxf(m0, m1);
}
#undef HAND_DPP

// The arguments of the kernel that runs (one struct), made anew where they are used: kept over a loop over layers or steps
// they and what follows from them fill the scalar registers several times over, and the vector registers behind them.
template <typename Args> __device__ __forceinline__ const Args &kernel_args() {
  typedef const __attribute__((address_space(4))) Args *Ptr;
  Ptr p = (Ptr)__builtin_amdgcn_kernarg_segment_ptr();
  asm volatile("" : "+s"(p));
  return *(const Args *)p;
}

}  // namespace spark
