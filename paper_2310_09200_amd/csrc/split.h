// Two-term half-precision split of FP32 values (internal; not installed).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

namespace bb {

typedef float f32x2 __attribute__((ext_vector_type(2)));

// hi = H(v), lo = H(v - hi) of two values, packed; fp16's lo words in one
// instruction each (v_fma_mix: v * 1 - hi in FP32, rounded to fp16).
template <class H>
__device__ __forceinline__ void split2(float v0, float v1, uint32_t& hi, uint32_t& lo) {
  typedef H h2 __attribute__((ext_vector_type(2)));
  const f32x2 v = {v0, v1};
  const h2 h = __builtin_convertvector(v, h2);
  hi = __builtin_bit_cast(uint32_t, h);
  if constexpr (std::is_same<H, _Float16>::value) {
    uint32_t r;
    asm("v_fma_mixlo_f16 %0, %1, 1.0, -%2 op_sel_hi:[0,0,1]" : "=v"(r) : "v"(v0), "v"(hi));
    asm("v_fma_mixhi_f16 %0, %1, 1.0, -%2 op_sel:[0,0,1] op_sel_hi:[0,0,1]"
        : "+v"(r)
        : "v"(v1), "v"(hi));
    lo = r;
  } else {
    const f32x2 d = {v0 - (float)h[0], v1 - (float)h[1]};
    lo = __builtin_bit_cast(uint32_t, __builtin_convertvector(d, h2));
  }
}

}  // namespace bb
