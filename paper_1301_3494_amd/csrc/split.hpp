// Device code shared by the kernels that write BF16x3 operands.
#pragma once
#include <hip/hip_runtime.h>

#include <cstdint>

namespace pdmrg {

// A value split for BF16x3: its FP32 rounding f = hi + lo with hi and lo
// bf16 (both rounded to nearest even), packed as one word, hi in the low half.
typedef float pf2 __attribute__((ext_vector_type(2)));
typedef __bf16 pb2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ uint32_t pack_split(float f) {
    const pf2 x{f, 0.0f};
    const pb2 h = __builtin_convertvector(x, pb2);
    const pb2 l = __builtin_convertvector(x - __builtin_convertvector(h, pf2), pb2);
    return (__builtin_bit_cast(uint32_t, h) & 0xffffu) | (__builtin_bit_cast(uint32_t, l) << 16);
}

}  // namespace pdmrg
