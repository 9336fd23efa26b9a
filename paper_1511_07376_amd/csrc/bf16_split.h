// A float as the exact sum of three bfloat16 parts.
#pragma once

#include <hip/hip_runtime.h>

namespace cnn {

typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x2 __attribute__((ext_vector_type(2)));

// The leading bfloat16 of v[0] (low half) and of v[1] (high half); with
// `rest`, v becomes what it leaves.  Three calls give the three parts.
__device__ inline unsigned split_step(float* v, bool rest) {
    const unsigned u = __builtin_bit_cast(unsigned, __builtin_convertvector((f32x2{v[0], v[1]}), bf16x2));
    if (rest) {
        v[0] -= __uint_as_float(u << 16);
        v[1] -= __uint_as_float(u & 0xffff0000u);
    }
    return u;
}

}  // namespace cnn
