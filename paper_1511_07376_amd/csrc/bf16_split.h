// A float as the exact sum of three bfloat16 parts.
#pragma once

#include <hip/hip_runtime.h>

namespace cnn {

typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x2 __attribute__((ext_vector_type(2)));

// The leading bfloat16 of v[0] (low half) and of v[1] (high half); with
// `rest`, v becomes what it leaves.  Three calls give the three parts.  What
// the second call leaves is the third part, exactly, unless it has bits below
// bfloat16's smallest subnormal, 2^-133 (possible for magnitudes below 2^-107
// only).
__device__ inline unsigned split_step(float* v, bool rest) {
    const unsigned u = __builtin_bit_cast(unsigned, __builtin_convertvector((f32x2{v[0], v[1]}), bf16x2));
    if (rest) {
        v[0] -= __uint_as_float(u << 16);
        v[1] -= __uint_as_float(u & 0xffff0000u);
    }
    return u;
}

// To be called between the second and the third call of split_step: gathers in
// `lost` whether a third part is not exact (its low 16 bits are then not all
// zero; split_lost).  In asm, since the compiler regroups a chain of ORs over a
// whole slab and keeps the operands in registers until its end.
__device__ inline void note_lost(unsigned& lost, const float* v) {
    asm("v_or3_b32 %0, %0, %1, %2" : "+v"(lost) : "v"(v[0]), "v"(v[1]));
}
__device__ inline bool split_lost(unsigned lost) { return (lost & 0xffff) != 0; }

}  // namespace cnn
