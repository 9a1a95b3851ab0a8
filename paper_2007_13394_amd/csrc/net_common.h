// Small device helpers shared by the learned correction's kernels.
#pragma once

#include <type_traits>

#include "pm_internal.h"

namespace pm {
namespace {

typedef short v4s __attribute__((ext_vector_type(4)));
typedef float v4f __attribute__((ext_vector_type(4)));
typedef __bf16 v2bf __attribute__((ext_vector_type(2)));
typedef __bf16 v8bf __attribute__((ext_vector_type(8)));

__device__ __forceinline__ float silu(float z) { return z * __builtin_amdgcn_rcpf(1.f + __expf(-z)); }
__device__ __forceinline__ float dsilu(float z)
{
    // reciprocal with one Newton step (3 instructions; an IEEE division takes about ten)
    const float d = 1.f + __expf(-z), r = __builtin_amdgcn_rcpf(d);
    const float s = d < 1e38f ? r * fmaf(-d, r, 2.f) : 0.f;
    return s + z * s * (1.f - s);
}
// round to the nearest BF16 (ties to even; the hardware conversion) and back
__device__ __forceinline__ uint16_t to_bf16(float f) { return __builtin_bit_cast(uint16_t, (__bf16)f); }
__device__ __forceinline__ float from_bf16(uint16_t b) { return __uint_as_float((uint32_t)b << 16); }
__device__ __forceinline__ float bf16r(float f) { return from_bf16(to_bf16(f)); }
// The CNN input: density contrast q 2^-S - 1 of the int64 mesh, rounded to BF16.
__device__ __forceinline__ uint16_t delta_bf16(int64_t q, double qs) { return to_bf16((float)((double)q * qs - 1.0)); }

// x / D for 0 <= x < N as one 24-bit multiply and a shift: v_mul_u32_u24 is
// full rate, while the 32-bit multiplies that a division by a constant
// otherwise becomes are quarter rate.  Exactness on the range is checked at
// compile time.
template <unsigned D, unsigned N>
struct Div24 {
    static constexpr unsigned M = (65536u + D - 1) / D;
    static constexpr bool exact()
    {
        for (unsigned x = 0; x < N; x++)
            if (((x * M) >> 16) != x / D) return false;
        return (unsigned long long)N * M < (1ull << 32);
    }
    static_assert(exact(), "multiply-shift division not exact on the range");
    __device__ static __forceinline__ int div(int x)
    {
        // written out, since the compiler turns a 24-bit multiply whose
        // operands it can bound back into the quarter-rate v_mul_lo_u32
        unsigned r;
        asm("v_mul_u32_u24 %0, %1, %2" : "=v"(r) : "s"(M), "v"((unsigned)x));
        return (int)(r >> 16);
    }
};

// Index of voxel (z, y, x) of an n^3 mesh (n <= 4096): the row index in 24-bit
// arithmetic, then one 64-bit multiply-add.
__device__ __forceinline__ int64_t vox_index(int z, int y, int x, int n)
{
    return (int64_t)(unsigned)(__mul24(z, n) + y) * (unsigned)n + (unsigned)x;
}

}  // namespace
}  // namespace pm
