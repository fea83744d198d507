// What the matrix-core kernels for many hidden rows share: operand types, compile-time loops, and the two lane tricks of
// the bracketed selection's epilogue.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

namespace sv {

typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef float f32x16_t __attribute__((ext_vector_type(16)));
typedef float f32x4_t __attribute__((ext_vector_type(4)));

// loops whose index must be a compile-time constant inside the body (an instruction's immediate operand)
template <int I, int N, typename F>
__device__ __forceinline__ void static_for(F&& f) {
    if constexpr (I < N) {
        f(std::integral_constant<int, I>{});
        static_for<I + 1, N>(f);
    }
}

// dst with lanes LO and HI replaced by the two halves of the wavefront-uniform mask m (two v_writelane_b32).
// The mask comes straight from a vector comparison: on this architecture a vector instruction that reads a
// scalar register written by the vector instruction just before it needs two wait states in between; the
// compiler inserts them for its own instructions, not for the operands of an asm block, hence the s_nop.
template <int LO, int HI>
__device__ __forceinline__ uint32_t write_lanes(uint32_t dst, uint64_t m) {
    static_assert(LO >= 0 && LO < 64 && HI >= 0 && HI < 64, "lanes of a 64-wide wavefront");
    asm("s_nop 1\n\tv_writelane_b32 %0, %1, %3\n\tv_writelane_b32 %0, %2, %4"
        : "+v"(dst)
        : "s"((uint32_t)m), "s"((uint32_t)(m >> 32)), "n"(LO), "n"(HI));
    return dst;
}

// 2 x + (this lane's bit of the wavefront-wide mask m): one add-with-carry whose carry-in is the mask.  The mask
// must come from a scalar instruction (see write_lanes for why not straight from a vector comparison).
__device__ __forceinline__ uint32_t shift_in_lane_bit(uint32_t x, uint64_t m) {
    uint64_t carry_out;
    asm volatile("v_addc_co_u32_e64 %0, %1, %0, %0, %2" : "+v"(x), "=s"(carry_out) : "s"(m));
    return x;
}

}  // namespace sv
