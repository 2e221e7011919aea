// Device helpers of all kernels: pieces of a wavefront's work that several translation units share.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>
#include <utility>

namespace {

typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));

// two fp32 values -> bf16 (nearest even), the first in the low half
__device__ __forceinline__ uint32_t pack_bf16(float a, float b) {
    const f32x2 two = {a, b};
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(two, bf16x2));
}

// f(integral_constant<int, 0>) ... f(integral_constant<int, N - 1>): a loop whose counter is a constant in every iteration
// by construction (an unrolling pragma is a request; when it is not honoured, register arrays indexed by the counter go
// to scratch memory)
template <int... I, typename F>
__device__ __forceinline__ void static_for_impl(std::integer_sequence<int, I...>, F&& f) {
    (f(std::integral_constant<int, I>{}), ...);
}
template <int N, typename F>
__device__ __forceinline__ void static_for(F&& f) {
    static_for_impl(std::make_integer_sequence<int, N>{}, static_cast<F&&>(f));
}

// 16 bytes per lane from global memory straight into LDS: lane L's piece lands at lds_base + 16 L (lds_base is
// wave-uniform).  Written as an instruction rather than through the builtin: the compiler orders every later LDS read
// behind a builtin load it cannot tell apart (a full vmcnt wait in the middle of the pipeline); here the kernel itself
// waits (vmcnt) before the barrier that publishes a stage.
__device__ __forceinline__ void lds_load16(const void* gsrc, const void* lds_base) {
    const uint32_t base = static_cast<uint32_t>(reinterpret_cast<uintptr_t>(
        (const __attribute__((address_space(3))) void*)lds_base));
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off" : : "s"(base), "v"(gsrc) : "memory", "m0");
}

// sum over the two halves of the wavefront
__device__ __forceinline__ float half_swap_sum(float x) {
    auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

// Reductions over the 64 lanes of a wavefront on the vector ALU (data-parallel-primitive operand modifiers inside a row of
// 16 lanes, then the gfx950 row and half swaps): every lane ends with the result.  The shuffle intrinsics go through the
// LDS crossbar instead, a round trip of its own per step.
template <typename F>
__device__ __forceinline__ float wave_reduce(float x, F op) {
    auto dpp = [](float v, auto ctrl) __attribute__((always_inline)) {
        return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), decltype(ctrl)::value, 0xf, 0xf, true));
    };
    x = op(x, dpp(x, std::integral_constant<int, 0xB1>{}));    // lane ^ 1 (quad_perm 1,0,3,2)
    x = op(x, dpp(x, std::integral_constant<int, 0x4E>{}));    // lane ^ 2 (quad_perm 2,3,0,1): the quad's result in its four lanes
    x = op(x, dpp(x, std::integral_constant<int, 0x141>{}));   // mirror inside 8 lanes: the other quad
    x = op(x, dpp(x, std::integral_constant<int, 0x140>{}));   // mirror inside the row of 16: the other half row
    // (the swaps exchange rows between their two operands and return both.  Their elements are copied to scalars before the
    // bit cast: applied to an element of the returned vector the cast reads element 0 with this compiler.)
    auto r = __builtin_amdgcn_permlane16_swap(__builtin_bit_cast(unsigned, x), __builtin_bit_cast(unsigned, x), false, false);
    const unsigned r0 = r[0], r1 = r[1];
    x = op(__builtin_bit_cast(float, r0), __builtin_bit_cast(float, r1));        // the neighbouring row
    auto q = __builtin_amdgcn_permlane32_swap(__builtin_bit_cast(unsigned, x), __builtin_bit_cast(unsigned, x), false, false);
    const unsigned q0 = q[0], q1 = q[1];
    return op(__builtin_bit_cast(float, q0), __builtin_bit_cast(float, q1));     // the other half of the wavefront
}

__device__ __forceinline__ float wave_sum(float x) {
    return wave_reduce(x, [](float a, float b) { return a + b; });
}

__device__ __forceinline__ float wave_max(float x) {
    return wave_reduce(x, [](float a, float b) { return fmaxf(a, b); });
}

}  // namespace
