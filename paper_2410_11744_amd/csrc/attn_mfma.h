// What the two matrix-core attention kernels share: vector types, compile-time loops, direct loads to LDS, the
// LDS arrangement of K and V rows.
#pragma once
#include <utility>

#include "dyspec_device.h"

namespace dyspec {

// Compile-time loop: f(integral_constant<int, 0>), ..., f(integral_constant<int, N-1>).
template <typename F, int... I>
__device__ __forceinline__ void static_for_impl(F&& f, std::integer_sequence<int, I...>)
{
    (f(std::integral_constant<int, I>{}), ...);
}
template <int N, typename F>
__device__ __forceinline__ void static_for(F&& f)
{
    static_for_impl(static_cast<F&&>(f), std::make_integer_sequence<int, N>{});
}
template <typename F>
__device__ __forceinline__ void with_bool(bool b, F&& f)
{
    if (b) f(std::true_type{}); else f(std::false_type{});
}

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float floatx16 __attribute__((ext_vector_type(16)));
typedef float floatx2 __attribute__((ext_vector_type(2)));
typedef __attribute__((address_space(1))) const void* global_ptr;
typedef __attribute__((address_space(3))) void* lds_ptr;
typedef short short4v __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) short4v* lds_short4;
typedef __attribute__((address_space(3))) const bf16x8* lds_bf16x8;

// v_exp_f32 without the denormal-range fix-up: inputs below -126 give 0, which is what the
// softmax wants.
__device__ __forceinline__ float fast_exp2(float x) { return __builtin_amdgcn_exp2f(x); }
__device__ __forceinline__ float and_bits(float x, int m) { return __int_as_float(__float_as_int(x) & m); }
// One wave-wide direct load: lane i moves 16 bytes from (base + voff_i) to LDS byte
// lds_base + 16*i.  Issued as inline assembly so that the compiler does not pair every later
// LDS read with a wait for these loads; the caller waits (wait_direct_loads) before the
// barrier that publishes the stage.
__device__ __forceinline__ void direct_load_16(const void* base, uint32_t voff, uint32_t lds_base)
{
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2"
                 :: "s"(lds_base), "v"(voff), "s"(base) : "m0", "memory");
}
__device__ __forceinline__ void wait_direct_loads() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }
__device__ __forceinline__ uint32_t lds_address(const void* p)
{
    return (uint32_t)(size_t)(lds_ptr)(p);
}

// max of three without the NaN-quieting moves fmaxf would add in front
__device__ __forceinline__ float max3(float a, float b, float c)
{
    float r;
    asm("v_max3_f32 %0, %1, %2, %3" : "=v"(r) : "v"(a), "v"(b), "v"(c));
    return r;
}

// Rows of K, V and Q sit unpadded in LDS, in 16-byte chunks XOR-swizzled so that the 16-byte reads of K (lane n:
// key row n) and the transposing reads of V of a wave spread over all 64 banks: chunk c of K row r sits at
// chunk position c ^ swz_k(r), of V row r at c ^ swz_v(r).
template <int D> __device__ __forceinline__ constexpr int swz_k(int r) { return D == 128 ? (r & 15) : ((r >> 1) & 7); }
template <int D> __device__ __forceinline__ constexpr int swz_v(int r) { return D == 128 ? ((r & 3) << 2) : 0; }

}  // namespace dyspec
