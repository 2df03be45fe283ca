// Cross-lane helpers of the tree builders and the verification walk: DPP moves, lane reads, wave-wide maximum, sum
// and scan; LDS accesses between waves that do not meet at a barrier.
#pragma once
#include "vocab_common.h"

namespace dyspec {

// LDS by its own address space: 32-bit addresses and ds instructions also where a generic pointer would
// leave the compiler in doubt.
template <typename T> using lds_t = T __attribute__((address_space(3)));
template <typename T> __device__ __forceinline__ lds_t<T>* lds_at(uint32_t byte_address) { return (lds_t<T>*)byte_address; }
__device__ __forceinline__ uint32_t lds_base(const void* p) { return (uint32_t)(size_t)(lds_t<const void>*)p; }
// A word shared by waves that do not meet at a barrier: read and written as it stands, in program
// order.  (The LDS operations of a wave take effect in the order they are issued; relaxed atomics keep the
// compiler from caching or splitting them, the empty asm from moving other accesses across.)
template <typename T> __device__ __forceinline__ T lds_now(lds_t<T>* p)
{
    asm volatile("" ::: "memory");
    const T v = __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    asm volatile("" ::: "memory");
    return v;
}
template <typename T> __device__ __forceinline__ void lds_set(lds_t<T>* p, T v)
{
    asm volatile("" ::: "memory");
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    asm volatile("" ::: "memory");
}
typedef unsigned long long u64;
__device__ __forceinline__ u64 ballot(bool b) { return __builtin_amdgcn_ballot_w64(b); }

// A value known to be the same in every lane, declared so (scalar registers, scalar branches).
__device__ __forceinline__ uint32_t uniform(uint32_t x) { return (uint32_t)__builtin_amdgcn_readfirstlane((int)x); }
__device__ __forceinline__ u64 uniform(u64 x) { return (u64)uniform((uint32_t)x) | ((u64)uniform((uint32_t)(x >> 32)) << 32); }
__device__ __forceinline__ int uniform(int x) { return __builtin_amdgcn_readfirstlane(x); }
__device__ __forceinline__ float uniform(float x) { return __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(x))); }
__device__ __forceinline__ double uniform(double x) { return __longlong_as_double((long long)uniform((u64)__double_as_longlong(x))); }
template <typename T> __device__ __forceinline__ T* uniform(T* p) { return (T*)(T __attribute__((address_space(1)))*)uniform((u64)p); }      // global memory

// Cross-lane moves of the vector ALU (DPP) for the serial builder's reductions and scan; a
// shuffle would go through the LDS crossbar and wait for it at every step.
constexpr int kDppXor1 = 0xB1;          // quad_perm [1,0,3,2]
constexpr int kDppXor2 = 0x4E;          // quad_perm [2,3,0,1]
constexpr int kDppHalfMirror = 0x141;   // lane i of a group of 8 <-> lane 7-i
constexpr int kDppMirror = 0x140;       // lane i of a row of 16 <-> lane 15-i
constexpr int kDppBcast15 = 0x142;      // lane 15 of a row to the next row
constexpr int kDppBcast31 = 0x143;      // lane 31 to rows 2 and 3
constexpr int kDppWaveShl1 = 0x130;     // lane i: lane i + 1's
constexpr int kDppWaveShr1 = 0x138;     // lane i: lane i - 1's
template <int CTRL, int ROW_MASK = 0xf>
__device__ __forceinline__ int dpp_or_zero(int x)   // the picked lane's x; 0 where there is none or the row is masked off
{
    return __builtin_amdgcn_update_dpp(0, x, CTRL, ROW_MASK, 0xf, ROW_MASK == 0xf);     // (no source lane: 0 either way)
}
template <int CTRL, int ROW_MASK = 0xf>
__device__ __forceinline__ double dpp_or_zero(double x)
{
    return __hiloint2double(dpp_or_zero<CTRL, ROW_MASK>(__double2hiint(x)), dpp_or_zero<CTRL, ROW_MASK>(__double2loint(x)));
}
// Largest value of the wave (values >= -1, no NaN), the same in every lane.
__device__ __forceinline__ double wave_max_dpp(double x)
{
    x = fmax(x, dpp_or_zero<kDppXor1>(x));
    x = fmax(x, dpp_or_zero<kDppXor2>(x));
    x = fmax(x, dpp_or_zero<kDppHalfMirror>(x));
    x = fmax(x, dpp_or_zero<kDppMirror>(x));
    double r[4];
#pragma unroll
    for (int k = 0; k < 4; ++k)
        r[k] = __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(x), 16 * k), __builtin_amdgcn_readlane(__double2loint(x), 16 * k));
    return fmax(fmax(r[0], r[1]), fmax(r[2], r[3]));
}
// The same for non-negative integers.
__device__ __forceinline__ int wave_max_dpp_int(int x)
{
    x = max(x, dpp_or_zero<kDppXor1>(x));
    x = max(x, dpp_or_zero<kDppXor2>(x));
    x = max(x, dpp_or_zero<kDppHalfMirror>(x));
    x = max(x, dpp_or_zero<kDppMirror>(x));
    return max(max(__builtin_amdgcn_readlane(x, 0), __builtin_amdgcn_readlane(x, 16)),
               max(__builtin_amdgcn_readlane(x, 32), __builtin_amdgcn_readlane(x, 48)));
}
// Sum over the wave, the same in every lane.
__device__ __forceinline__ double wave_sum_dpp(double x)
{
    x += dpp_or_zero<kDppXor1>(x);
    x += dpp_or_zero<kDppXor2>(x);
    x += dpp_or_zero<kDppHalfMirror>(x);
    x += dpp_or_zero<kDppMirror>(x);
    double r[4];
#pragma unroll
    for (int k = 0; k < 4; ++k)
        r[k] = __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(x), 16 * k), __builtin_amdgcn_readlane(__double2loint(x), 16 * k));
    return (r[0] + r[1]) + (r[2] + r[3]);
}
// Sums over each row of 16 lanes of N values a lane (N = 2, 8 or 16), scattered: lane l gets the sum of value l % N.  Values are
// added to the mirrored lane's until the lane's lower bits can name what is left; from there on every step exchanges half of the
// values with a lane that differs in the bit which names the half.  (Mirrored lanes differ in the lower bits as well: the steps
// of the higher bits come first, while nothing depends on the lower ones.)  N = 16: 15 adds against 64.
template <int N>
__device__ __forceinline__ double row_sums(double (&x)[N])
{
    static_assert(N == 2 || N == 8 || N == 16, "bits 0 .. log2 N - 1 of the lane name the value");
    const int lane = threadIdx.x & (kWave - 1);
    auto all = [&](auto ctrl_c) __attribute__((always_inline)) {
#pragma unroll
        for (int k = 0; k < N; ++k) x[k] += dpp_or_zero<decltype(ctrl_c)::value>(x[k]);
    };
    auto fold = [&](auto n_c, auto ctrl_c, int bit) __attribute__((always_inline)) {
        constexpr int H = decltype(n_c)::value / 2;        // value k stays with bit clear, k + H with bit set
        const bool up = lane & bit;
#pragma unroll
        for (int k = 0; k < H; ++k) {
            const double keep = up ? x[k + H] : x[k], give = up ? x[k] : x[k + H];
            x[k] = keep + dpp_or_zero<decltype(ctrl_c)::value>(give);
        }
    };
    const std::integral_constant<int, kDppMirror> mirror;
    const std::integral_constant<int, kDppHalfMirror> half_mirror;
    const std::integral_constant<int, kDppXor2> xor2;
    const std::integral_constant<int, kDppXor1> xor1;
    if constexpr (N == 16) fold(std::integral_constant<int, 16>{}, mirror, 8); else all(mirror);
    if constexpr (N >= 8) fold(std::integral_constant<int, 8>{}, half_mirror, 4); else all(half_mirror);
    if constexpr (N >= 8) fold(std::integral_constant<int, 4>{}, xor2, 2); else all(xor2);
    fold(std::integral_constant<int, 2>{}, xor1, 1);
    return x[0];
}
__device__ __forceinline__ float readlane_f32(float x, int l);
// The same in fp32.
__device__ __forceinline__ float wave_sum_f32_dpp(float x)
{
    x += __int_as_float(dpp_or_zero<kDppXor1>(__float_as_int(x)));
    x += __int_as_float(dpp_or_zero<kDppXor2>(__float_as_int(x)));
    x += __int_as_float(dpp_or_zero<kDppHalfMirror>(__float_as_int(x)));
    x += __int_as_float(dpp_or_zero<kDppMirror>(__float_as_int(x)));
    return (readlane_f32(x, 0) + readlane_f32(x, 16)) + (readlane_f32(x, 32) + readlane_f32(x, 48));
}
// Inclusive scan over the wave in lane order.
__device__ __forceinline__ double wave_scan_dpp(double x)
{
    x += dpp_or_zero<0x111>(x);                  // row_shr:1, 2, 4, 8: scan inside each row of 16
    x += dpp_or_zero<0x112>(x);
    x += dpp_or_zero<0x114>(x);
    x += dpp_or_zero<0x118>(x);
    x += dpp_or_zero<kDppBcast15, 0xa>(x);       // rows 1 and 3 add the total of the row before
    x += dpp_or_zero<kDppBcast31, 0xc>(x);       // rows 2 and 3 add the total of the first two rows
    return x;
}

__device__ __forceinline__ double readlane_f64(double x, int l)
{
    return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(x), l), __builtin_amdgcn_readlane(__double2loint(x), l));
}
__device__ __forceinline__ float readlane_f32(float x, int l)
{
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(x), l));
}
}  // namespace dyspec
