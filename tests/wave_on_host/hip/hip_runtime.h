// What the device headers of csrc/ need to be compiled for the host, one wave of 64 lanes: every lane is a coroutine, and a
// cross-lane operation goes on once all lanes have come to it.  Lanes must meet the same cross-lane operations in the same order.
// Stands in for the HIP runtime's header (-I tests/wave_on_host, clang: address spaces and vector types are understood).
#pragma once
#include <math.h>
#include <setjmp.h>
#include <stdint.h>
#include <string.h>
#include <ucontext.h>

#include <functional>
#include <vector>

#define __host__
#define __device__
#define __forceinline__ inline
#ifndef __HIP_MEMORY_SCOPE_WORKGROUP
#define __HIP_MEMORY_SCOPE_WORKGROUP 3
#endif

typedef int hipError_t;
typedef void* hipStream_t;
constexpr hipError_t hipSuccess = 0;
constexpr int hipFuncAttributeMaxDynamicSharedMemorySize = 0;
inline hipError_t hipGetDevice(int* d) { *d = 0; return hipSuccess; }
inline hipError_t hipFuncSetAttribute(const void*, int, int) { return hipSuccess; }

struct uint2 { uint32_t x, y; };
struct uint4 { uint32_t x, y, z, w; };
struct float2 { float x, y; };
struct float4 { float x, y, z, w; };
inline uint2 make_uint2(uint32_t x, uint32_t y) { return { x, y }; }
inline uint4 make_uint4(uint32_t x, uint32_t y, uint32_t z, uint32_t w) { return { x, y, z, w }; }
inline float4 make_float4(float x, float y, float z, float w) { return { x, y, z, w }; }
inline uint32_t __umulhi(uint32_t a, uint32_t b) { return (uint32_t)(((uint64_t)a * b) >> 32); }
template <typename A, typename B> inline A bits_as(B b) { A a; static_assert(sizeof(A) == sizeof(B), ""); memcpy(&a, &b, sizeof(a)); return a; }
inline int __double2hiint(double x) { return (int)(bits_as<uint64_t>(x) >> 32); }
inline int __double2loint(double x) { return (int)(uint32_t)bits_as<uint64_t>(x); }
inline double __hiloint2double(int hi, int lo) { return bits_as<double>(((uint64_t)(uint32_t)hi << 32) | (uint32_t)lo); }
inline double __longlong_as_double(long long x) { return bits_as<double>(x); }
inline long long __double_as_longlong(double x) { return bits_as<long long>(x); }
inline float __uint_as_float(uint32_t x) { return bits_as<float>(x); }
inline float __int_as_float(int x) { return bits_as<float>(x); }
inline int __float_as_int(float x) { return bits_as<int>(x); }
inline int min(int a, int b) { return a < b ? a : b; }
inline int max(int a, int b) { return a > b ? a : b; }
inline unsigned min(unsigned a, unsigned b) { return a < b ? a : b; }

namespace host_wave {
struct Lane { int x = 0; };
inline Lane now;                            // the lane that runs (threadIdx)
inline ucontext_t lane_start[64];
inline jmp_buf caller, lane_at[64];         // (a lane is entered by its context, from then on by jumps: those make no system call)
inline bool ended[64];
inline int slot[2][64], turn[64];           // values of the operation under way, by parity of the lane's count of operations
inline const std::function<void()>* body;
inline void run_lane(int l) { (*body)(); ended[l] = true; _longjmp(caller, 1); }
// All lanes through f.
inline void run(const std::function<void()>& f)
{
    static std::vector<char> stacks(64 * (1 << 18));
    body = &f;
    for (int l = 0; l < 64; ++l) {
        ended[l] = false;
        turn[l] = 0;
        getcontext(&lane_start[l]);
        lane_start[l].uc_stack.ss_sp = stacks.data() + ((size_t)l << 18);
        lane_start[l].uc_stack.ss_size = 1 << 18;
        lane_start[l].uc_link = nullptr;
        makecontext(&lane_start[l], reinterpret_cast<void (*)()>(run_lane), 1, l);
    }
    static volatile bool left, entered;
    for (entered = false, left = true; left; entered = true) {
        left = false;
        for (now.x = 0; now.x < 64; ++now.x) {
            if (ended[now.x]) continue;
            if (_setjmp(caller) == 0) {
                if (entered) _longjmp(lane_at[now.x], 1);
                setcontext(&lane_start[now.x]);
            }
            left = left || !ended[now.x];
        }
    }
}
// The lanes' values of x, once all have come here; they stand until the operation after the next.
inline const int* meet(int x)
{
    const int l = now.x, k = turn[l]++ & 1;
    slot[k][l] = x;
    if (_setjmp(lane_at[l]) == 0) _longjmp(caller, 1);
    return slot[k];
}
inline unsigned long long ballot(bool b)
{
    const int* const v = meet(b);
    unsigned long long m = 0;
    for (int l = 0; l < 64; ++l) m |= (unsigned long long)(v[l] & 1) << l;
    return m;
}
inline int readlane(int x, int l) { return meet(x)[l & 63]; }
inline int readfirstlane(int x) { return meet(x)[0]; }
// Data-parallel moves: the lane's source, or -1 where it has none.
inline int source(int ctrl, int l)
{
    const int row = l & ~15, at = l & 15;
    if (ctrl < 0x100) return (l & ~3) + ((ctrl >> (2 * (l & 3))) & 3);                    // quad_perm
    if (ctrl >= 0x101 && ctrl <= 0x10f) return at + (ctrl & 15) < 16 ? l + (ctrl & 15) : -1;   // row_shl
    if (ctrl >= 0x111 && ctrl <= 0x11f) return at >= (ctrl & 15) ? l - (ctrl & 15) : -1;  // row_shr
    if (ctrl == 0x130) return l < 63 ? l + 1 : -1;                                        // wave_shl:1
    if (ctrl == 0x138) return l > 0 ? l - 1 : -1;                                         // wave_shr:1
    if (ctrl == 0x140) return row + 15 - at;                                              // row_mirror
    if (ctrl == 0x141) return (l & ~7) + 7 - (l & 7);                                     // row_half_mirror
    if (ctrl == 0x142) return l >= 16 ? row - 1 : -1;                                     // row_bcast:15
    if (ctrl == 0x143) return l >= 32 ? 31 : -1;                                          // row_bcast:31
    __builtin_trap();
}
inline int update_dpp(int old, int x, int ctrl, int row_mask, int bank_mask, bool bound)
{
    const int l = now.x, s = source(ctrl, l);
    const int* const v = meet(x);
    if (!((row_mask >> (l >> 4)) & 1) || !((bank_mask >> ((l >> 2) & 3)) & 1)) return old;
    return s >= 0 ? v[s] : bound ? 0 : old;
}
}  // namespace host_wave
#define threadIdx host_wave::now
#define __builtin_amdgcn_ballot_w64 host_wave::ballot
#define __builtin_amdgcn_readlane host_wave::readlane
#define __builtin_amdgcn_readfirstlane host_wave::readfirstlane
#define __builtin_amdgcn_update_dpp host_wave::update_dpp
template <typename T> inline T __shfl_xor(T x, int m, int) { static_assert(sizeof(T) == 4, ""); return bits_as<T>(host_wave::meet(bits_as<int>(x))[host_wave::now.x ^ m]); }
template <typename T> T __shfl_up(T, int, int);
void __syncthreads();
int atomicMin(int*, int);
int atomicMax(int*, int);
