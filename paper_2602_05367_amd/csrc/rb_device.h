// Small device helpers shared by the kernels of this library: element types,
// conversions and the fp32 -> output store.
#pragma once
#include <hip/hip_runtime.h>
#include <hip/hip_fp16.h>
#include <cstdint>

#include "rabit.h"

namespace rb {

struct bf16_t { uint16_t bits; };

__device__ __forceinline__ float to_float(__half v) { return __half2float(v); }
__device__ __forceinline__ float to_float(bf16_t v) { return __uint_as_float((uint32_t)v.bits << 16); }

// fp32 -> bfloat16, round to nearest even (NaN kept quiet)
__device__ __forceinline__ uint16_t f32_to_bf16_rne(float f)
{
    uint32_t u = __float_as_uint(f);
    if ((u & 0x7fffffffu) > 0x7f800000u) return (uint16_t)((u >> 16) | 0x0040u);
    u += 0x7fffu + ((u >> 16) & 1u);
    return (uint16_t)(u >> 16);
}

__device__ __forceinline__ void store_out(void *Y, int out_dtype, size_t idx, float v)
{
    if (out_dtype == RB_F16) {
        static_cast<__half *>(Y)[idx] = __float2half_rn(v);
    } else if (out_dtype == RB_BF16) {
        static_cast<uint16_t *>(Y)[idx] = f32_to_bf16_rne(v);
    } else {
        static_cast<float *>(Y)[idx] = v;
    }
}

// A kernel's pointer as a number: for each pointer argument of a launch the runtime looks up which allocation it lies in, some 0.05 us of
// host time, which is most of a small call
typedef unsigned long long Address;
inline Address address_of(const void *p) { return (Address)reinterpret_cast<uintptr_t>(p); }
template <typename T> __device__ __forceinline__ T *global_at(Address a)
{
    return (T *)reinterpret_cast<__attribute__((address_space(1))) T *>(a);
}

// both words of a pair moved up by n < 16 bits; what the upper one takes over from the lower one lies in its lowest n bits.  In assembly:
// the compiler would use one instruction per word, and the 64-bit shift takes as long as one of them (1.8 ns a wavefront)
__device__ __forceinline__ void shift_left(unsigned long long pair, int n, uint32_t &lower, uint32_t &upper)
{
    unsigned long long r;
    if (__builtin_constant_p(n)) {
        switch (n) {
#define RB_SHIFT(N) case N: asm("v_lshlrev_b64 %0, " #N ", %1" : "=v"(r) : "v"(pair)); break;
            RB_SHIFT(1) RB_SHIFT(2) RB_SHIFT(3) RB_SHIFT(4) RB_SHIFT(5) RB_SHIFT(6) RB_SHIFT(7) RB_SHIFT(8) RB_SHIFT(9) RB_SHIFT(10)
            RB_SHIFT(11) RB_SHIFT(12) RB_SHIFT(13) RB_SHIFT(14) RB_SHIFT(15)
#undef RB_SHIFT
        default: r = pair;
        }
    } else {
        asm("v_lshlrev_b64 %0, %1, %2" : "=v"(r) : "s"(n), "v"(pair));
    }
    lower = (uint32_t)r;
    upper = (uint32_t)(r >> 32);
}

// OR over each group of eight consecutive lanes, left in all eight: two exchanges inside the quad,
// then one with the mirrored lane of the group (7 - i, which sits in the other quad).  Data-parallel
// moves: every lane of the wavefront must be active.
__device__ __forceinline__ uint32_t or_over_8(uint32_t v)
{
    v |= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0xB1, 0xf, 0xf, false);    // quad_perm [1,0,3,2]
    v |= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x4E, 0xf, 0xf, false);    // quad_perm [2,3,0,1]
    v |= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x141, 0xf, 0xf, false);   // row_half_mirror
    return v;
}

}  // namespace rb
