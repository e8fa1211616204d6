// Storage formats of a swept field (binary64, binary32, bfloat16) as the
// kernels load and store them: aligned pairs of cells through global-memory
// pointers, and the bfloat16 rounding.
#pragma once

#include <hip/hip_runtime.h>

#include "jc_types.h"

namespace jc {

namespace {

// Global-memory views of the generic pointers held in the tables: loads
// and stores through them are global (not flat) instructions, which count
// only against the vector-memory counter, so waiting for an LDS write does
// not also wait for every load still in flight.
#define JC_GLOBAL __attribute__((address_space(1)))

typedef double v2d __attribute__((ext_vector_type(2)));
typedef float v2f __attribute__((ext_vector_type(2)));

// bfloat16: the upper half of a binary32, rounded to nearest even
__device__ __forceinline__ float bf16_to_f32(uint32_t h)
{
    return __uint_as_float(h << 16);
}

// Round to nearest even without a branch: adding 0x7fff plus the kept
// half's lowest bit carries into the upper half exactly when the dropped
// half is above one half, or equal to it with an odd kept half (equal, bit
// for bit, to the comparison form for every binary32 pattern).  A NaN
// stays a (quiet) NaN.
__device__ __forceinline__ uint32_t f32_to_bf16(float f)
{
    const uint32_t x = __float_as_uint(f);
    const uint32_t rounded = (x + 0x7fffu + ((x >> 16) & 1u)) >> 16;
    const uint32_t quiet_nan = (x >> 16) | 0x40u;
    return __builtin_isnan(f) ? quiet_nan : rounded;   // an unordered self-compare
}

// Fixed-order sum over the lanes of a wave.
__device__ __forceinline__ double wave_sum(double v)
{
    for (int o = 32; o > 0; o >>= 1)
        v = v + __shfl_xor(v, o, 64);
    return v;
}

// Storage formats of a swept field: arithmetic type C, and loads / stores
// of the 2-element aligned pair (x, x + 1) that one thread owns.
template <typename T> struct Tr;

template <> struct Tr<double> {
    using C = double;
    __device__ static void ld(const double* p, double& a, double& b)
    {
        const v2d v = *(const v2d JC_GLOBAL*)(p);
        a = v.x;
        b = v.y;
    }
    __device__ static void st(double* p, double a, double b)
    {
        v2d v;
        v.x = a;
        v.y = b;
        *(v2d JC_GLOBAL*)(p) = v;
    }
    __device__ static void st1(double* p, double a) { *(double JC_GLOBAL*)(p) = a; }
    // streaming store: the new iterate is not read again before the next
    // sweep, so it should not displace lines the current sweep re-reads
    __device__ static void stn(double* p, double a, double b)
    {
        v2d v;
        v.x = a;
        v.y = b;
        __builtin_nontemporal_store(v, (v2d JC_GLOBAL*)(p));
    }
    // a pair converted to storage once, stored whole or by element
    using P = v2d;
    __device__ static P pack(double a, double b)
    {
        v2d v;
        v.x = a;
        v.y = b;
        return v;
    }
    __device__ static void unpack(P v, C& a, C& b)
    {
        a = v.x;
        b = v.y;
    }
    __device__ static void stp(double* p, P v) { *(v2d JC_GLOBAL*)(p) = v; }
    __device__ static void stpn(double* p, P v) { __builtin_nontemporal_store(v, (v2d JC_GLOBAL*)(p)); }
    __device__ static void st1a(double* p, P v) { *(double JC_GLOBAL*)(p) = v.x; }
    __device__ static void st1b(double* p, P v) { *(double JC_GLOBAL*)(p) = v.y; }
};

template <> struct Tr<float> {
    using C = float;
    __device__ static void ld(const float* p, float& a, float& b)
    {
        const v2f v = *(const v2f JC_GLOBAL*)(p);
        a = v.x;
        b = v.y;
    }
    __device__ static void st(float* p, float a, float b)
    {
        v2f v;
        v.x = a;
        v.y = b;
        *(v2f JC_GLOBAL*)(p) = v;
    }
    __device__ static void st1(float* p, float a) { *(float JC_GLOBAL*)(p) = a; }
    __device__ static void stn(float* p, float a, float b)
    {
        v2f v;
        v.x = a;
        v.y = b;
        __builtin_nontemporal_store(v, (v2f JC_GLOBAL*)(p));
    }
    using P = v2f;
    __device__ static P pack(float a, float b)
    {
        v2f v;
        v.x = a;
        v.y = b;
        return v;
    }
    __device__ static void unpack(P v, C& a, C& b)
    {
        a = v.x;
        b = v.y;
    }
    __device__ static void stp(float* p, P v) { *(v2f JC_GLOBAL*)(p) = v; }
    __device__ static void stpn(float* p, P v) { __builtin_nontemporal_store(v, (v2f JC_GLOBAL*)(p)); }
    __device__ static void st1a(float* p, P v) { *(float JC_GLOBAL*)(p) = v.x; }
    __device__ static void st1b(float* p, P v) { *(float JC_GLOBAL*)(p) = v.y; }
};

template <> struct Tr<bf16> {
    using C = float;
    __device__ static void ld(const bf16* p, float& a, float& b)
    {
        const uint32_t w = *(const uint32_t JC_GLOBAL*)(p);    // x at the lower address
        a = bf16_to_f32(w & 0xffffu);
        b = bf16_to_f32(w >> 16);
    }
    __device__ static void st(bf16* p, float a, float b)
    {
        *(uint32_t JC_GLOBAL*)(p) = f32_to_bf16(a) | (f32_to_bf16(b) << 16);
    }
    __device__ static void st1(bf16* p, float a) { *(uint16_t JC_GLOBAL*)(p) = (uint16_t)f32_to_bf16(a); }
    __device__ static void stn(bf16* p, float a, float b)
    {
        __builtin_nontemporal_store(f32_to_bf16(a) | (f32_to_bf16(b) << 16), (uint32_t JC_GLOBAL*)(p));
    }
    using P = uint32_t;                           // x in the low half
    __device__ static P pack(float a, float b) { return f32_to_bf16(a) | (f32_to_bf16(b) << 16); }
    __device__ static void unpack(P v, C& a, C& b)
    {
        a = bf16_to_f32(v & 0xffffu);
        b = bf16_to_f32(v >> 16);
    }
    __device__ static void stp(bf16* p, P v) { *(uint32_t JC_GLOBAL*)(p) = v; }
    __device__ static void stpn(bf16* p, P v) { __builtin_nontemporal_store(v, (uint32_t JC_GLOBAL*)(p)); }
    __device__ static void st1a(bf16* p, P v) { *(uint16_t JC_GLOBAL*)(p) = (uint16_t)(v & 0xffffu); }
    __device__ static void st1b(bf16* p, P v) { *(uint16_t JC_GLOBAL*)(p) = (uint16_t)(v >> 16); }
};

}  // namespace

}  // namespace jc
