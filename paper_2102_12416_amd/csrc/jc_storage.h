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

// bfloat16: the upper half of a binary32, rounded to nearest even.
__device__ __forceinline__ float bf16_lo(uint32_t w) { return __uint_as_float(w << 16); }
__device__ __forceinline__ float bf16_hi(uint32_t w) { return __uint_as_float(w & 0xffff0000u); }

// A pair rounded and packed (a in the low half) by the conversion instruction
// of gfx950: one instruction for ten (shift, bit field, add and NaN select of
// each value).  Compared with the shift form -- add 0x7fff plus the kept
// half's lowest bit, NaN kept quiet -- over all 2^32 binary32 patterns in
// both halves: the same bits, denormals and NaN included
// (tests/device_check.hip).
__device__ __forceinline__ uint32_t bf16_pair(float a, float b)
{
    typedef __bf16 v2b __attribute__((ext_vector_type(2)));
    v2f v;
    v.x = a;
    v.y = b;
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, v2b));
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
        a = bf16_lo(w);
        b = bf16_hi(w);
    }
    __device__ static void st(bf16* p, float a, float b)
    {
        *(uint32_t JC_GLOBAL*)(p) = bf16_pair(a, b);
    }
    __device__ static void st1(bf16* p, float a) { *(uint16_t JC_GLOBAL*)(p) = (uint16_t)bf16_pair(a, a); }
    __device__ static void stn(bf16* p, float a, float b)
    {
        __builtin_nontemporal_store(bf16_pair(a, b), (uint32_t JC_GLOBAL*)(p));
    }
    using P = uint32_t;                           // x in the low half
    __device__ static P pack(float a, float b) { return bf16_pair(a, b); }
    __device__ static void unpack(P v, C& a, C& b)
    {
        a = bf16_lo(v);
        b = bf16_hi(v);
    }
    __device__ static void stp(bf16* p, P v) { *(uint32_t JC_GLOBAL*)(p) = v; }
    __device__ static void stpn(bf16* p, P v) { __builtin_nontemporal_store(v, (uint32_t JC_GLOBAL*)(p)); }
    __device__ static void st1a(bf16* p, P v) { *(uint16_t JC_GLOBAL*)(p) = (uint16_t)(v & 0xffffu); }
    __device__ static void st1b(bf16* p, P v) { *(uint16_t JC_GLOBAL*)(p) = (uint16_t)(v >> 16); }
};

}  // namespace

}  // namespace jc
