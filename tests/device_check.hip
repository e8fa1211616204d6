// Device checks of the helpers that the sweeps share, built by
// __graft_entry__.build() and run by tests/test_gpu_device_helpers.py: the
// bfloat16 rounding of jc_storage.h over all 2^32 binary32 patterns in both
// halves of a pair, and the divisions of jc_div6.h, the rarely taken branch
// among them, against the device's IEEE division.
#include <hip/hip_runtime.h>

#include "jc_div6.h"
#include "jc_storage.h"

namespace {

// Round to nearest even by shifts; NaN stays NaN, made quiet.
__device__ uint32_t bf16_shift(uint32_t u)
{
    if ((u & 0x7fffffffu) > 0x7f800000u)
        return (u >> 16) | 0x40u;
    return (u + 0x7fffu + ((u >> 16) & 1u)) >> 16;
}

// 2^32 patterns, 2^24 threads of 256 patterns each; the other half of the pair
// holds another pattern (its complement).
__global__ void __launch_bounds__(256) k_bf16(unsigned long long* bad)
{
    const uint32_t t = blockIdx.x * 256u + threadIdx.x;
    unsigned int n = 0;
    for (uint32_t k = 0; k < 256u; ++k) {
        const uint32_t u = k << 24 | t;
        const uint32_t lo = jc::bf16_pair(__uint_as_float(u), __uint_as_float(~u));
        n += (lo & 0xffffu) != bf16_shift(u);
        n += (lo >> 16) != bf16_shift(~u);
    }
    if (n)
        atomicAdd(bad, (unsigned long long)n);
}

template <typename C> __device__ bool same(C a, C b) { return (a != a && b != b) || (a == b && signbit(a) == signbit(b)); }

// All binary32 patterns through div6 and, beside another value, div6_pair.
__global__ void __launch_bounds__(256) k_div6_f32(unsigned long long* bad)
{
    const uint32_t t = blockIdx.x * 256u + threadIdx.x;
    unsigned int n = 0;
    for (uint32_t k = 0; k < 256u; ++k) {
        const float s = __uint_as_float(k << 24 | t), p = __uint_as_float(~(k << 24 | t));
        float a, b;
        jc::div6_pair(s, p, a, b);
        n += !same(jc::div6(s), s / 6.0f) + !same(a, s / 6.0f) + !same(b, p / 6.0f);
    }
    if (n)
        atomicAdd(bad, (unsigned long long)n);
}

// value[i] in place `place` of div6_quad beside the three values after it.
__global__ void __launch_bounds__(256) k_div6_quad(const double* value, int count, int place, unsigned long long* bad)
{
    const int i = (int)(blockIdx.x * 256u + threadIdx.x);
    if (i >= count)
        return;
    double s[4], v[4];
    for (int k = 0; k < 4; ++k)
        s[(place + k) & 3] = value[(i + k) % count];
    jc::div6_quad(s[0], s[1], s[2], s[3], v[0], v[1], v[2], v[3]);
    unsigned int n = 0;
    for (int k = 0; k < 4; ++k)
        n += !same(v[k], s[k] / 6.0);
    if (n)
        atomicAdd(bad, (unsigned long long)n);
}

}  // namespace

extern "C" int check_bf16_pair(void* bad, void* stream)
{
    hipLaunchKernelGGL(k_bf16, dim3(1u << 16), dim3(256), 0, static_cast<hipStream_t>(stream),
                       static_cast<unsigned long long*>(bad));
    return (int)hipGetLastError();
}

extern "C" int check_div6_f32(void* bad, void* stream)
{
    hipLaunchKernelGGL(k_div6_f32, dim3(1u << 16), dim3(256), 0, static_cast<hipStream_t>(stream),
                       static_cast<unsigned long long*>(bad));
    return (int)hipGetLastError();
}

extern "C" int check_div6_quad(const void* values, int count, int place, void* bad, void* stream)
{
    if (count < 4 || place < 0 || place > 3)
        return (int)hipErrorInvalidValue;
    hipLaunchKernelGGL(k_div6_quad, dim3((unsigned)((count + 255) / 256)), dim3(256), 0, static_cast<hipStream_t>(stream),
                       static_cast<const double*>(values), count, place, static_cast<unsigned long long*>(bad));
    return (int)hipGetLastError();
}
