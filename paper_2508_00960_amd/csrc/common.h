// Scalar helpers shared by the kernels: storage types, activations.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace phantom {

typedef __bf16 bf16_t;

enum { ACT_IDENTITY = 0, ACT_RELU = 1, ACT_GELU = 2 };

template <typename T> __device__ __forceinline__ float to_f32(T v) { return (float)v; }
template <typename T> __device__ __forceinline__ T from_f32(float v) { return (T)v; }

// sigma(a): identity, ReLU, or GELU = a * Phi(a) in its erf form (no tanh approximation)
__device__ __forceinline__ float act_apply(int act, float a)
{
    if (act == ACT_RELU) return a > 0.f ? a : 0.f;
    if (act == ACT_GELU) return 0.5f * a * (1.f + erff(a * 0.70710678118654752f));
    return a;
}

// sigma'(a).  ReLU'(0) = 0.  GELU' = Phi(a) + a * phi(a).
__device__ __forceinline__ float act_deriv(int act, float a)
{
    if (act == ACT_RELU) return a > 0.f ? 1.f : 0.f;
    if (act == ACT_GELU) {
        float Phi = 0.5f * (1.f + erff(a * 0.70710678118654752f));
        float phi = 0.39894228040143268f * __expf(-0.5f * a * a);
        return Phi + a * phi;
    }
    return 1.f;
}

// The same for the activations whose derivative can be read off their output (all but GELU).  The bf16 epilogues use these
// where GELU cannot occur: erff and expf inlined eight times per unrolled pass made them 70 KB of code that every
// workgroup fetches cold.
template <int N> __device__ __forceinline__ void piecewise_both(int act, float (&x)[N], float (&deriv)[N])      // in place
{
    if (act == ACT_RELU) {                             // uniform
#pragma unroll
        for (int u = 0; u < N; ++u) { deriv[u] = x[u] > 0.f ? 1.f : 0.f; x[u] = x[u] > 0.f ? x[u] : 0.f; }
    } else {
#pragma unroll
        for (int u = 0; u < N; ++u) deriv[u] = 1.f;
    }
}

// GELU and its derivative together, for bf16 outputs: erf by the five-term rational formula of Abramowitz &
// Stegun 7.1.26 (absolute error of erf below 1.5e-7, far under a bf16 rounding step), whose exp(-z^2) with
// z = |a| / sqrt(2) is the same exponential that phi(a) needs: one v_exp, one v_rcp and some 18 other instructions instead of
// two library calls per element.  The epilogues that evaluate it run on every element of a layer's output
// with nothing left to overlap them with.  1 / (1 + p z) is v_rcp and one Newton step, which leave about half a unit in the last place, as the
// division did that took eleven instructions (31 in all).  Errors as before: s and s' 4.2e-7 and 2.9e-7 at most on [-12, 12].  Epilogue of a layer
// update of 1024 + 960 at batch 4096 8430 -> 6870 clocks; 8 such layers forward 215.4 -> 209.2 us, 4 of 2048 + 96 at 8192 364.1 -> 348.6.
__device__ __forceinline__ void gelu_both(float a, float &y, float &d)
{
    const float x = fmaf(fminf(fabsf(a), 1e18f), 0.3275911f * 0.70710678118654752f, 1.f);      // (finite: the Newton step makes 0 * infinity of an infinite one)
    const float r = __builtin_amdgcn_rcpf(x);
    const float t = fmaf(r, fmaf(-x, r, 1.f), r);
    const float e = __builtin_amdgcn_exp2f(a * a * (-0.5f * 1.4426950408889634f));
    // half the formula's coefficients: h = (1 - erf(z)) / 2 = Phi(-|a|)
    const float h = t * fmaf(t, fmaf(t, fmaf(t, fmaf(t, 0.5f * 1.061405429f, 0.5f * -1.453152027f), 0.5f * 1.421413741f), 0.5f * -0.284496736f), 0.5f * 0.254829592f) * e;
    const float Phi = a < 0.f ? h : 1.f - h;
    y = a * Phi;
    d = fmaf(a, 0.39894228040143268f * e, Phi);
}

// A piece of the kernel's one argument, read from the kernel-argument segment where it is needed, at a byte offset that the compiler
// cannot see through.  As ordinary arguments (or by a word-by-word selection between two blocks) all of them move to the top of
// the kernel and, out of scalar registers, are spilled one by one before the next is loaded: a chain of load-wait-spill rounds in
// front of the first product (four blocks of 600 bytes: 3 us).  An epilogue's part is read behind the reduction loop, for the same reason: with
// both parts at the top the scalar registers do not hold them.
template <typename Part>
__device__ __forceinline__ Part args_at(size_t offset)
{
    constexpr int WORDS = sizeof(Part) / 4;
    union Words { Part p; uint32_t w[WORDS]; __device__ Words() {} };
    Words out;
#if defined(__HIP_DEVICE_COMPILE__)
    asm volatile("" : "+s"(offset) :: "memory");
    typedef const uint32_t __attribute__((address_space(4))) *ArgWords;
    const ArgWords in = (ArgWords)((const char __attribute__((address_space(4))) *)__builtin_amdgcn_kernarg_segment_ptr() + offset);
#pragma unroll
    for (int i = 0; i < WORDS; ++i) out.w[i] = in[i];
#endif
    return out.p;
}

// Reads one word of every 64 bytes of a piece of the kernel's argument, so that a later args_at finds it in the scalar cache.
template <typename Part>
__device__ __forceinline__ void touch_args(size_t offset)
{
#if defined(__HIP_DEVICE_COMPILE__)
    typedef const uint32_t __attribute__((address_space(4))) *ArgWords;
    const ArgWords in = (ArgWords)((const char __attribute__((address_space(4))) *)__builtin_amdgcn_kernarg_segment_ptr() + offset);
    constexpr int LINES = (int)(sizeof(Part) + 63) / 64;
    uint32_t w[LINES];
#pragma unroll
    for (int i = 0; i < LINES; ++i) w[i] = in[min(i * 16, (int)(sizeof(Part) / 4) - 1)];
#pragma unroll
    for (int i = 0; i < LINES; ++i) asm volatile("" :: "s"(w[i]));
#endif
}

// x / d with magic = ceil(2^32 / d) (0 for d = 1), x below 2^31: a few scalar instructions in the place of some thirty
__device__ __forceinline__ int div_by(int x, int d, uint32_t magic)
{
    const uint32_t q = __umulhi((uint32_t)x, magic);       // at most one too high
    return d == 1 ? x : (int)(q - (q * (uint32_t)d > (uint32_t)x ? 1u : 0u));
}
__host__ __device__ constexpr uint32_t div_magic(int d) { return d > 1 ? (uint32_t)((0x100000000ull + (uint32_t)d - 1) / (uint32_t)d) : 0u; }

}  // namespace phantom
