// Device-side helpers shared by the gfx950 kernels: I/O element access for float32 and
// bfloat16 storage, and the float32 evaluation of softplus and SiLU used by the layer
// (delta = softplus(dt + dt_bias); gate = silu(z)).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace mamba {

typedef uint16_t bf16_t;  // bfloat16 bit pattern in memory

constexpr float kLog2e = 1.4426950408889634f;
constexpr float kLn2 = 0.6931471805599453f;

__device__ __forceinline__ float bf16_to_f32(uint32_t bits) { return __uint_as_float(bits << 16); }
__device__ __forceinline__ float bf16_lo(uint32_t pair) { return __uint_as_float(pair << 16); }
__device__ __forceinline__ float bf16_hi(uint32_t pair) { return __uint_as_float(pair & 0xffff0000u); }

// float32 -> bfloat16, round to nearest even (one rounding, at the store).
__device__ __forceinline__ uint32_t f32_to_bf16(float f)
{
    return (uint32_t)__builtin_bit_cast(uint16_t, (__bf16)f);
}
__device__ __forceinline__ uint32_t f32x2_to_bf16x2(float lo, float hi)
{
    typedef float f2 __attribute__((ext_vector_type(2)));
    typedef __bf16 b2 __attribute__((ext_vector_type(2)));
    f2 v = {lo, hi};
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, b2));
}

__device__ __forceinline__ float ld_io(const float *p, int64_t i) { return p[i]; }
__device__ __forceinline__ float ld_io(const bf16_t *p, int64_t i) { return bf16_to_f32(p[i]); }
__device__ __forceinline__ void st_io(float *p, int64_t i, float v) { p[i] = v; }
__device__ __forceinline__ void st_io(bf16_t *p, int64_t i, float v) { p[i] = (bf16_t)f32_to_bf16(v); }

// 2^v and log2(v) on the hardware transcendental unit (v_exp_f32 / v_log_f32, ~1 ulp).
__device__ __forceinline__ float exp2_hw(float v) { return __builtin_amdgcn_exp2f(v); }
__device__ __forceinline__ float log2_hw(float v) { return __builtin_amdgcn_logf(v); }
__device__ __forceinline__ float rcp_hw(float v) { return __builtin_amdgcn_rcpf(v); }

// Kernel arguments that are used last would be fetched last, a trip to the scalar cache ahead of a kernel's final stores; a value
// requested early but used only under a condition would be requested there.  Naming them where they should be there keeps both.
template <typename P> __device__ __forceinline__ void arg_here(P p) { asm volatile("" ::"s"(p)); }
template <typename... P> __device__ __forceinline__ void args_here(P... p) { (arg_here(p), ...); }
__device__ __forceinline__ void values_here(float &v) { asm volatile("" : "+v"(v)); }

// softplus(v) = log(1 + e^v) = max(v, 0) + log1p(w), w = e^-|v| <= 1, to ~1e-7 relative (plus the
// rounding of the exp2 argument for large |v|).  The sum s = 1 + w drops w's low bits; they are
// recovered exactly as r = w - (s - 1) and added back: log1p(w) = log(s) + log1p(r / s), which is
// log(s) + r to first order (s is in [1, 2] and |r| <= 2^-24, so r and r / s differ by < 2^-25).
// No threshold and no overflow: w never exceeds 1.
__device__ __forceinline__ float softplus_f32(float v)
{
    const float w = exp2_hw(-fabsf(v) * kLog2e);
    const float s = 1.0f + w;
    const float r = w - (s - 1.0f);
    return fmaxf(v, 0.0f) + fmaf(log2_hw(s), kLn2, r);
}

// silu(v) = v / (1 + e^-v)
__device__ __forceinline__ float silu_f32(float v)
{
    return v * rcp_hw(1.0f + exp2_hw(-v * kLog2e));
}

// Transcendental instructions in runs.  ns an instruction takes of a SIMD with 4 wavefronts, each kind alone: mul 1.2, fma 1.5, exp2
// 3.6 to 4.0.  At every change between the two kinds time is lost, those of different wavefronts included.  So a run keeps what is next to it in the
// program out of it (the fences: scalar, memory and LDS instructions may cross, vector ones not) and keeps the other wavefronts of
// the SIMD from cutting in (the priority of a wave, raised for the length of the run; the others issue what is not vector
// work, and have their turn after it).  A bare loop of state updates (mul, exp2, mul, fma, fma; sixteen exponentials a run), ns of
// a SIMD per update at 2, 3 and 4 wavefronts: 11.9, 11.6 and 11.5 in the compiler's order, 11.2, 11.0 and 10.7 in runs, 8.3, 9.2 and 8.1
// with the priority, less than the parts alone add up to (9.0 to 9.4).
constexpr int kSchedMemoryOnly = 0x4 | 0x10 | 0x20 | 0x40 | 0x80 | 0x100 | 0x200;
template <typename F> __device__ __forceinline__ void transcendental_run(F issue)
{
    __builtin_amdgcn_sched_barrier(kSchedMemoryOnly);
    __builtin_amdgcn_s_setprio(1);
    issue();
    __builtin_amdgcn_s_setprio(0);
    __builtin_amdgcn_sched_barrier(kSchedMemoryOnly);
}
template <int COUNT> __device__ __forceinline__ void exp2_run(float (&v)[COUNT])
{
    transcendental_run([&]() __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < COUNT; ++i) v[i] = exp2_hw(v[i]);
    });
}
// softplus_f32 and silu_f32 of COUNT values, to the bit
template <int COUNT> __device__ __forceinline__ void softplus_run(float (&v)[COUNT])
{
    float w[COUNT], s[COUNT], g[COUNT];
#pragma unroll
    for (int i = 0; i < COUNT; ++i) w[i] = -fabsf(v[i]) * kLog2e;
    exp2_run(w);
#pragma unroll
    for (int i = 0; i < COUNT; ++i) s[i] = 1.0f + w[i];
    transcendental_run([&]() __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < COUNT; ++i) g[i] = log2_hw(s[i]);
    });
#pragma unroll
    for (int i = 0; i < COUNT; ++i) v[i] = fmaxf(v[i], 0.0f) + fmaf(g[i], kLn2, w[i] - (s[i] - 1.0f));
}
template <int COUNT> __device__ __forceinline__ void silu_run(float (&v)[COUNT])
{
    float w[COUNT];
#pragma unroll
    for (int i = 0; i < COUNT; ++i) w[i] = -v[i] * kLog2e;
    exp2_run(w);
#pragma unroll
    for (int i = 0; i < COUNT; ++i) w[i] = 1.0f + w[i];
    transcendental_run([&]() __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < COUNT; ++i) w[i] = rcp_hw(w[i]);
    });
#pragma unroll
    for (int i = 0; i < COUNT; ++i) v[i] = v[i] * w[i];
}

}  // namespace mamba
