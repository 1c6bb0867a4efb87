// Device helpers shared by the kernels that form decays and scaled operands from the bf16 streams.
#pragma once
#include <hip/hip_runtime.h>

namespace wkv6 {

typedef _Float16 half2v __attribute__((ext_vector_type(2)));

constexpr float kLog2e = 1.4426950408889634f;

__device__ __forceinline__ float bf16_lo(unsigned bits) { return __uint_as_float(bits << 16); }
__device__ __forceinline__ float bf16_hi(unsigned bits) { return __uint_as_float(bits & 0xffff0000u); }

__device__ __forceinline__ unsigned pack_h2(float a, float b) {
    half2v p;
    p.x = static_cast<_Float16>(a);
    p.y = static_cast<_Float16>(b);
    return __builtin_bit_cast(unsigned, p);
}

// packed fp16 multiply of two pairs
__device__ __forceinline__ unsigned mul_h2(unsigned a, unsigned b) {
    return __builtin_bit_cast(unsigned, __builtin_bit_cast(half2v, a) * __builtin_bit_cast(half2v, b));
}

// w = exp(-exp(x)) through two base-2 exponentials (x=-inf -> 1, x=+inf -> 0):
// log2(e) * exp(x) = exp2(x * log2(e) + log2(log2(e))), so the factor of the second exponential
// rides in the argument of the first.
// Also hands back the scaled inner exponential log2(e) * exp(x), which the Finch-C2 key factor needs.
__device__ __forceinline__ float decay_of(float x, float& e_log2e) {
    constexpr float kLog2Log2e = 0.5287663729448977f;
    e_log2e = __builtin_amdgcn_exp2f(__builtin_fmaf(x, kLog2e, kLog2Log2e));
    return __builtin_amdgcn_exp2f(-e_log2e);
}

// Finch-C2 key factor 1 - w = 1 - exp(-e), e = exp(x), without the cancellation of the plain
// subtraction for long-memory channels (w close to 1): below e = 2^-5 the alternating series
// e (1 - e/2 + e^2/6 - e^3/24), whose first dropped term is under 1e-8 of the result there;
// above it the subtraction loses at most five bits of an fp32 value.
__device__ __forceinline__ float one_minus_decay(float e_log2e, float w) {
    const float e = e_log2e * 0.6931471805599453f;      // exp(x) from the decay's own inner exponential
    const float series = e * __builtin_fmaf(e, __builtin_fmaf(e, __builtin_fmaf(e, -1.f / 24.f, 1.f / 6.f), -0.5f), 1.f);
    return e < 0.03125f ? series : 1.f - w;
}

// MODE.FP16_OVFL = 1 (hwreg id 1, bit 23, one bit): fp16 results that overflow, conversions
// included, are clamped to +-65504 instead of becoming infinite, so operands beyond the fp16
// range saturate as the header promises; true infinities are preserved.
__device__ __forceinline__ void clamp_fp16_overflow() { __builtin_amdgcn_s_setreg(1 | (23 << 6) | (0 << 11), 1); }

// Raw buffer descriptor (stride 0, 32-bit data format) over span_bytes - off bytes from base + off, empty if that
// is negative.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t chunk_rsrc(const char* base, long long off, long long span_bytes) {
    long long left = span_bytes - off;
    if (left < 0) left = 0;
    if (left > 0x7fffffffLL) left = 0x7fffffffLL;
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<char*>(base + off), 0, static_cast<int>(left), 0x00020000);
}

}  // namespace wkv6
