// Device-side helpers shared by the gfx950 kernels: bf16 <-> fp32, the
// saturating FP8 cast, the SwiGLU product and its derivatives, reductions.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace ssg {

constexpr int kE4M3 = 0;
constexpr int kE5M2 = 1;
constexpr int kBF16 = 2;            // operand type of the unquantized (bf16) GEMMs, beside the two FP8 formats

template <int FMT> struct Fp8Traits;
// overflow_above = fmax plus half the spacing of the top binade: a magnitude beyond it is kept finite only by
// the clamp of the saturating cast (a value between fmax and it rounds to fmax by itself)
template <> struct Fp8Traits<kE4M3> { static constexpr float fmax = 448.0f, overflow_above = 464.0f; };
template <> struct Fp8Traits<kE5M2> { static constexpr float fmax = 57344.0f, overflow_above = 61440.0f; };

__device__ __forceinline__ float bf16_bits_to_f32(uint32_t b) { return __uint_as_float(b << 16); }

// fp32 -> bf16 bits, round to nearest even (NaN stays NaN).
__device__ __forceinline__ uint32_t f32_to_bf16_bits(float f) {
    uint32_t u = __float_as_uint(f);
    if ((u & 0x7fffffffu) > 0x7f800000u) return (u >> 16) | 0x40u;
    u += 0x7fffu + ((u >> 16) & 1u);
    return u >> 16;
}

// Two fp32 -> one packed pair of bf16 (lo in bits 0..15), round to nearest even, with the chip's
// conversion instruction (v_cvt_pk_bf16_f32): one operation instead of a dozen per pair.
typedef __bf16 ssg_bf16x2 __attribute__((ext_vector_type(2)));
typedef float ssg_f32x2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ uint32_t pack_bf16x2(float lo, float hi) {
    const ssg_f32x2 f = {lo, hi};
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(f, ssg_bf16x2));
}

// Per-tensor scale (Section 2; Q of Eq. 2): fl32(fmax / amax), 1 for an empty
// range, clamped to the largest finite float; optionally rounded down to a
// power of two by clearing the mantissa.
__device__ __forceinline__ float scale_from_amax(float amax, float fmax, int pow2) {
    float s = 1.0f;
    if (amax > 0.0f) {
        s = __fdiv_rn(fmax, amax);
        s = fminf(s, 3.402823466e+38f);
    }
    if (pow2) s = __uint_as_float(__float_as_uint(s) & 0xff800000u);
    return s;
}

// The per-channel factors of Smooth-SwiGLU (Section 4.4) from the channel's largest |h|: s = fl32(448 / a) and
// s^-1 = fl32(a / 448), both 1 for an all-zero channel.
__device__ __forceinline__ float smooth_factor(float a) { return scale_from_amax(a, 448.0f, 0); }
__device__ __forceinline__ float smooth_factor_inv(float a) { return a > 0.0f ? __fdiv_rn(a, 448.0f) : 1.0f; }

// Two fp32 values -> two FP8 codes in the low 16 bits.  The hardware
// conversion rounds to nearest even through the subnormal range but turns
// out-of-range magnitudes into NaN/Inf codes, so the value is clamped to the
// largest finite magnitude first.  NaN keeps its sign and becomes S.1111111.
template <int FMT>
__device__ __forceinline__ uint32_t satcast_pk2(float a, float b) {
    constexpr float fmax = Fp8Traits<FMT>::fmax;
    float ca = __builtin_amdgcn_fmed3f(a, -fmax, fmax);
    float cb = __builtin_amdgcn_fmed3f(b, -fmax, fmax);
    uint32_t p;
    if (FMT == kE4M3) p = (uint32_t)__builtin_amdgcn_cvt_pk_fp8_f32(ca, cb, 0, false);
    else              p = (uint32_t)__builtin_amdgcn_cvt_pk_bf8_f32(ca, cb, 0, false);
    p &= 0xffffu;
    if (__builtin_expect(a != a, 0)) p = (p & 0xff00u) | 0x7fu | ((__float_as_uint(a) >> 24) & 0x80u);
    if (__builtin_expect(b != b, 0)) p = (p & 0x00ffu) | ((0x7fu | ((__float_as_uint(b) >> 24) & 0x80u)) << 8);
    return p;
}

template <int FMT>
__device__ __forceinline__ uint32_t satcast_pk4(float a, float b, float c, float d) {
    return satcast_pk2<FMT>(a, b) | (satcast_pk2<FMT>(c, d) << 16);
}

// Bit 23 of MODE (FP16_OVFL): from here on this wavefront's conversions to FP8 saturate by themselves.  So do those to bf16, which have
// to overflow to infinity: no wavefront rounds to bf16 in between.
template <int ON = 1> __device__ __forceinline__ void saturating_conversions() {
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_setreg(1 | 23 << 6, ON);
    __builtin_amdgcn_sched_barrier(0);
}
// The same for eight values, in a wavefront of saturating_conversions(), where the vector ALU counts: what is not finite becomes a
// code above the largest finite one (E4M3 0x7f, E5M2 0x7c to 0x7f, either sign), which nothing finite does; one test of the codes for all eight, and
// the per-element patch only when it fires.  The second conversion of a word writes its upper half in place; the first
// leaves there what was in the register of its own operand.
// (Every finite value of all 2^32 gets the code that the clamp gives it.  Q of 4096 x 11008 bf16 with the transposed copy: a test, a
// branch and a patch for each value 41.4 us; clamped, one NaN probe of a fused multiply-add per value 36.3; so 35.2.  One step
// at T = 1024, d = 4096, f = 11008 with delayed scaling, whose dH epilogue casts, 513 and 503 of the last two.)
template <int FMT>
__device__ __forceinline__ uint2 satcast_pk8(const float (&v)[8]) {
    uint32_t w[2], over = 0;
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        const float a = v[4 * h], b = v[4 * h + 1], c = v[4 * h + 2], d = v[4 * h + 3];
        int p = __float_as_int(a);
        p = FMT == kE4M3 ? __builtin_amdgcn_cvt_pk_fp8_f32(a, b, p, false) : __builtin_amdgcn_cvt_pk_bf8_f32(a, b, p, false);
        p = FMT == kE4M3 ? __builtin_amdgcn_cvt_pk_fp8_f32(c, d, p, true) : __builtin_amdgcn_cvt_pk_bf8_f32(c, d, p, true);
        w[h] = (uint32_t)p;
        over |= (w[h] & 0x7f7f7f7fu) + (FMT == kE4M3 ? 0x01010101u : 0x04040404u);
    }
    if (__builtin_expect((over & 0x80808080u) != 0u, 0))
        return make_uint2(satcast_pk4<FMT>(v[0], v[1], v[2], v[3]), satcast_pk4<FMT>(v[4], v[5], v[6], v[7]));
    return make_uint2(w[0], w[1]);
}

// SwiGLU neuron of Section 4.1 in fp32: u * Swish(g), Swish(g) = g * sigma(g).
// Every operation is a single rounded fp32 operation in a fixed order so that
// the GEMM epilogue and the stand-alone pass produce identical bits.
//
// sigma(g) = 1 / (1 + e^x) with x = -g, held between -1000 (e^x is 0 there) and 88: nothing overflows (the large-|g| regime is the
// one the method is about), and below g = -87.4 the reciprocal is no normal number any more and flushed to zero.
// e^x = 2^y e^d with y = x log2 e, rounded, and d = x - y ln 2, |d| < 2^-17, from two fused multiply-adds against a split constant:
// the hardware exp2 (1 ulp) sees an argument that is a float, and the error does not grow with |g|; the reciprocal is
// the hardware one (1 ulp).  Total error of u*g*sigma(g): < 6 ulp; measured on 4 M pairs, g normal of deviation 1 and 8, at
// most 3.0 ulp, .55 and .53 on average (e^-|g| with a choice by sign, and the remainder in units of log2: 3.6, .56 and .58).
// What bounds the epilogues and casts that form it is the vector ALU as much as memory (two transcendentals of 16 cycles a
// wavefront and 8 other instructions of 4; the other form had 11).
__device__ __forceinline__ float sigmoid_f32(float g) {
    constexpr float kLog2e = 1.44269502162933349609375f;
    constexpr float kLn2Hi = 0.693147182464599609375f;            // float(ln 2)
    constexpr float kLn2Lo = -1.904654299957768e-09f;             // ln 2 - kLn2Hi
    const float x = __builtin_amdgcn_fmed3f(-g, -1000.0f, 88.0f);
    const float y = __fmul_rn(x, kLog2e);
    const float d = __fmaf_rn(y, -kLn2Lo, __fmaf_rn(y, -kLn2Hi, x));
    const float e = __builtin_amdgcn_exp2f(y);
    return __builtin_amdgcn_rcpf(__fadd_rn(1.0f, __fmaf_rn(e, d, e)));
}
__device__ __forceinline__ float swiglu_f32(float u, float g) {
    float sw = __fmul_rn(g, sigmoid_f32(g));
    return __fmul_rn(u, sw);
}
// d h / d u = g*sigma(g);  d h / d g = u * sigma(g) * (1 + g * (1 - sigma(g)))
// The gradients are rounded to bf16 right away and compared with a GEMM-level tolerance, so the
// sigmoid here uses the hardware exp2 / reciprocal (about 2 ulp, plus |g| * 2^-24 from the scaled
// argument) instead of the correctly rounded sequence of the forward pass: ~4x fewer VALU
// instructions in an epilogue that is otherwise ALU bound.
__device__ __forceinline__ float sigmoid_fast_f32(float g) {
    // 1 / (1 + 2^(-g log2 e)); for g below about -88 the power overflows to +inf and the quotient is 0
    // where the true value is below the smallest normal number
    const float t = __builtin_amdgcn_exp2f(g * -1.44269504088896340736f);
    return __builtin_amdgcn_rcpf(1.0f + t);
}
__device__ __forceinline__ void swiglu_grad_f32(float u, float g, float dh, float &du, float &dg) {
    const float sg = sigmoid_fast_f32(g);
    const float sw = g * sg;
    du = dh * sw;
    dg = (dh * u) * __fmaf_rn(sw, 1.0f - sg, sg);
}

// |x| of a non-NaN float as an unsigned integer orders like the float; NaN -> 0.
__device__ __forceinline__ uint32_t abs_bits_ignore_nan(float v) {
    uint32_t u = __float_as_uint(v) & 0x7fffffffu;
    return u > 0x7f800000u ? 0u : u;
}

__device__ __forceinline__ uint32_t wave_max_u32(uint32_t v) {
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) {
        uint32_t o = (uint32_t)__shfl_xor((int)v, off, 64);
        v = v > o ? v : o;
    }
    return v;
}

}  // namespace ssg
