// Scalar numerics of the quantiser.  Each step is defined once for host and device in plain terms (integer
// arithmetic, correctly rounded division): the host-side test helpers run these.  The gfx950 kernels run forms of a
// few instructions with the same results, in front of each of which stands what it leaves out; a test compares the two on the
// GPU for every fp32 bit pattern and every width.
//
// The paper (Section "Quantization") fixes "16-bit shift and scaling factors" per
// group and uniform min-max quantisation; the concrete choices are:
// IEEE fp16, shift rounded toward -inf, scale toward +inf (so the stored range
// always covers [lo, hi] and no entry clips), saturation at +-65504, and the code
// decided by round-half-even((d - shift) * (1/scale)) in fp32.
#pragma once
#include <stdint.h>

#if defined(__HIPCC__)
#include <hip/hip_runtime.h>
#define KVTC_HD __host__ __device__ __forceinline__
#else
#define KVTC_HD inline
#endif

namespace kvtc {

KVTC_HD uint32_t f32_bits(float x) { return __builtin_bit_cast(uint32_t, x); }
KVTC_HD float bits_f32(uint32_t u) { return __builtin_bit_cast(float, u); }

// fp32 -> fp16 bit pattern with directed rounding, pure integer arithmetic.
// up = true: toward +inf, false: toward -inf.  Magnitudes above 65504 (and NaN)
// saturate to +-65504.
KVTC_HD uint16_t f16_round_dir(float x, bool up) {
    const uint32_t u = f32_bits(x);
    const uint32_t sign = u >> 31;
    uint32_t a = u & 0x7fffffffu;
    if (a > 0x477fe000u) a = 0x477fe000u;              // 65504.0f
    const uint32_t e = a >> 23;
    const uint32_t m = a & 0x7fffffu;
    uint32_t h, rem;
    if (e >= 113u) {                                     // fp16 normal
        h = ((e - 112u) << 10) | (m >> 13);
        rem = m & 0x1fffu;
    } else if (e >= 102u) {                              // fp16 subnormal
        const uint32_t mant = m | 0x800000u;
        const uint32_t sh = 126u - e;                    // 14 .. 24
        h = mant >> sh;
        rem = mant & ((1u << sh) - 1u);
    } else {                                             // below half the smallest subnormal
        h = 0u;
        rem = a;
    }
    const bool away = up ? (sign == 0u) : (sign != 0u);  // round the magnitude away from zero?
    if (rem != 0u && away) h += 1u;
    return (uint16_t)((sign << 15) | h);
}

KVTC_HD float f16_bits_to_f32(uint16_t hbits) {
    const uint32_t sign = (uint32_t)(hbits >> 15) << 31;
    const uint32_t e = (hbits >> 10) & 0x1fu;
    const uint32_t m = hbits & 0x3ffu;
    if (e == 0u) {                                       // zero / subnormal: m * 2^-24, exact in fp32
        const float v = (float)m * 5.9604644775390625e-08f;
        return bits_f32(f32_bits(v) | sign);
    }
    if (e == 31u) return bits_f32(sign | 0x7f800000u | (m << 13));
    return bits_f32(sign | ((e + 112u) << 23) | (m << 13));
}

#if defined(__HIPCC__)
// The device's forms of what stands above and below.
// fp32 -> fp16 with directed rounding: truncated towards zero, and one step away from it where that lost something on the side asked
// for (the value clamped first, so there is no step beyond 65504).  Not for NaN.  5 instructions for 20 and three branches.
__device__ __forceinline__ uint32_t f16_round_dir_dev(float x, bool up, float& back) {
    const float c = __builtin_amdgcn_fmed3f(x, -65504.0f, 65504.0f);
    uint32_t h = __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_pkrtz(c, 0.0f));
    const float t = (float)__builtin_bit_cast(_Float16, (uint16_t)h);
    h += (up ? t < c : t > c) ? 1u : 0u;
    back = (float)__builtin_bit_cast(_Float16, (uint16_t)h);
    return h;
}
// 1 / v to nearest, for the values that occur here: 2^b - 1 (b <= 16) and the positive fp16 numbers (one step of Newton's method on the
// hardware's estimate).
__device__ __forceinline__ float rcp_rn_dev(float v) {
    const float y = __builtin_amdgcn_rcpf(v);
    return __builtin_fmaf(__builtin_fmaf(-v, y, 1.0f), y, y);
}
#endif

struct GroupQ {
    uint16_t shift16, scale16;
    float shift, inv;        // fp32 values used for the code decision
};

KVTC_HD float div_rn(float a, float b) {
#if defined(__HIP_DEVICE_COMPILE__)
    return __fdiv_rn(a, b);
#else
    return a / b;
#endif
}

// Header of one (token, group) from the group's fp32 min and max.
KVTC_HD GroupQ group_header_plain(float lo, float hi, int bits) {
    GroupQ g;
    g.shift16 = f16_round_dir(lo, false);
    g.shift = f16_bits_to_f32(g.shift16);
    const float qmax = (float)((1u << bits) - 1u);
    const float range = hi - g.shift;                    // one fp32 subtraction
    g.scale16 = f16_round_dir(div_rn(range, qmax), true);
    const float sc = f16_bits_to_f32(g.scale16);
    g.inv = sc > 0.0f ? div_rn(1.0f, sc) : 0.0f;
    return g;
}

// The same as the kernels work it out, but for a range of -0, whose scale has no sign here; no group has one (its minimum would have to be +0 and its
// maximum -0).
KVTC_HD GroupQ group_header(float lo, float hi, int bits) {
#if defined(__HIP_DEVICE_COMPILE__)
    GroupQ g;
    // (range / qmax to nearest: quotient by the reciprocal, corrected by its exact remainder.  From 1e10 on a scale has long reached 65504,
    // and the remainder of infinity would not be a number.)
    g.shift16 = (uint16_t)f16_round_dir_dev(lo, false, g.shift);
    const float top = (float)((1u << bits) - 1u), rtop = rcp_rn_dev(top);
    const float span = __builtin_amdgcn_fmed3f(__fsub_rn(hi, g.shift), -1e10f, 1e10f);
    const float q0 = __fmul_rn(span, rtop);
    float sc;
    g.scale16 = (uint16_t)f16_round_dir_dev(__builtin_fmaf(__builtin_fmaf(-q0, top, span), rtop, q0), true, sc);
    g.inv = sc > 0.0f ? rcp_rn_dev(sc) : 0.0f;
    return g;
#else
    return group_header_plain(lo, hi, bits);
#endif
}

// The code of one coefficient from its group's decoded header: two fp32 operations (subtract the
// shift, multiply by the rounded reciprocal of the scale), round half to even, clamp to
// [0, qmax = 2^bits - 1].  inv == 0 (zero scale) gives 0.
KVTC_HD float code_of(float d, float shift, float inv, float qmax) {
#if defined(__HIP_DEVICE_COMPILE__)
    const float q = __fmul_rn(__fsub_rn(d, shift), inv);
    return __builtin_amdgcn_fmed3f(__builtin_rintf(q), 0.0f, qmax);
#else
    volatile float t = d - shift;            // kept apart: the host compiler must not fuse them
    volatile float q = t * inv;
    float rq = __builtin_nearbyintf(q);
    if (!(rq >= 0.0f)) rq = 0.0f;
    if (rq > qmax) rq = qmax;
    return rq;
#endif
}

#if defined(__HIPCC__)
// The code of a coefficient as the low bits of a float: with the reciprocal scaled by 2^-bits, (d - shift) / scale lies in [0, 1), and adding
// 2^(23 - bits), whose last place is 2^-bits, rounds it to nearest even exactly as code_of rounds (a power of two moves no rounding).  The clamp of
// the multiplication does the rest of code_of: below zero and not a number give 0.  Above the largest code is nothing unless the scale is saturated (such tiles
// take another way): a scale rounded up covers the group's range.  Four instructions with the one that packs it, where
// round, clamp and convert to an integer made six.
__device__ __forceinline__ uint32_t code_float(float d, float shift, float inv_b, float base) {
    const float t = __builtin_amdgcn_fmed3f(__fmul_rn(__fsub_rn(d, shift), inv_b), 0.0f, 1.0f);
    return __float_as_uint(__fadd_rn(t, base));
}
__host__ __device__ constexpr uint32_t code_base_bits(uint32_t bits) { return (150u - bits) << 23; }      // 2^(23 - bits)
#endif

}  // namespace kvtc
