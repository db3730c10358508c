// Rotary positional embedding of keys, undone before they are coded and redone after they are
// decoded, for gfx950.  (Paper, Section "Feature decorrelation": the positional rotation hides the
// low-rank structure of keys, so it is removed before the transform and compression works on keys
// as they were before the rotation; decoded keys are rotated again before attention reads them.)
//
// The rotation is RoFormer's: inside every head, features are paired, and the pair (a, b) of the
// token at position m is turned by m * theta_j, theta_j = base^(-2j / d_head):
//     a' = a cos - b sin,  b' = a sin + b cos        (undoing it: the opposite angle).
// Pair j is (j, j + d_head/2) ("half", the rotate-half form) or (2j, 2j+1) ("interleaved").
//
// Streaming kernels, in place: 2 x element size bytes of traffic per value.  Angles, sines,
// cosines, products and sums are all double precision -- an angle reaches 10^5 radians, where a
// float has lost the sine -- and the result is rounded once to the tensor's type, so it equals a
// float64 reference rounded the same way.  A lane owns one pair index of its token in every head:
// one sincos serves all heads, and neighbouring lanes touch neighbouring elements (bf16 in whole pieces of 16 bytes: eight pair indices to a lane).  The
// frequencies theta_j are computed on the host and travel as kernel arguments.
#include <hip/hip_runtime.h>
#include "kvtc_dev.h"

namespace kvtc {

constexpr int kRopeHeads = 2;           // whose pieces a lane of the wide kernel has on their way
constexpr int kRopeMaxHalf = 128;      // d_head / 2 at most (the frequency table is a kernel argument)

struct RopeArgs {
    void* x;
    int64_t n_tokens, token_stride, head_stride;     // strides in elements
    const int32_t* positions;                        // device, [n_tokens], or nullptr: position0 + token
    int64_t position0;
    int32_t n_heads, d_head, inverse;
    double theta[kRopeMaxHalf];                      // [d_head / 2]
};

__device__ __forceinline__ double load_val(const uint16_t* p) { return (double)__uint_as_float((uint32_t)*p << 16); }
__device__ __forceinline__ double load_val(const float* p) { return (double)*p; }
__device__ __forceinline__ void store_val(uint16_t* p, double v) {
    // double -> float -> bf16, both to nearest even (the float step can move a result only if it lies within 2^-29
    // relative of a bf16 rounding boundary)
    const uint32_t u = __float_as_uint((float)v);
    if ((u & 0x7fffffffu) > 0x7f800000u) { *p = (uint16_t)((u >> 16) | 0x40u); return; }      // NaN stays NaN
    *p = (uint16_t)((u + 0x7fffu + ((u >> 16) & 1u)) >> 16);
}
__device__ __forceinline__ void store_val(float* p, double v) { *p = (float)v; }
// the same by the conversion instruction (the compiler must not make one rounding of the two)
__device__ __forceinline__ void round_val(uint16_t* p, double v) {
    float f = (float)v;
    asm("" : "+v"(f));
    *p = __builtin_bit_cast(uint16_t, (__bf16)f);
}

// INTERLEAVED = 0: pair j = (j, j + half); 1: pair j = (2j, 2j + 1)
template <typename T, int INTERLEAVED>
__global__ void __launch_bounds__(256) rope_kernel(const RopeArgs a) {
    const int half = a.d_head / 2;
    const int64_t n_items = a.n_tokens * (int64_t)half;          // one item = one (token, pair index)
    T* x = static_cast<T*>(a.x);
    for (int64_t item = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; item < n_items; item += (int64_t)gridDim.x * blockDim.x) {
        const int64_t t = item / half;
        const int j = (int)(item - t * half);
        const int64_t pos = a.positions ? (int64_t)a.positions[t] : a.position0 + t;
        double s, c;
        sincos((double)pos * a.theta[j], &s, &c);
        if (a.inverse) s = -s;
        T* row = x + t * a.token_stride;
        const int ia = INTERLEAVED ? 2 * j : j, ib = INTERLEAVED ? 2 * j + 1 : j + half;
        for (int h = 0; h < a.n_heads; ++h) {
            T* head = row + (int64_t)h * a.head_stride;
            const double va = load_val(head + ia), vb = load_val(head + ib);
            store_val(head + ia, __dsub_rn(__dmul_rn(va, c), __dmul_rn(vb, s)));
            store_val(head + ib, __dadd_rn(__dmul_rn(va, s), __dmul_rn(vb, c)));
        }
    }
}

// sin and cos of an angle of at most 2^31: what is left of it beyond the nearest multiple of pi/2 -- taken off in three parts with fused operations (Cody and Waite's
// reduction), to 2^-53 -- by the series about 0, to its 17th and 16th power.  (At pi/4 the next terms are r^19 / 19! = 2^-63.4 and r^18 / 18! = 2^-58.8, below half a last place.)
__device__ __forceinline__ void sincos_reduced(double angle, double* s, double* c) {
    const double n = __builtin_rint(angle * 0.63661977236758134308);                 // 2 / pi
    double r = __builtin_fma(n, -1.5707963267948966, angle);
    r = __builtin_fma(n, -6.123233995736766e-17, r);
    r = __builtin_fma(n, 1.4973849048591833e-33, r);
    const double q = r * r;
    double u = 1.0 / 355687428096000.0, v = 1.0 / 20922789888000.0;                  // 17!, 16!
    u = __builtin_fma(u, q, -1.0 / 1307674368000.0);
    v = __builtin_fma(v, q, -1.0 / 87178291200.0);
    u = __builtin_fma(u, q, 1.0 / 6227020800.0);
    v = __builtin_fma(v, q, 1.0 / 479001600.0);
    u = __builtin_fma(u, q, -1.0 / 39916800.0);
    v = __builtin_fma(v, q, -1.0 / 3628800.0);
    u = __builtin_fma(u, q, 1.0 / 362880.0);
    v = __builtin_fma(v, q, 1.0 / 40320.0);
    u = __builtin_fma(u, q, -1.0 / 5040.0);
    v = __builtin_fma(v, q, -1.0 / 720.0);
    u = __builtin_fma(u, q, 1.0 / 120.0);
    v = __builtin_fma(v, q, 1.0 / 24.0);
    u = __builtin_fma(u, q, -1.0 / 6.0);
    v = __builtin_fma(v, q, -0.5);
    u = __builtin_fma(u * q, r, r);
    v = __builtin_fma(v, q, 1.0);
    const uint32_t k = (uint32_t)(int32_t)n;
    const double a = k & 1u ? v : u, b = k & 1u ? u : v;
    *s = k & 2u ? -a : a;
    *c = (k + 1u) & 2u ? -b : b;
}

// The same for bf16, 16 bytes at a time: a lane owns eight neighbouring pairs of a token in every `shares`-th of `heads_each` heads, so that a wave moves whole lines, and the pieces
// of two heads are on their way while those before are turned.  A product is fused into the sum: one rounding fewer than above.  Bound by the caches' rate: 32768
// tokens of 8 heads of 128 features, 64 MB, in place 21 us (29 by the kernel above, which takes a library's sine and cosine and about 30 instructions to a pair in
// 2-byte accesses; a copy of the same bytes 20), 4000 tokens 5.1 (6.1), 300000 229 (325).
// With four heads on their way at a time 22.  fp32 tensors stay with the kernel above, whose 4-byte accesses are as fast: 32768 tokens 40 us, in 16-byte pieces 41 to 48.
template <int INTERLEAVED>
__global__ void __launch_bounds__(256) rope_wide_kernel(const RopeArgs a, uint32_t lanes, uint32_t shares, int heads_each) {
    typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
    union Piece { u32x4 v; uint16_t e[8]; };
    const uint32_t item = blockIdx.x * 256u + threadIdx.x, unit = item / lanes, g = item - unit * lanes, t = unit / shares;
    if (t >= a.n_tokens) return;
    const int half = a.d_head / 2, j0 = (int)g * 8, second = INTERLEAVED ? 8 : half, step = (int)shares;
    const int h0 = (int)(blockIdx.y * (uint32_t)heads_each + (unit - t * shares)), h1 = min((int)blockIdx.y * heads_each + heads_each, a.n_heads);
    const int64_t stride = step * a.head_stride;
    uint16_t* from = static_cast<uint16_t*>(a.x) + (int64_t)t * a.token_stride + (int64_t)h0 * a.head_stride + (INTERLEAVED ? 2 * j0 : j0);
    Piece p[kRopeHeads], q[kRopeHeads];
    auto load = [&](int h) {
#pragma unroll
        for (int k = 0; k < kRopeHeads; ++k)
            if (h + k * step < h1) {
                p[k].v = *reinterpret_cast<const u32x4*>(from + k * stride);
                q[k].v = *reinterpret_cast<const u32x4*>(from + k * stride + second);
            }
    };
    load(h0);                                                       // (the first heads travel under the sines and cosines)
    const double pos = (double)(a.positions ? (int64_t)a.positions[t] : a.position0 + t);
    double s[8], c[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        sincos_reduced(pos * a.theta[j0 + i], &s[i], &c[i]);
        if (a.inverse) s[i] = -s[i];
    }
    for (int h = h0; h < h1; h += kRopeHeads * step) {
#pragma unroll
        for (int k = 0; k < kRopeHeads; ++k)
            if (h + k * step < h1) {
#pragma unroll
                for (int i = 0; i < 8; ++i) {
                    uint16_t& ea = INTERLEAVED ? (i < 4 ? p[k].e[2 * i % 8] : q[k].e[2 * i % 8]) : p[k].e[i];
                    uint16_t& eb = INTERLEAVED ? (i < 4 ? p[k].e[2 * i % 8 + 1] : q[k].e[2 * i % 8 + 1]) : q[k].e[i];
                    const double va = load_val(&ea), vb = load_val(&eb);
                    round_val(&ea, __builtin_fma(va, c[i], -(vb * s[i])));
                    round_val(&eb, __builtin_fma(va, s[i], vb * c[i]));
                }
                *reinterpret_cast<u32x4*>(from + k * stride) = p[k].v;
                *reinterpret_cast<u32x4*>(from + k * stride + second) = q[k].v;
            }
        from += kRopeHeads * stride;
        load(h + kRopeHeads * step);
    }
}

// Whole pieces where a bf16 tensor allows them -- pairs, strides and address in multiples of 16 bytes, angles that sincos_reduced takes -- and where it gains: a lane works out eight
// sines and cosines before it begins, half a microsecond, which few heads and few tokens do not give back.  (us, above and so, tokens of 128 features: one head, 1 2.1 and 2.6,
// 2000 2.7 2.9, 4000 3.3 3.0; two, 1000 2.7 2.9, 2000 3.1 3.0; three, 4 2.5 2.6, 16 2.7 2.7; five, 1 2.5 2.6, 4 2.9 2.7; eight, 1 3.3 2.9.)  Nor in token-major tensors of heads of
// less than a cache line, where a wave's lanes are at as many lines: many heads, or heads of 16 features, beyond 16384 tokens (16 heads of 32, 33000 tokens 17.5 and 18.2, of 16, 70000, 20.3 and 27.5).
bool rope_wide(const RopeArgs& a) {
    double most = 1.0;
    for (int j = 0; j < a.d_head / 2; ++j) most = a.theta[j] > most ? a.theta[j] : most;
    const double first = (double)a.position0, last = first + (double)a.n_tokens;
    const double far = a.positions ? 0x1p31 : (first < 0.0 && -first > last ? -first : last);
    // items of eight pairs, at least
    const int64_t items = a.n_tokens * (a.d_head / 16), least = a.n_heads == 1 ? 20000 : a.n_heads == 2 ? 14000 : a.n_heads == 3 ? 128 : a.n_heads < 6 ? 32 : 0;
    const bool narrow = a.head_stride < a.token_stride && a.n_tokens > 16384 && (a.d_head < 64 ? a.n_heads >= 16 || (a.d_head == 16 && a.n_heads > 1) : false);
    return items >= least && !narrow && a.d_head % 16 == 0 && a.token_stride % 8 == 0 && a.head_stride % 8 == 0 && reinterpret_cast<uintptr_t>(a.x) % 16 == 0 &&
           far * most <= 0x1p31 && a.n_tokens * (a.d_head / 16) <= 0x3fffffffLL / a.n_heads;
}
// Heads are shared out only where there is not one workgroup for every compute unit, or, of token-major tensors, where a token's row is long: the sines and cosines are worked out again
// for each share.  Within a row the shares are neighbouring lanes, so that a wave is at whole lines of a row and a row's lines belong to one workgroup; head-major, they are
// workgroups.  (Token-major, a workgroup to a share of heads in turn, neighbouring lanes: 8 heads of 32 features, 8000 tokens 6.0 and 4.3 us, 16 of 128, 8000, 15.9 and 11.0, 32 of 128, 4000, 15.9 and
// 11.0; at least 512 features to a step also for short rows: 8 heads of 64, 33000 tokens, 12.2 and 20.)
hipError_t launch_rope_wide(const RopeArgs& a, int interleaved, hipStream_t stream) {
    const uint32_t lanes = (uint32_t)a.d_head / 16u, heads = (uint32_t)a.n_heads;
    auto grid_of = [&](uint32_t shares) { return (uint32_t)((a.n_tokens * lanes * shares + 255) / 256); };
    const bool long_rows = a.n_heads * (int64_t)a.d_head >= 2048;
    uint32_t shares = 1, heads_grid = 1;
    int heads_each = a.n_heads;
    if (a.head_stride < a.token_stride) {
        while (shares < heads && (grid_of(shares) < (uint32_t)compute_units() || (long_rows && shares * (uint32_t)a.d_head < 512u))) shares = shares * 2 < heads ? shares * 2 : heads;
    } else {
        while (heads_each > 1 && (int64_t)grid_of(1) * ((a.n_heads + heads_each - 1) / heads_each) < compute_units()) heads_each = (heads_each + 1) / 2;
        heads_grid = (uint32_t)((a.n_heads + heads_each - 1) / heads_each);
    }
    if (heads_grid > 65535u) return hipErrorInvalidValue;
    if (interleaved) hipLaunchKernelGGL((rope_wide_kernel<1>), dim3(grid_of(shares), heads_grid), dim3(256), 0, stream, a, lanes, shares, heads_each);
    else hipLaunchKernelGGL((rope_wide_kernel<0>), dim3(grid_of(shares), heads_grid), dim3(256), 0, stream, a, lanes, shares, heads_each);
    return hipGetLastError();
}

hipError_t launch_rope(const RopeArgs& a, kvtc_dtype dtype, int interleaved, int grid, hipStream_t stream) {
    if (dtype == KVTC_BF16 && rope_wide(a)) return launch_rope_wide(a, interleaved, stream);
    if (dtype == KVTC_BF16) {
        if (interleaved) hipLaunchKernelGGL((rope_kernel<uint16_t, 1>), dim3(grid), dim3(256), 0, stream, a);
        else hipLaunchKernelGGL((rope_kernel<uint16_t, 0>), dim3(grid), dim3(256), 0, stream, a);
    } else {
        if (interleaved) hipLaunchKernelGGL((rope_kernel<float, 1>), dim3(grid), dim3(256), 0, stream, a);
        else hipLaunchKernelGGL((rope_kernel<float, 0>), dim3(grid), dim3(256), 0, stream, a);
    }
    return hipGetLastError();
}

}  // namespace kvtc
