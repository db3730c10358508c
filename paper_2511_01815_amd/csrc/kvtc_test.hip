// Kernels that only tests launch: the quantiser's device forms against the plain ones, value by value.
#include <hip/hip_runtime.h>
#include "kvtc_numeric.h"
#include "../../include/kvtc_test_hooks.h"

namespace kvtc {
kvtc_status set_error(kvtc_status st, const char* fmt, ...);

__device__ __forceinline__ bool same_header(const GroupQ& a, const GroupQ& b) {
    return a.shift16 == b.shift16 && a.scale16 == b.scale16 && f32_bits(a.shift) == f32_bits(b.shift) && f32_bits(a.inv) == f32_bits(b.inv);
}

// Every 32-bit pattern as a float v (but NaN): its two roundings to fp16; the header of a range from 0 to v (but -0); the header of the group
// between v and a value made of a mixture of v's bits; and, of up to 8 bits, the codes of three values of that group.  counts[0] counts
// the values, [1..3] what is not the same: roundings, headers, codes.
__global__ void __launch_bounds__(256) numeric_kernel(int bits, unsigned long long* counts) {
    const uint32_t step = gridDim.x * blockDim.x;
    uint32_t values = 0, rounding = 0, header = 0, code = 0;
    for (uint64_t n = blockIdx.x * blockDim.x + threadIdx.x; n < (1ull << 32); n += step) {
        const uint32_t u = (uint32_t)n;
        const float v = bits_f32(u);
        if (v != v) continue;
        ++values;
#pragma unroll
        for (int up = 0; up < 2; ++up) {
            float back;
            const uint16_t h = f16_round_dir(v, up != 0);
            if ((uint16_t)f16_round_dir_dev(v, up != 0, back) != h || f32_bits(back) != f32_bits(f16_bits_to_f32(h))) ++rounding;
        }
        if (u != 0x80000000u && !same_header(group_header(0.0f, v, bits), group_header_plain(0.0f, v, bits))) ++header;
        uint32_t m = (u ^ (u >> 15)) * 0x2c1b3c6du;
        m = (m ^ (m >> 12)) * 0x297a2d39u;
        // another value of about the same size, of any size, or v's neighbour: by two bits of the mixture
        const uint32_t w_bits = (m & 3u) == 0u ? m : (m & 3u) == 1u ? u + 1u : (u & 0xff800000u) ^ (m & 0x81ffffffu);
        const float w = bits_f32(w_bits);
        if (w != w || v == 0.0f || w == 0.0f) continue;
        const float lo = fminf(v, w), hi = fmaxf(v, w);
        const GroupQ g = group_header(lo, hi, bits);
        if (!same_header(g, group_header_plain(lo, hi, bits))) ++header;
        if (bits <= 8 && g.scale16 != 0x7bffu) {
            const float qmax = (float)((1u << bits) - 1u), base = bits_f32(code_base_bits(bits));
            const float inside = fminf(fmaxf(lo + (hi - lo) * ((float)(m >> 8) * 0x1p-24f), lo), hi);
#pragma unroll
            for (int k = 0; k < 3; ++k) {
                const float d = k == 0 ? lo : k == 1 ? hi : inside;
                if (code_float(d, g.shift, __builtin_ldexpf(g.inv, -bits), base) - code_base_bits(bits) != (uint32_t)code_of(d, g.shift, g.inv, qmax)) ++code;
            }
        }
    }
    atomicAdd(&counts[0], (unsigned long long)values);
    if (rounding) atomicAdd(&counts[1], (unsigned long long)rounding);
    if (header) atomicAdd(&counts[2], (unsigned long long)header);
    if (code) atomicAdd(&counts[3], (unsigned long long)code);
}
}  // namespace kvtc

extern "C" kvtc_status kvtc_test_numeric(int bits, uint64_t* counts_dev, kvtc_stream stream) {
    using namespace kvtc;
    if (bits < 1 || bits > 16 || !counts_dev) return set_error(KVTC_E_ARG, "kvtc_test_numeric: bad argument");
    hipLaunchKernelGGL(numeric_kernel, dim3(256 * 16), dim3(256), 0, static_cast<hipStream_t>(stream), bits, reinterpret_cast<unsigned long long*>(counts_dev));
    const hipError_t e = hipGetLastError();
    return e == hipSuccess ? KVTC_OK : set_error(KVTC_E_HIP, "kvtc_test_numeric: launch failed: %s", hipGetErrorString(e));
}
