// Calibration on the GPU, the data-heavy part of the bit allocation (declared in include/kvtc.h,
// "Calibration"): the table of block errors that the dynamic programme reads.  (Paper, Section
// "Quantization" and appendix "Dynamic programming algorithm": for every candidate block of subsequent
// PCA coordinates and every quantiser type, the block of calibration coefficients is quantised as the
// coder would quantise it, and the squared error is compared with dropping the block.)
//
// A workgroup owns a candidate block at one width or at two neighbouring ones, a long block's tokens by halves, so every sum has a
// fixed order and the table is reproducible.  Four lanes or more own a token: its coefficients sit in registers, min and max come
// from lane exchanges, and the errors use the coder's own scalar numerics (fp16 shift rounded down,
// scale rounded up, code by subtract, multiply by the rounded reciprocal, round to even, clamp),
// accumulated in double from exactly representable terms.
//
// Also here: the first and second moments of the calibration tokens (sum of x and sum of x x^T, in
// double), the one pass over the calibration data that the PCA needs (paper, Section "Feature
// decorrelation", eq. 2: mean and SVD of the centred matrix; its right singular vectors are the
// eigenvectors of the centred second-moment matrix, which the caller forms and decomposes on the host).
#include <hip/hip_runtime.h>
#include <type_traits>

#include "kvtc_dev.h"
#include "kvtc_numeric.h"

namespace kvtc {
kvtc_status set_error(kvtc_status st, const char* fmt, ...);
}
using namespace kvtc;

namespace {

constexpr int kCalibMaxBits = 8;
constexpr int kCalibMaxN = 1024;
constexpr int kCalibThreads = 1024;   // 16 waves: the pair with the longest block is the tail of the launch
constexpr int kCalibMaxBlocks = 1 << 21;          // blocks per launch
constexpr int kCalibTok = 4;          // tokens a lane group works on at once

// Minimum or maximum over groups of L lanes (4, 16 or 64), in every lane: register exchanges inside a row of 16
// lanes (quads, then the mirrored half row, then the mirrored row: each partner holds the other half's result),
// lane swaps through the LDS crossbar beyond.
template <int CTRL> __device__ __forceinline__ float dpp_f32(float v) {
    return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), CTRL, 0xf, 0xf, true));
}
template <int L, typename F> __device__ __forceinline__ float group_reduce(float v, F f) {
    v = f(v, dpp_f32<0xB1>(v));          // quad_perm [1,0,3,2]
    v = f(v, dpp_f32<0x4E>(v));          // quad_perm [2,3,0,1]
    if constexpr (L >= 16) {
        v = f(v, dpp_f32<0x141>(v));     // row_half_mirror
        v = f(v, dpp_f32<0x140>(v));     // row_mirror
    }
    if constexpr (L == 64) {
        v = f(v, __shfl_xor(v, 16, 64));
        v = f(v, __shfl_xor(v, 32, 64));
    }
    return v;
}

// min and max of a lane's next two values.  (The instructions themselves: of a value that comes from memory the compiler first makes a quiet NaN if it is
// a signalling one, an instruction per value that changes nothing here -- either makes the block's error not a number.)
__device__ __forceinline__ void min_max_of(float a, float b, float& lo, float& hi) {
    asm("v_min3_f32 %0, %1, %2, %0" : "+v"(lo) : "v"(a), "v"(b));
    asm("v_max3_f32 %0, %1, %2, %0" : "+v"(hi) : "v"(a), "v"(b));
}

// This thread's part of sum (d - d_hat)^2 - d^2 = d_hat (d_hat - 2 d) over its tokens, at W widths from `bits` on.  L lanes own a
// token, PER coordinates each (n <= L * PER; FULL: n == L * PER).  kCalibTok tokens at a time, so that the header --
// 40 instructions, as many as eight codes -- is worked out once per token and width by one lane of four and handed round, and not by all
// lanes that share the token.
// d_hat = shift + code * scale is exact in double: all its terms are multiples of 2^-24 below 2^26.
// The code is rounded by adding 2^23 (to nearest even, as code_of does it: the sum's last place is 1), clamped there, and its bits are the low
// half of the double 2^52 + 0x4b000000 + code: a subtraction in place of a conversion, which takes twice as long.
template <int L, int PER, bool FULL, int W>
__device__ __forceinline__ void block_error(const float* coef, int64_t t_begin, int64_t n_tokens, int64_t ld, int start, int n, int bits, double (&e)[W]) {
#pragma clang fp contract(off)               // (a product is rounded before the 2^23 is added)
    constexpr int GRP = kCalibThreads / L, STEP = GRP * kCalibTok;
    constexpr float kMagic = 8388608.0f;
    const double kMagicD = __builtin_bit_cast(double, 0x433000004b000000ull);
    const int tid = threadIdx.x, grp = tid / L, gl = tid % L, lane = tid & 63, mine = lane & 3;
    float top[W];
#pragma unroll
    for (int w = 0; w < W; ++w) top[w] = kMagic + (float)((1u << (bits + w)) - 1u);
    auto coord = [&](int k) { return (k >> 2) * 4 * L + 4 * gl + (k & 3); };         // four neighbours at a time: 16-byte loads
#pragma unroll
    for (int w = 0; w < W; ++w) e[w] = 0.0;
    for (int64_t s0 = t_begin; s0 < n_tokens; s0 += STEP) {          // every lane runs the same trips
        const int64_t t0 = s0 + grp * kCalibTok;
        float d[kCalibTok][PER];
        float lo = 0.0f, hi = 0.0f;
#pragma unroll
        for (int s = 0; s < kCalibTok; ++s) {
            const float* row = coef + (t0 + s < n_tokens ? t0 + s : n_tokens - 1) * ld + start;
            float l = __builtin_inff(), h = -__builtin_inff();
#pragma unroll
            for (int k = 0; k < PER; ++k) d[s][k] = FULL || coord(k) < n ? row[coord(k)] : 0.0f;
#pragma unroll
            for (int k = 0; k < PER; k += 2) {
                if (FULL) {
                    min_max_of(d[s][k], d[s][k + 1], l, h);
                } else {
                    const bool in0 = coord(k) < n, in1 = coord(k + 1) < n;
                    min_max_of(in0 ? d[s][k] : __builtin_nanf(""), in1 ? d[s][k + 1] : __builtin_nanf(""), l, h);      // (passed over)
                }
            }
            l = group_reduce<L>(l, [](float a, float b) { return fminf(a, b); });
            h = group_reduce<L>(h, [](float a, float b) { return fmaxf(a, b); });
            if (mine == s) { lo = l; hi = h; }
        }
        // a token behind the last one counts nothing: without shift and scale its d_hat is zero
        const bool counts = t0 + mine < n_tokens;
        GroupQ q[W];
#pragma unroll
        for (int w = 0; w < W; ++w) {
            q[w] = group_header(lo, hi, bits + w);
            q[w].shift = counts ? q[w].shift : 0.0f;
            q[w].scale16 = counts ? q[w].scale16 : (uint16_t)0;
            // an infinite coefficient makes error and energy infinite and their difference not a number, where the form above would
            // give -inf, the best value a minimising allocation can see (the subtraction in double: a finite range stays finite)
            e[w] = __builtin_fma((double)hi - (double)lo, 0.0, e[w]);
        }
#pragma unroll
        for (int s = 0; s < kCalibTok; ++s) {
            const int from = (lane & ~3) | s;
            const float shift = __shfl(q[0].shift, from, 64);
            const double sh = (double)shift;
            float inv[W];
            double sc[W];
#pragma unroll
            for (int w = 0; w < W; ++w) {
                inv[w] = __shfl(q[w].inv, from, 64);
                sc[w] = (double)f16_bits_to_f32((uint16_t)__shfl((int)q[w].scale16, from, 64));
            }
#pragma unroll
            for (int k = 0; k < PER; ++k) {
                const double dd = (double)d[s][k];
                const float over = __fsub_rn(d[s][k], shift);
                const bool in = FULL || coord(k) < n;
#pragma unroll
                for (int w = 0; w < W; ++w) {
                    const float q_f = over * inv[w], m = __builtin_amdgcn_fmed3f(q_f + kMagic, kMagic, top[w]);
                    const double code = __builtin_bit_cast(double, 0x4330000000000000ull | f32_bits(m)) - kMagicD;
                    const double dh = __builtin_fma(code, sc[w], sh);
                    e[w] = __builtin_fma(in ? dh : 0.0, __builtin_fma(-2.0, dd, dh), e[w]);
                }
            }
        }
    }
}

// Grid in z: parts 0 to 2 W - 1 are the halves of the halved blocks, ahead of everything else -- a block of more than 256 coordinates has a workgroup
// per half and width, or its workgroups would be the tail of the launch --, the last part all others (the only part where nothing is halved).
// (A part more costs a microsecond for 400 workgroups that find nothing to do.)
template <int W> constexpr int kCalibParts = 2 * W + 1;
// Blocks of more than 64 coordinates are cut in two halves of the tokens, whose sums are ADDED to the zeroed result: with
// two terms on top of zero the order of arrival cannot show, so the table stays reproducible.  Not where all tokens fit one step of
// such a block's lane groups: a half would take as long as the whole, and the launch that zeroes would be a quarter of the call
// (one block of 16 coordinates, 50 tokens, one width: 10.7 us with it, 8.5 without).
constexpr int kCalibHalveAbove = kCalibThreads / 64 * kCalibTok;
__device__ __forceinline__ bool calib_halved(const kvtc_calib_block& b, int64_t n_tokens) {
    return b.n > 64 && n_tokens > (b.n > 256 ? kCalibHalveAbove : kCalibThreads / 16 * kCalibTok);
}
__device__ __forceinline__ bool calib_bad_block(const kvtc_calib_block& b, int64_t ld) {
    return b.n < 1 || b.n > kCalibMaxN || b.start < 0 || (int64_t)b.start + b.n > ld;
}

__global__ void __launch_bounds__(256) calib_zero_kernel(double* change, int64_t n) {
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)gridDim.x * 256) change[i] = 0.0;
}

// block_error of a block of at most 256 coordinates
template <int W>
__device__ __forceinline__ void short_block_error(const float* coef, int64_t b, int64_t m, int64_t ld, int start, int n, int bits, double (&e)[W]) {
    if (n <= 16) {
        if (n == 16) block_error<4, 4, true>(coef, b, m, ld, start, n, bits, e); else block_error<4, 4, false>(coef, b, m, ld, start, n, bits, e);
    } else if (n <= 64) {
        if (n == 64) block_error<4, 16, true>(coef, b, m, ld, start, n, bits, e); else block_error<4, 16, false>(coef, b, m, ld, start, n, bits, e);
    } else {
        if (n == 256) block_error<16, 16, true>(coef, b, m, ld, start, n, bits, e); else block_error<16, 16, false>(coef, b, m, ld, start, n, bits, e);
    }
}

// change[block][b - 1] = sum over tokens and the block's coordinates of (d - d_hat)^2 - d^2.  Grid: (block, W widths, part).
// What bounds it is vector arithmetic (per coefficient: six fp32 instructions and one in fp64 for both widths, four and four for each).
// 175 blocks x 8 widths x 2048 tokens (the default set at 1024 features): 4.59 ms with
// a workgroup of 256 threads per block that evaluated all widths and 16 or 64 lanes per token, 0.386 ms with one of 1024
// threads per block and width (half of it for the headers), 0.206 ms with 16 coordinates per lane, 0.165 ms with two widths to a workgroup, which
// share the loads, the minima and maxima and the conversions, and without conversions of the codes (126 blocks at 768 features: 147 -> 97 us), 0.155 ms with fewer instructions to a header.
template <int W>
__global__ void __launch_bounds__(kCalibThreads) calib_block_errors_kernel(const float* coef, int64_t n_tokens, int64_t ld, const kvtc_calib_block* blocks,
                                                                          int max_bits, double* change) {
    __shared__ double red[W][kCalibThreads];
    const kvtc_calib_block blk = blocks[blockIdx.x];
    const int start = blk.start, n = blk.n, bits = W * (int)blockIdx.y + 1, part = gridDim.z == 1 ? kCalibParts<W> - 1 : (int)blockIdx.z;
    double* out = change + (size_t)blockIdx.x * max_bits + bits - 1;
    const int n_out = min(W, max_bits - (bits - 1));      // (an odd number of widths: the last workgroup has one)
    // the list lives on the device, out of the host's sight: a block outside a row (or longer than a lane group holds) gets NaN
    if (calib_bad_block(blk, ld)) {
        if ((int)threadIdx.x < n_out && part == kCalibParts<W> - 1) out[threadIdx.x] = __builtin_nan("");
        return;
    }
    const bool halved = gridDim.z != 1 && calib_halved(blk, n_tokens), alone = halved && n > 256;          // alone: one width
    if (halved != (part < kCalibParts<W> - 1) || (part >= 2 && halved && !alone)) return;
    const int w0 = alone ? part / 2 : 0, w1 = alone ? w0 + 1 : n_out;      // the widths this workgroup stores
    if (w0 >= n_out) return;
    const int64_t half = halved ? (n_tokens + 1) / 2 : n_tokens, b = halved && part % 2 ? half : 0, m = halved && part % 2 ? n_tokens : half;
    static_assert(W == 1 || W == 2, "the widths of a long block");
    double e[W];
#pragma unroll
    for (int w = 0; w < W; ++w) e[w] = 0.0;
    if (n > 256) {
        for (int w = w0; w < w1; ++w) {
            double one[1];
            if (n == 1024) block_error<64, 16, true>(coef, b, m, ld, start, n, bits + w, one); else block_error<64, 16, false>(coef, b, m, ld, start, n, bits + w, one);
            (w == 0 ? e[0] : e[W - 1]) = one[0];
        }
    } else if (W == 1 || n_out == W) {
        short_block_error<W>(coef, b, m, ld, start, n, bits, e);
    } else {
        double one[1];
        short_block_error<1>(coef, b, m, ld, start, n, bits, one);
        e[0] = one[0];
    }
    // fixed-order reduction over the workgroup
#pragma unroll
    for (int w = 0; w < W; ++w) red[w][threadIdx.x] = e[w];
    __syncthreads();
    for (int d = kCalibThreads / 2; d > 0; d >>= 1) {
        if ((int)threadIdx.x < d) {
#pragma unroll
            for (int w = 0; w < W; ++w) red[w][threadIdx.x] += red[w][threadIdx.x + d];
        }
        __syncthreads();
    }
    if ((int)threadIdx.x >= w0 && (int)threadIdx.x < w1 && (int)threadIdx.x < n_out) {
        if (halved) unsafeAtomicAdd(out + threadIdx.x, red[threadIdx.x][0]);
        else out[threadIdx.x] = red[threadIdx.x][0];
    }
}


// ---- moments ------------------------------------------------------------------------------------
// The second-moment matrix is symmetric: a workgroup owns a 32 x 32 tile on or above the diagonal and stores it both ways.
// Its four waves take a quarter of the tokens each and are summed in wave order at the end.  Products on the fp64
// matrix cores (v_mfma_f64_16x16x4: 16 x 16 features, 4 tokens), 2 x 2 of them per wave: the even and the odd features
// of each 32-feature strip, so that a lane's operands for both are one dword (bf16) of its token's row and a wave reads
// 64 contiguous bytes of four tokens.  Operands go straight from memory to registers, kGramAhead groups of four tokens
// ahead of their use; strips are re-read from L2.  A diagonal tile also sums its own operands: the first moment.
// Bound by the fp64 matrix rate -- 8192 tokens x 1024 features are 8.9 GFLOP = 0.11 ms at 78 TFLOP/s -- behind which hides no vector
// instruction: every one counts, so addresses are scalar and a whole group's loads carry no mask.  Tiles that
// do not fill another round of the compute units are split, by the parity of their features, in halves or quarters where those still fit
// one to a compute unit: 528 tiles on 256 of them end as two rounds and a quarter, not three.
// Measured: 1.24 ms with vector fp64 from LDS over the whole matrix, plus 2.03 ms for a separate pass of sums; both
// together 0.25 ms with whole tiles and masked loads, 0.20 with the last tiles split, 0.167 without masks and without the
// diagonal's sums in every tile (300 tiles: 171, 127, 103 us; 10 tiles: 77, 53, 38).
constexpr int kGramStrip = 32;
constexpr int kGramWaves = 4;
constexpr int kGramAhead = 8;

typedef double f64x4 __attribute__((ext_vector_type(4)));
typedef float f32x2 __attribute__((ext_vector_type(2)));

struct __attribute__((packed, aligned(8))) Doubles2 { double x, y; };       // two entries of the matrix: it is 8-byte aligned, no more
__device__ __forceinline__ double gram_value(uint32_t v, int odd) { return (double)bits_f32(odd ? v & 0xffff0000u : v << 16); }
__device__ __forceinline__ double gram_value(f32x2 v, int odd) { return (double)v[odd]; }
template <typename XT> struct GramVec { using type = uint32_t; };
template <> struct GramVec<float> { using type = f32x2; };

// element offset of feature f inside a token (blocks of 2^blk_log2 features lie blk_jump elements apart; 0 = contiguous)
__device__ __forceinline__ int64_t feature_offset(int f, int blk_log2, int64_t blk_jump) {
    return (int64_t)f + (blk_log2 ? (int64_t)(f >> blk_log2) * blk_jump : (int64_t)0);
}

// Features of parity a0 .. a0 + MA - 1 of strip bi against parity b0 .. b0 + MB - 1 of strip bj.
template <typename XT, int MA, int MB>
__device__ __forceinline__ void gram_tile(const XT* x, int64_t n_tokens, int p, int64_t ld, int blk_log2, int64_t blk_jump, int tile, int a0, int b0,
                                          double (*red)[18][64], double* sum, double* gram) {
    using V = typename GramVec<XT>::type;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, l16 = lane & 15, k = lane >> 4;
    // tile number -> (bi <= bj): column bj of the triangle starts at bj (bj + 1) / 2
    int bj = (int)((__builtin_sqrtf(8.0f * (float)tile + 1.0f) - 1.0f) * 0.5f);
    while ((int64_t)bj * (bj + 1) / 2 > tile) --bj;
    while ((int64_t)(bj + 1) * (bj + 2) / 2 <= tile) ++bj;
    const int bi = tile - (int)((int64_t)bj * (bj + 1) / 2);
    const bool diag = bi == bj;
    // a strip lies inside one block of the layout: its offset is the same for all lanes, and a lane's own is below 2^26 bytes
    typedef const char __attribute__((address_space(1))) * global_ptr;
    typedef const V __attribute__((address_space(1))) * global_v;
    const uint64_t xa = (uint64_t)uniform_ptr(x + feature_offset(bi * kGramStrip, blk_log2, blk_jump));
    const uint64_t xb = (uint64_t)uniform_ptr(x + feature_offset(bj * kGramStrip, blk_log2, blk_jump));
    const uint32_t own = (uint32_t)(k * (int)ld + 2 * l16) * (uint32_t)sizeof(XT);
    const int64_t quarter = (n_tokens + 4 * kGramWaves - 1) / (4 * kGramWaves) * 4;          // whole groups of four tokens
    const int64_t first = __builtin_amdgcn_readfirstlane(wave) * quarter;
    const int64_t left = n_tokens - first < quarter ? n_tokens - first : quarter;
    const int n_groups = left > 0 ? (int)(left / 4) : 0, n_blocks = n_groups / kGramAhead;

    f64x4 acc[MA][MB];
#pragma unroll
    for (int a = 0; a < MA; ++a)
#pragma unroll
        for (int b = 0; b < MB; ++b) acc[a][b] = f64x4{0.0, 0.0, 0.0, 0.0};
    double s[MA];
#pragma unroll
    for (int a = 0; a < MA; ++a) s[a] = 0.0;
    V va[kGramAhead], vb[kGramAhead];
    auto fetch = [&](int g, int u) {                             // whole group g; behind the last one the last one again
        const uint64_t at = (uint64_t)(first + 4 * (int64_t)(g < n_groups ? g : n_groups - 1)) * (uint64_t)(ld * (int64_t)sizeof(XT));      // scalar addresses
        va[u] = *(global_v)((global_ptr)(xa + at) + own);
        vb[u] = *(global_v)((global_ptr)(xb + at) + own);
    };
    auto step = [&](const V& a_in, const V& b_in, auto diag_tag) {
        double da[MA], db[MB];
#pragma unroll
        for (int a = 0; a < MA; ++a) da[a] = gram_value(a_in, a0 + a);
#pragma unroll
        for (int b = 0; b < MB; ++b) db[b] = gram_value(b_in, b0 + b);
#pragma unroll
        for (int a = 0; a < MA; ++a)
#pragma unroll
            for (int b = 0; b < MB; ++b) acc[a][b] = __builtin_amdgcn_mfma_f64_16x16x4f64(da[a], db[b], acc[a][b], 0, 0, 0);
        if constexpr (decltype(diag_tag)::value) {
#pragma unroll
            for (int a = 0; a < MA; ++a) s[a] += da[a];
        }
    };
    // a copy of the sweep for the diagonal: as a choice per step the sums were computed in every tile and dropped
    auto sweep = [&](auto diag_tag) {
        if (n_groups > 0) {
#pragma unroll
            for (int u = 0; u < kGramAhead; ++u) fetch(u, u);
            for (int b = 0; b < n_blocks; ++b) {
#pragma unroll
                for (int u = 0; u < kGramAhead; ++u) {
                    const V a_in = va[u], b_in = vb[u];
                    step(a_in, b_in, diag_tag);
                    fetch((b + 1) * kGramAhead + u, u);
                    __builtin_amdgcn_sched_barrier(0);
                }
            }
#pragma unroll
            for (int u = 0; u < kGramAhead; ++u)
                if (u < n_groups - n_blocks * kGramAhead) step(va[u], vb[u], diag_tag);
        }
        if (left > 4 * (int64_t)n_groups) {                      // one to three tokens: the rest of the group reads as zeros
            V a_in = V{}, b_in = V{};
            if (4 * n_groups + k < left) {
                const uint64_t at = (uint64_t)(first + 4 * (int64_t)n_groups) * (uint64_t)(ld * (int64_t)sizeof(XT));
                a_in = *(global_v)((global_ptr)(xa + at) + own);
                b_in = *(global_v)((global_ptr)(xb + at) + own);
            }
            step(a_in, b_in, diag_tag);
        }
    };
    if (diag) sweep(std::true_type()); else sweep(std::false_type());
#pragma unroll
    for (int a = 0; a < MA; ++a)
#pragma unroll
        for (int b = 0; b < MB; ++b)
#pragma unroll
            for (int r = 0; r < 4; ++r) red[wave][(a * MB + b) * 4 + r][lane] = acc[a][b][r];
#pragma unroll
    for (int a = 0; a < MA; ++a) red[wave][16 + a][lane] = s[a];
    __syncthreads();
    auto total = [&](int v, int l) {
        double t = red[0][v][l];
#pragma unroll
        for (int w = 1; w < kGramWaves; ++w) t += red[w][v][l];
        return t;
    };
    // wave r stores accumulator register r: rows 4 r + lane / 16 of the 16 x 16 results, columns lane % 16
    static_assert(kGramWaves == 4, "a wave per accumulator register");
    const int r = wave;
    double m[MA][MB];
#pragma unroll
    for (int a = 0; a < MA; ++a)
#pragma unroll
        for (int b = 0; b < MB; ++b) m[a][b] = total((a * MB + b) * 4 + r, lane);
    const int i = bi * kGramStrip + 2 * (4 * r + k) + a0, j = bj * kGramStrip + 2 * l16 + b0;
    auto put = [&](double* to, double u, double v, int n) {      // n neighbours
        if (n == 2) *reinterpret_cast<Doubles2*>(to) = Doubles2{u, v};
        else *to = u;
    };
#pragma unroll
    for (int a = 0; a < MA; ++a) put(gram + (size_t)(i + a) * p + j, m[a][0], m[a][MB - 1], MB);
    if (!diag) {
#pragma unroll
        for (int b = 0; b < MB; ++b) put(gram + (size_t)(j + b) * p + i, m[0][b], m[MA - 1][b], MA);
    } else if (a0 >= b0 && a0 < b0 + MB && tid < 16 * MA) {      // (one of the parts that see these features) lane l16 + 16 k holds the tokens 4 g + k of feature pair l16
        const int v = 16 + tid % MA, l = tid / MA;
        sum[bi * kGramStrip + 2 * l + a0 + tid % MA] = ((total(v, l) + total(v, l + 16)) + total(v, l + 32)) + total(v, l + 48);
    }
}

template <typename XT>
__global__ void __launch_bounds__(64 * kGramWaves, 3) calib_gram_kernel(const XT* x, int64_t n_tokens, int p, int64_t ld, int blk_log2, int64_t blk_jump,
                                                                     int n_whole, int split, double* sum, double* gram) {
    __shared__ double red[kGramWaves][18][64];
    const int b = (int)blockIdx.x - n_whole;
    if (b < 0) gram_tile<XT, 2, 2>(x, n_tokens, p, ld, blk_log2, blk_jump, (int)blockIdx.x, 0, 0, red, sum, gram);
    else if (split == 2) gram_tile<XT, 2, 1>(x, n_tokens, p, ld, blk_log2, blk_jump, n_whole + b / 2, 0, b % 2, red, sum, gram);
    else gram_tile<XT, 1, 1>(x, n_tokens, p, ld, blk_log2, blk_jump, n_whole + b / 4, b / 2 % 2, b % 2, red, sum, gram);
}

}  // namespace

namespace kvtc {
// x: n_tokens tokens of p features (p a multiple of 64) at the given layout; sum [p], gram [p][p]
hipError_t launch_calib_moments(const void* x, kvtc_dtype dtype, int64_t n_tokens, int p, int64_t ld, int blk_log2, int64_t blk_jump,
                                double* sum, double* gram, hipStream_t stream) {
    const int64_t strips = p / kGramStrip, tiles = strips * (strips + 1) / 2, cus = compute_units(), rest = tiles % cus;
    const int split = rest * 4 <= cus ? 4 : (rest * 2 <= cus ? 2 : 1);
    const int64_t whole = split == 1 ? tiles : tiles - rest;
    const dim3 grid((unsigned)(whole + (tiles - whole) * split)), threads(64 * kGramWaves);
    if (dtype == KVTC_BF16)
        hipLaunchKernelGGL(calib_gram_kernel<uint16_t>, grid, threads, 0, stream, static_cast<const uint16_t*>(x), n_tokens, p, ld, blk_log2, blk_jump, (int)whole, split, sum, gram);
    else
        hipLaunchKernelGGL(calib_gram_kernel<float>, grid, threads, 0, stream, static_cast<const float*>(x), n_tokens, p, ld, blk_log2, blk_jump, (int)whole, split, sum, gram);
    return hipGetLastError();
}
}  // namespace kvtc

extern "C" {

kvtc_status kvtc_calib_block_errors(const float* coef_dev, int64_t n_tokens, int64_t ld, const kvtc_calib_block* blocks_dev, int n_blocks,
                                    int max_bits, double* change_dev, kvtc_stream stream) {
    if (n_blocks < 0 || n_tokens < 0) return set_error(KVTC_E_ARG, "kvtc_calib_block_errors: n_blocks=%d, n_tokens=%lld", n_blocks, (long long)n_tokens);
    if (max_bits < 1 || max_bits > kCalibMaxBits) return set_error(KVTC_E_ARG, "kvtc_calib_block_errors: max_bits=%d outside 1..%d", max_bits, kCalibMaxBits);
    if (n_blocks == 0) return KVTC_OK;
    if (!coef_dev || !blocks_dev || !change_dev) return set_error(KVTC_E_ARG, "kvtc_calib_block_errors: null argument");
    if (ld < 1) return set_error(KVTC_E_ARG, "kvtc_calib_block_errors: ld=%lld", (long long)ld);
    if ((reinterpret_cast<uintptr_t>(coef_dev) & 3u) || (reinterpret_cast<uintptr_t>(change_dev) & 7u) || (reinterpret_cast<uintptr_t>(blocks_dev) & 3u))
        return set_error(KVTC_E_ARG, "kvtc_calib_block_errors: misaligned buffer");
    const int64_t n_out = (int64_t)n_blocks * max_bits;
    const bool halves = n_tokens > kCalibHalveAbove;
    if (halves)
        hipLaunchKernelGGL(calib_zero_kernel, dim3((unsigned)(n_out < 262144 ? (n_out + 255) / 256 : 1024)), dim3(256), 0, static_cast<hipStream_t>(stream), change_dev, n_out);
    // two widths to a workgroup (the last one's alone where their number is odd), unless there is one or the compute units take a workgroup each with one
    // (13 blocks x 8 widths: 25 us with two, 18 with one; 30 blocks: 45 and 32; 300 blocks of 256 coordinates x 1 width x 2048 tokens: 132 with two, 87
    // with one; 175 blocks x 5 widths x 150 tokens: 39.1 with six widths evaluated, 32.8 with five)
    const int widths = max_bits == 1 || (int64_t)n_blocks * max_bits <= compute_units() ? 1 : 2;
    void (*const fn)(const float*, int64_t, int64_t, const kvtc_calib_block*, int, double*) = widths == 1 ? &calib_block_errors_kernel<1> : &calib_block_errors_kernel<2>;
    // a launch has fewer than 2^32 threads across: beyond 2^22 - 1 blocks of 1024 threads the list takes several
    for (int64_t at = 0; at < n_blocks; at += kCalibMaxBlocks) {
        const int n = n_blocks - at < kCalibMaxBlocks ? (int)(n_blocks - at) : kCalibMaxBlocks;
        hipLaunchKernelGGL(fn, dim3((unsigned)n, (unsigned)((max_bits + widths - 1) / widths), halves ? 2 * widths + 1 : 1), dim3(kCalibThreads), 0, static_cast<hipStream_t>(stream), coef_dev, n_tokens, ld,
                           blocks_dev + at, max_bits, change_dev + at * max_bits);
    }
    const hipError_t err = hipGetLastError();
    if (err != hipSuccess) return set_error(KVTC_E_HIP, "kvtc_calib_block_errors: launch failed: %s", hipGetErrorString(err));
    return KVTC_OK;
}

}  // extern "C"
