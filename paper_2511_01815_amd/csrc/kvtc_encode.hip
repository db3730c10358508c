// Fused encode kernel for gfx950: projection onto the kept PCA basis on the bf16 matrix
// cores, then per-token group min-max quantisation and bit-packing, one launch.
// (Paper, Section "Method", mode "Compression"; Sections "Feature decorrelation" and
// "Quantization".)
//
// Work decomposition.  A workgroup (4 wavefronts, or 8 for plans of more than 320 padded coordinates)
// owns a tile of tokens and ALL kept coordinates of those tokens, because a group's min/max
// needs every coordinate of the group before any of its codes exists.
// The product is computed transposed, D^T = V_kept^T X^T, with the 32x32x16 bf16 MFMA:
// M = coordinates, N = tokens, K = features.  Then a lane owns one token (column) and, by
// permuting the rows of the A operand, 16 *consecutive* coordinates of it per 32-coordinate
// tile -- exactly one 16-coordinate block of the record format, so quantisation and packing
// are lane-local with static bit offsets.
//   * V_kept is pre-swizzled at plan creation into A-operand fragments.  Up to 640 padded coordinates
//     slabs of it move global -> LDS without register staging, a ring stage or two ahead of the
//     MFMAs; beyond, and in the kernel for short jobs, every fragment is used by one wave alone and
//     goes straight to its registers.  The tile's X rows move global -> LDS.  Every byte of X is read
//     from HBM once, the basis is re-read (from L2) once per tile, so larger token tiles mean less
//     traffic per token.
//   * The coordinates are split over WC wavefronts that share the tokens; the other wavefronts
//     take further tokens.  A wavefront holds TT x NTW accumulator tiles of 32 x 32.
// Epilogue: block min/max -> LDS -> per (token, group) header (fp16 shift down, scale up)
// -> codes -> written into the record image in LDS -> one contiguous, coalesced store of the
// tile's records.
#include <hip/hip_runtime.h>
#include <type_traits>
#include "kvtc_dev.h"
#include "kvtc_numeric.h"

namespace kvtc {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));

__device__ __forceinline__ bf16x8 as_bf16x8(uint4 v) { return __builtin_bit_cast(bf16x8, v); }

// The X slab of one step in LDS: TOK rows of KS*16 features, written by global->LDS transfers
// in 16-byte columns.  Column c of row r is stored at column c ^ swz(r) so that the 8 lanes
// served together by a 128-bit LDS read (8 consecutive tokens, same column) fall on 8 different
// 16-byte bank groups.
template <typename XT, int KS> struct XSlab;
template <int KS> struct XSlab<uint16_t, KS> {                 // bf16 input: KS*32 bytes per row
    static constexpr int ROW_B = KS * 32, COLS = ROW_B / 16, ROWS_PER_DMA = 64 / COLS;
    static __device__ __forceinline__ int swz(int r) { return (r * COLS / 8) & (COLS - 1); }
    // B fragment of (row, k-step, lane half): 8 consecutive features
    static __device__ __forceinline__ bf16x8 frag(const char* slab, int row, int ks, int h) {
        const int c = (2 * ks + h) ^ swz(row);
        return as_bf16x8(*reinterpret_cast<const uint4*>(slab + row * ROW_B + c * 16));
    }
};
template <int KS> struct XSlab<float, KS> {                    // fp32 input: KS*64 bytes per row
    static constexpr int ROW_B = KS * 64, COLS = ROW_B / 16, ROWS_PER_DMA = 64 / COLS;
    static __device__ __forceinline__ int swz(int r) { return (r * COLS / 8) & (COLS - 1); }
    static __device__ __forceinline__ bf16x8 frag(const char* slab, int row, int ks, int h) {
        const int c0 = (4 * ks + 2 * h) ^ swz(row), c1 = (4 * ks + 2 * h + 1) ^ swz(row);
        const float4 a = *reinterpret_cast<const float4*>(slab + row * ROW_B + c0 * 16);
        const float4 b = *reinterpret_cast<const float4*>(slab + row * ROW_B + c1 * 16);
        bf16x8 r;                                                // round to bf16, nearest even
        r[0] = (__bf16)a.x; r[1] = (__bf16)a.y; r[2] = (__bf16)a.z; r[3] = (__bf16)a.w;
        r[4] = (__bf16)b.x; r[5] = (__bf16)b.y; r[6] = (__bf16)b.z; r[7] = (__bf16)b.w;
        return r;
    }
};

// OR `len` bits of v into the record image at bit position pos (pos, len per lane).
__device__ __forceinline__ void put_bits(uint32_t* rec, uint32_t pos, uint32_t v, uint32_t len) {
    const uint32_t dw = pos >> 5, s = pos & 31u;
    atomicOr(rec + dw, v << s);
    if (s + len > 32u) atomicOr(rec + dw + 1, v >> (32u - s));
}

// The 16 codes of a block, BITS wide each and given as code_float makes them, as a bit string of BITS halfwords written to the record
// image at a halfword address (blocks start and end on halfword boundaries: 16 codes x BITS bits).
// Plain LDS stores: two blocks may share a dword but never a halfword, so nothing is OR-ed
// and the image needs no clearing.  (Codes are added up, shifted, with the floats' upper bits; what those come to is subtracted at the end.)
template <int BITS>
__device__ __forceinline__ void emit_block(const uint32_t (&u)[16], char* dst) {
    constexpr int ND = (BITS + 1) / 2;
    constexpr uint32_t BASE = code_base_bits(BITS);
    uint32_t q[ND], extra[ND];
#pragma unroll
    for (int j = 0; j < ND; ++j) extra[j] = 0u;
#pragma unroll
    for (int i = 0; i < 16; ++i) {
        const int pos = i * BITS, dw = pos >> 5, sh = pos & 31;
        if (sh == 0) q[dw] = u[i];
        else asm("v_lshl_add_u32 %0, %1, %2, %0" : "+v"(q[dw]) : "v"(u[i]), "n"(sh));        // (of two of these sums the compiler makes three instructions)
        extra[dw] += BASE << sh;
        if (sh + BITS > 32) q[dw + 1] = __builtin_amdgcn_ubfe(u[i], 32 - sh, BITS - (32 - sh));
    }
#pragma unroll
    for (int j = 0; j < ND; ++j) q[j] -= extra[j];
    __builtin_memcpy(__builtin_assume_aligned(dst, 2), q, 2 * BITS);
}

// The LDS rings of the bulk encode: stages of the basis, some k-steps (16 features each) to a stage, and slabs of X, sized so that a narrow plan (<= 10
// coordinate tiles, two workgroups per compute unit; three of 6 tiles) stays within 72 KB (44 KB) and a wide one (one workgroup) within 152 KB.
// token tiles (of 32) per wave: three where the registers allow it (8 coordinate tiles over two waves: 192 accumulator registers), which cuts the
// basis traffic per token by a third; one where a plan is so narrow that X is all there is to fetch, and half as much LDS holds its whole lines
__host__ __device__ constexpr int enc_tt(int ntp, int nw, int wc) { return nw == 4 && wc == 2 && ntp == 8 ? 3 : (ntp <= 2 ? 1 : 2); }
// X by whole lines of 128 bytes (bf16): eight rows of four k-steps to a transfer.  By half lines, a stage's two k-steps, every line is asked for at
// two times; its first half leaves it in the L2 in place of some of the basis, and with reads that do not, the second half is fetched from HBM again (32-layer
// cache at 16x: 1290 -> 1750 us).  By whole lines an input beyond the last-level cache goes past the L2s (ONCE).  Of 4, 8 and 10 tiles only then: their
// slabs of X, 64 KB at two workgroups to a compute unit, leave the basis a stage of one or two k-steps ahead, and an input that comes from that cache was
// faster by half lines (one tensor of 50000 tokens at 16x: 49 us, by lines 55).  Not of 6 tiles: by lines a third workgroup does not fit the LDS
// (two of 75000 tokens at 20x: 92 us with three, 108 with two).  us, before and after: 32-layer cache, encode, 16x 1280 -> 1224; 16 tensors of 32768 at
// 8x, both ways, 1196 -> 1170; two-tile plans at 40x, 16 tensors of 20000 tokens: 147 -> 123, fp32 319 -> 270 (there by smaller tiles alone).
__host__ __device__ constexpr bool enc_lines(int ntp, int elem_bytes, bool once) { return elem_bytes == 2 && ntp != 6 && (once || ntp <= 2 || ntp > 10); }
// k-steps per stage of the basis ring, and k-steps whose X is fetched together: four where it comes by lines, else those of a stage
__host__ __device__ constexpr int enc_ks(int ntp, int elem_bytes, bool once) {
    if (enc_lines(ntp, elem_bytes, once)) return ntp <= 2 ? 4 : (ntp == 8 || ntp == 4 ? 1 : 2);
    return ntp < 8 || (ntp == 8 && elem_bytes == 2) || (ntp > 10 && ntp <= (elem_bytes == 2 ? 20 : 16)) ? 2 : 1;      // fp32 X slabs are twice as large
}
__host__ __device__ constexpr int enc_kx(int ntp, int elem_bytes, bool once) { return enc_lines(ntp, elem_bytes, once) ? 4 : enc_ks(ntp, elem_bytes, once); }
// stages of the basis ring, and slabs of the X ring: as many of the former as fit the variant's LDS share, 2..4; of the latter as many where a slab is
// a stage's X, else two
__host__ __device__ constexpr int enc_x_slab(int ntp, int elem_bytes, int nw, int wc, bool once) {
    return 32 * enc_tt(ntp, nw, wc) * (nw / wc) * enc_kx(ntp, elem_bytes, once) * 16 * elem_bytes;
}
__host__ __device__ constexpr int enc_stages(int ntp, int elem_bytes, int nw, int wc, bool once) {
    const bool same = enc_kx(ntp, elem_bytes, once) == enc_ks(ntp, elem_bytes, once);
    const int v_b = enc_ks(ntp, elem_bytes, once) * ntp * 1024, x_b = enc_x_slab(ntp, elem_bytes, nw, wc, once);
    const int budget = (nw == 4 && wc == 2 && ntp == 6 ? 44 : (nw == 4 ? 72 : 152)) * 1024;
    const int n = same ? budget / (v_b + x_b) : (budget - 2 * x_b) / v_b;
    return n < 2 ? 2 : (n > 4 ? 4 : n);
}
__host__ __device__ constexpr int enc_ring_bytes(int ntp, int elem_bytes, int nw, int wc, bool once) {
    const int n = enc_stages(ntp, elem_bytes, nw, wc, once);
    return n * enc_ks(ntp, elem_bytes, once) * ntp * 1024 +
           (enc_kx(ntp, elem_bytes, once) == enc_ks(ntp, elem_bytes, once) ? n : 2) * enc_x_slab(ntp, elem_bytes, nw, wc, once);
}

// Fewest coordinate tiles worked on for a plan that runs as ntp of them (the padding is left out in the variants of 6, 8, 10 and 20), and what
// follows for the transfers of a stage's basis pieces: whether every wave has an i-th one whatever the plan, and how many a wave has at least.
__host__ __device__ constexpr int enc_min_tiles(int ntp) { return ntp > 4 && ntp <= 10 ? ntp - 1 : (ntp == 20 ? 17 : ntp); }
template <int NTP, int NW, int TOTAL> __host__ __device__ constexpr bool enc_basis_pieces(int i) {
    for (int w = 0; w < NW; ++w)
        if (i * NW + w >= TOTAL || (i * NW + w) % NTP >= enc_min_tiles(NTP)) return false;
    return true;
}
template <int NTP, int NW, int TOTAL> __host__ __device__ constexpr int enc_least_pieces() {
    int least = TOTAL;
    for (int w = 0; w < NW; ++w) {
        int n = 0;
        for (int i = w; i < TOTAL; i += NW) n += i % NTP < enc_min_tiles(NTP);
        least = n < least ? n : least;
    }
    return least;
}

// Steps after which basis ring and X ring are where they began.
__host__ __device__ constexpr int enc_common(int a, int b) {
    int n = a;
    while (n % b != 0) n += a;
    return n;
}
// Transfers a wave may have in flight at the end of step u (of a loop that is unrolled by a multiple of spc, and in which step t asks for the basis of step t + d
// and, where t is a multiple of spc, then for the next slab of X): those younger than the basis of step u + 1 and, where that begins a slab, than the slab.
__host__ __device__ constexpr int enc_in_flight(int u, int d, int spc, int nv, int nx) {
    int n = 0;
    for (int t = u + 1 - d; t <= u; ++t) n += (t > u + 1 - d ? nv : 0) + ((t + 64 * spc) % spc == 0 ? nx : 0);
    const int slab = (spc - 1) * nv;
    return (u + 1) % spc == 0 && slab < n ? slab : n;
}

// LDS work area (behind the job table): [tables of the tile's plan: block table 64 dwords, group
// table 64 dwords, -(mu^T V_kept) of the padded coordinates][ring / epilogue images].  The tables
// arrive by asynchronous transfers at the start of a tile, ahead of the first ring stage, so
// no load of the tile loop is visible to the compiler (a visible vector load makes it wait for
// everything in flight, and costs an L2 round trip where it stands).
constexpr int kEncBlkOff = 0, kEncGrpOff = 256, kEncNegcOff = 512;
__host__ __device__ constexpr int enc_aux_bytes(int ntp) { return 512 + ntp * 32 * 4; }

// From a workgroup's coefficients (accumulator tiles of 32 coordinates x 32 tokens, a lane holding 16 consecutive coordinates of a
// token) to records in the stream.  Every wave of the workgroup calls it: ct0 = the wave's first coordinate tile, n_ct = how many it has (NTW or one
// fewer; HELPERS: any number, a wave with none only helps with the headers and the copy), tt0 = its first of TT token tiles;
// tok_n tokens of the images' pitch tok_wg are worked on.  LDS: the plan's tables at `work`, the images at `smem`.
// PART: of the groups and record bytes, those of `part` only.
struct EncPart {
    int g0, g1, ct0, ct1, hw0, hw1;         // groups, coordinate tiles, halfwords of codes: first and last + 1
    __device__ __forceinline__ EncPart(uint32_t a, uint32_t b)
        : g0((int)(a & 0xffu)), g1((int)((a >> 8) & 0xffu)), ct0((int)((a >> 16) & 0xffu)), ct1((int)(a >> 24)), hw0((int)(b & 0xffffu)), hw1((int)(b >> 16)) {}
};
template <int NTW, int TT, bool HELPERS, bool PART = false>
__device__ __forceinline__ void encode_epilogue(const f32x16 (&acc)[TT][NTW], int ct0, int n_ct, int tt0, int tok_n, int tok_wg, int ntp, int nth,
                                                const PlanEnc& P, const TileRef& tr, const KernelArgs& a, int tok_tile0, uint4* work, uint4* smem,
                                                const EncPart& part = EncPart(0u, 0u)) {
    // (through an empty asm, so that nothing of the epilogue's lane addresses is worked out ahead of the main loop and kept
    // through it: its registers are all taken)
    int tid = (int)threadIdx.x;
    asm volatile("" : "+v"(tid));
    const int l32 = tid & 31, h = (tid >> 5) & 1;
    const int T = tr.n_tokens;
    // mm[2*ntp][tok_wg] float2 | gq[G][tok_wg] float2 | rec[tok_wg][rd + 1] dwords
    const int G = P.n_groups;
    const int rd = P.rec_dwords;
    const uint32_t* blk_t = reinterpret_cast<const uint32_t*>(work) + kEncBlkOff / 4;
    const uint32_t* grp_t = reinterpret_cast<const uint32_t*>(work) + kEncGrpOff / 4;
    const int rstride = rd + 1;                 // odd-ish pitch keeps lanes on distinct banks
    float2* mm = reinterpret_cast<float2*>(smem);
    float2* gq = mm + 2 * ntp * tok_wg;
    uint32_t* rec = reinterpret_cast<uint32_t*>(gq + G * tok_wg);

    // A: block min/max
#pragma unroll
    for (int tt = 0; tt < TT; ++tt) {
        const int tw = (tt0 + tt) * 32 + l32;
#pragma unroll
        for (int ct = 0; ct < NTW; ++ct) {
            if (ct >= (HELPERS ? 0 : NTW - 1) && ct >= n_ct) continue;
            const f32x16& d = acc[tt][ct];
            float lo = d[0], hi = d[0];
#pragma unroll
            for (int i = 1; i < 16; ++i) { lo = fminf(lo, d[i]); hi = fmaxf(hi, d[i]); }
            mm[(2 * (ct0 + ct) + h) * tok_wg + tw] = make_float2(lo, hi);
            __builtin_amdgcn_sched_barrier(0);      // keep the accumulator reads from piling up
        }
    }
    // codes wider than 8 bits are OR-ed into the image (cleared here); the usual widths are stored
    const bool narrow_codes = P.code_bits_max <= 8;
    uint32_t* saturated = reinterpret_cast<uint32_t*>(work) + kEncNegcOff / 4;       // (-(mu^T V_kept) has been used)
    if (tid == 0) *saturated = 0u;
    if (!narrow_codes)
        for (int i = tid; i < tok_wg * rstride; i += nth) rec[i] = 0u;
    __syncthreads();

    // B: one header per (token, group)
    const int g_first = PART ? part.g0 : 0, g_last = PART ? part.g1 : G;
    for (int item = tid; item < tok_n * (g_last - g_first); item += nth) {
        const int tw = item % tok_n, g = item / tok_n + g_first;
        const uint32_t gi = grp_t[g];
        const int b0 = gi & 0xff, nb = (gi >> 8) & 0xff, bits = (gi >> 16) & 0xff;
        float lo = __builtin_inff(), hi = -__builtin_inff();
        for (int k0 = 0; k0 < nb; k0 += 4) {            // four reads in flight; behind the last block the last one again
            float2 m[4];
#pragma unroll
            for (int k = 0; k < 4; ++k) m[k] = mm[(b0 + min(k0 + k, nb - 1)) * tok_wg + tw];
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                lo = fminf(lo, m[k].x);
                hi = fmaxf(hi, m[k].y);
            }
        }
        const GroupQ q = group_header(lo, hi, bits);
        gq[g * tok_wg + tw] = make_float2(q.shift, __builtin_ldexpf(q.inv, -bits));      // exact
        rec[tw * rstride + g] = (uint32_t)q.shift16 | ((uint32_t)q.scale16 << 16);
        if (__builtin_expect(q.scale16 == 0x7bffu, 0)) *saturated = 1u;
        if (g == g_first && narrow_codes) rec[tw * rstride + rd - 1] = 0u;      // the padding behind the last block
    }
    __syncthreads();

    // C: codes of the lane's blocks, put into the record image.  (The halves of a wave have a block each: one width in most
    // tiles, two at most.  The choice by width is one for the wave, made for either half in turn -- as a choice per lane it was six levels of masks.)
    auto codes = [&](auto narrow_tag) {
#pragma unroll
        for (int ct = 0; ct < NTW; ++ct) {
            if (ct >= (HELPERS ? 0 : NTW - 1) && ct >= n_ct) continue;
            const uint32_t info = blk_t[2 * (ct0 + ct) + h];
            const uint32_t bits = PART && ((int)((info >> 8) & 0xffu) < part.g0 || (int)((info >> 8) & 0xffu) >= part.g1) ? 0u : info & 0xffu;
            const uint32_t bits0 = (uint32_t)__builtin_amdgcn_readlane((int)bits, 0), bits1 = (uint32_t)__builtin_amdgcn_readlane((int)bits, 32);
            if ((bits0 | bits1) == 0u) continue;
            const uint32_t g = (info >> 8) & 0xffu;
            const uint32_t pos0 = (info >> 16) * 16u;
            const float base = __uint_as_float(code_base_bits(bits)), qmax = (float)((1u << bits) - 1u);
#pragma unroll
            for (int tt = 0; tt < TT; ++tt) {
                const int tw = (tt0 + tt) * 32 + l32;
                const float2 sq = gq[g * tok_wg + tw];
                uint32_t* row = rec + tw * rstride;
                const f32x16& d = acc[tt][ct];
                uint32_t u[16];
                if constexpr (decltype(narrow_tag)::value) {
#pragma unroll
                    for (int i = 0; i < 16; ++i) u[i] = code_float(d[i], sq.x, sq.y, base);
                    char* dst = reinterpret_cast<char*>(row) + (pos0 >> 3);
#pragma unroll 1
                    for (uint32_t b = bits0;;) {
                        const bool mine = bits == b;
#pragma unroll
                        for (int i = 0; i < 16; ++i) asm volatile("" : "+v"(u[i]));      // (or every width's part codes are cut out ahead of the choice)
                        switch (b) {
                            case 0: break;
                            case 1: if (mine) emit_block<1>(u, dst); break;
                            case 2: if (mine) emit_block<2>(u, dst); break;
                            case 3: if (mine) emit_block<3>(u, dst); break;
                            case 4: if (mine) emit_block<4>(u, dst); break;
                            case 5: if (mine) emit_block<5>(u, dst); break;
                            case 6: if (mine) emit_block<6>(u, dst); break;
                            case 7: if (mine) emit_block<7>(u, dst); break;
                            default: if (mine) emit_block<8>(u, dst); break;
                        }
                        if (b == bits1) break;
                        b = bits1;
                    }
                } else if (bits != 0u) {
#pragma unroll
                    for (int i = 0; i < 16; ++i) u[i] = (uint32_t)code_of(d[i], sq.x, __builtin_ldexpf(sq.y, (int)bits), qmax);
#pragma unroll
                    for (int k = 0; k < 8; ++k) put_bits(row, pos0 + 2u * k * bits, u[2 * k] | (u[2 * k + 1] << bits), 2u * bits);
                }
                __builtin_amdgcn_sched_barrier(0);
            }
        }
    };
    if (__builtin_expect(narrow_codes && *saturated == 0u, 1)) {
        codes(std::true_type());
    } else {
        if (narrow_codes) {                  // a scale of 65504: its codes have to be clamped.  (The image has not been cleared.)
            for (int i = tid; i < tok_wg * rstride; i += nth)
                if (i % rstride >= G) rec[i] = 0u;
            __syncthreads();
        }
        codes(std::false_type());
    }
    __syncthreads();

    // D: the tile's records are contiguous in the stream: one coalesced copy, 16 bytes per lane when the
    // tile starts on a 16-byte boundary of the buffer and records are whole 16-byte pieces (then a piece
    // never straddles two rows of the image), else dword by dword
    {
        const int n_valid = min(tok_n, T - tok_tile0);
        uint32_t* out = reinterpret_cast<uint32_t*>(reinterpret_cast<uint8_t*>(a.stream_buf) + tr.offset) +
                        (size_t)tok_tile0 * rd;
        const uint32_t magic = 0xffffffffu / (uint32_t)rd + 1u;     // exact floor(i / rd) for i < 2^20
        const int total = n_valid * rd;
        if constexpr (PART) {
            // the headers, then the dwords that hold the part's codes: a first or last one that it shares by its half
            const int n_head = part.g1 - part.g0, d0 = part.hw0 / 2, per = n_head + (part.hw1 + 1) / 2 - d0;
            for (int i = tid; i < n_valid * per; i += nth) {
                const int t = i / per, k = i - t * per, d = k < n_head ? part.g0 + k : d0 + k - n_head;
                const uint32_t w = rec[t * rstride + d];
                uint32_t* to = out + (size_t)t * rd + d;
                const bool low = k < n_head || 2 * d >= part.hw0, high = k < n_head || 2 * d + 1 < part.hw1;
                if (low && high) *to = w;
                else reinterpret_cast<uint16_t*>(to)[low ? 0 : 1] = (uint16_t)(low ? w : w >> 16);
            }
        } else if ((rd & 3) == 0 && (reinterpret_cast<uintptr_t>(out) & 15u) == 0u) {
            for (int i = 4 * tid; i < total; i += 4 * nth) {
                const uint32_t t = __umulhi((uint32_t)i, magic);
                const uint32_t* src = rec + t * rstride + ((uint32_t)i - t * rd);
                *reinterpret_cast<uint4*>(out + i) = make_uint4(src[0], src[1], src[2], src[3]);
            }
        } else {
            for (int i = tid; i < total; i += nth) {
                const uint32_t t = __umulhi((uint32_t)i, magic);
                out[i] = rec[t * rstride + ((uint32_t)i - t * rd)];
            }
        }
    }
    __syncthreads();
}

// ONCE (where X comes by whole lines: bf16 but of 6 tiles; fp32, whose two k-steps are one, up to 4; and where the features lie on whole lines): the call's
// input is as much as the last-level cache, 256 MB, holds, or more (encode_pass_bytes); its lines, which are read once, are then not to push the basis, of up to a megabyte a tensor, out of the L2s (11 to 20 tiles, 16 tensors of 32768 tokens at 8x, 1 GB, encode and
// decode: 1228 -> 1180 us; of 4000 tokens, whose 131 MB a call finds in that cache: 115 without, 122 with).  fp32
// at 40x: two tiles, 16 tensors of 20000 tokens, 268 -> 252, four tiles, two of 40000, 116 -> 110; of 6 and 16 tiles 1 to 4 % slower so.  A copy of the whole tile: as a choice per
// transfer it cost the small calls 2 to 4 %, as two main loops in front of one epilogue all calls half of their speed, in moves of accumulators.
constexpr bool enc_can_pass(int ntp, int elem_bytes) { return elem_bytes == 2 ? ntp != 6 : ntp <= 4; }
template <typename XT, int NTP> constexpr bool enc_once() { return enc_can_pass(NTP, (int)sizeof(XT)); }
template <int NTW, int WC, typename XT, int NW, bool ONCE>
__device__ __forceinline__ void encode_tile(const PlanEnc& P, const TileRef& tr,
                                            const KernelArgs& a, uint4* work) {
    constexpr int NTP = NTW * WC;            // coordinate tiles of the padded plan
    constexpr int TT = enc_tt(NTP, NW, WC);  // token tiles (of 32) per wave
    constexpr int NTH = NW * 64;             // threads of the workgroup
    constexpr int WT = NW / WC;              // waves across tokens
    constexpr int TOK_WG = 32 * TT * WT;
    constexpr int KS = enc_ks(NTP, (int)sizeof(XT), ONCE);
    constexpr int NSTAGE = enc_stages(NTP, (int)sizeof(XT), NW, WC, ONCE);
    constexpr int SLAB_U4 = KS * NTP * 64;
    constexpr int KX = enc_kx(NTP, (int)sizeof(XT), ONCE), SPC = KX / KS;      // k-steps whose X comes together; steps (stages) to them
    constexpr int NXS = SPC == 1 ? NSTAGE : 2;                  // slabs of the X ring

    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wt = wave / WC;
    // The plan's coordinate tiles are shared out evenly: a wave has NTW of them or one fewer, whose place it does not multiply, and the padding is
    // not fetched.  What these kernels have at their disposal is power -- the clock gives way, to 1.5 GHz, under matrix instructions and a stream
    // from HBM at once --, so work that can be left out counts although it would fit the time (32-layer cache at 16x, plans of 7, 8 and 9 tiles that
    // run as 8 and 10: 1300 -> 1282 us).  Not up to four tiles, which are bound by HBM, nor in the 8-wave variants of 12 and 16: the conditions cost those 0.5 %.
    // In that of 20 the two waves of a SIMD are two places apart in the coordinates, or the ones with a tile more would share one: plans of 528 coordinates, 17 tiles, 16 tensors
    // of 32768 tokens 702 us as 20 tiles, 686 without the padding, 673 so.  (By turns in the two workgroups of a compute unit, for those of 7 and 9 tiles, it gave nothing.)
    const int nt = enc_min_tiles(NTP) < NTP ? (P.r + 31) / 32 : NTP, wc = (wave + (NTP == 20 ? 2 * wt : 0)) % WC;
    const int ct0 = wc * (nt / WC) + min(wc, nt % WC), n_ct = nt / WC + (wc < nt % WC ? 1 : 0);
    const bool full = enc_min_tiles(NTP) == NTP || n_ct >= NTW;
    const int l32 = lane & 31, h = lane >> 5;
    const int p = P.p;
    const int T = tr.n_tokens;
    const int tok_tile0 = tr.tile * TOK_WG;
    uint4* smem = work + enc_aux_bytes(NTP) / 16;

    // ---- the plan's tables -> LDS (first used in the epilogue) --------------------------
    {
        const uint32_t aux = lds_offset(work);
        if (wave == 0) dma4_async(P.blk, (uint32_t)lane * 4u, aux + kEncBlkOff);
        if (wave == 1) dma4_async(P.grp, (uint32_t)lane * 4u, aux + kEncGrpOff);       // 64 entries allocated
        static_assert(NTP * 8 <= NTH, "one 16-byte piece per thread covers -(mu^T V_kept)");
        if (wave * 64 < NTP * 8 && tid < NTP * 8)
            dma16_async(P.negc, (uint32_t)tid * 16u, aux + kEncNegcOff + (uint32_t)wave * 1024u);
    }

    f32x16 acc[TT][NTW];

    // ---- LDS: a ring of NSTAGE basis slabs (a stage each) and one of NXS X slabs ----------
    using XS = XSlab<XT, KX>;
    constexpr int XSLAB_B = TOK_WG * XS::ROW_B;
    constexpr int NX_TOTAL = TOK_WG / XS::ROWS_PER_DMA;         // X transfers per slab, dealt round-robin to the waves
    constexpr int NXD = (NX_TOTAL + NW - 1) / NW;
    constexpr int NV_TOTAL = SLAB_U4 / 64;                      // basis transfers per stage (1 KB each), dealt the same way
    constexpr int NV = (NV_TOTAL + NW - 1) / NW;
    // transfers per wave, lower bounds over waves: of the basis for any plan, and for a wave none of whose pieces is padding.  (With the first alone a wave that
    // had all its pieces waited, every step, for one that it had only just asked for: fp32 of 8 tiles, 64 tensors of 2100 tokens of 240 coordinates 179 us, so 161.
    // Where at most a third of a wave's pieces may be padding it made no difference, and the choice cost half a percent.)
    constexpr int NV_MIN = enc_least_pieces<NTP, NW, NV_TOTAL>(), NV_ALL = 2 * NV_MIN <= NV_TOTAL / NW ? NV_TOTAL / NW : NV_MIN, NX_MIN = NX_TOTAL / NW;
    bool pads = false;                                          // some of the wave's pieces are
    if constexpr (NV_MIN < NV_ALL) {
#pragma unroll
        for (int i = 0; i < NV; ++i) pads = pads || (i * NW + wave < NV_TOTAL && (i * NW + wave) % NTP >= nt);
    }
    static_assert(TOK_WG % XS::ROWS_PER_DMA == 0 && KX % KS == 0, "whole transfers, whole steps");
    static_assert(3 * (NV + NXD) < 64, "vmcnt range");
    static_assert(NW >= 2, "waves 0 and 1 fetch the plan's tables");
    char* ring = reinterpret_cast<char*>(smem);
    const uint4* vg = P.v_enc;
    const int n_slabs = p / (16 * KS);

    // per-lane source of each X transfer, from the tile's first row: row (clamped at the tensor's end) and swizzled column.  (A
    // scalar address and a 32-bit offset per lane: with 64-bit lane addresses the 8-tile variant spilled 13 registers and reloaded
    // six of them per ring pass; 32-layer cache at 16x 1406 -> 1347 us.)
    const char* xtile = reinterpret_cast<const char*>(reinterpret_cast<const XT*>(a.x) + (tr.x_row0 + tok_tile0) * a.ld_x);
    uint32_t xsrc[NXD];                                         // below 2^31: at most 256 rows of 2^21 elements
    uint32_t xdst[NXD];                                         // wave-uniform LDS byte offsets inside an X slab
#pragma unroll
    for (int j = 0; j < NXD; ++j) {
        const int row0 = (j * NW + wave) * XS::ROWS_PER_DMA;
        const int row = row0 + lane / XS::COLS;
        const int col = (lane % XS::COLS) ^ XS::swz(row);
        const int t = min(row, T - 1 - tok_tile0);              // tail rows re-read the last token
        xsrc[j] = (uint32_t)t * (uint32_t)(a.ld_x * (int64_t)sizeof(XT)) + (uint32_t)(col * 16);
        xdst[j] = (uint32_t)(NSTAGE * SLAB_U4 * 16 + row0 * XS::ROW_B);
    }
    const uint32_t lds_ring = lds_offset(ring);

    // All global traffic of the main loop is asynchronous global->LDS transfers issued
    // NSTAGE-1 steps ahead; the only wait is the one in front of the barrier that publishes
    // the next stage, and it leaves the younger stages in flight.
    // byte offset of slab s inside a token's features: KS * 16 features per slab; with a blocked layout
    // (heads or layers apart in memory) every whole block before it adds the gap between blocks
    const int blk_lg = a.x_blk_log2;
    const size_t blk_jump_b = (size_t)a.x_blk_jump * sizeof(XT);
    auto issue_basis = [&](int s, int stage) {
        const uint32_t base = lds_ring + stage * SLAB_U4 * 16;
        const uint4* vsrc = vg + (size_t)s * SLAB_U4;           // scalar addresses plus a lane offset
#pragma unroll
        for (int i = 0; i < NV; ++i)
            if (enc_basis_pieces<NTP, NW, NV_TOTAL>(i) || (i * NW + wave < NV_TOTAL && (i * NW + wave) % NTP < nt))
                dma16_async(vsrc + i * NTH, (uint32_t)tid * 16u, base + (i * NTH + wave * 64) * 16);
    };
    auto issue_x = [&](int c, int slab) {
        const uint32_t base = lds_ring + slab * XSLAB_B;
        const size_t xoff = (size_t)c * XS::ROW_B + (blk_lg ? (size_t)((c * (16 * KX)) >> blk_lg) * blk_jump_b : (size_t)0);
#pragma unroll
        for (int j = 0; j < NXD; ++j)
            if ((j + 1) * NW <= NX_TOTAL || j * NW + wave < NX_TOTAL)
                ONCE ? dma16_async_once(xtile + xoff, xsrc[j], base + xdst[j]) : dma16_async(xtile + xoff, xsrc[j], base + xdst[j]);
    };
    // (a wave with a tile fewer than NTW reads the next wave's, or padding, in its place)
    auto compute = [&](int stage, int slab, int ks0) {          // ks0: the step's first k-step inside the X slab
        const uint4* abase = reinterpret_cast<const uint4*>(ring + stage * SLAB_U4 * 16) + ct0 * 64 + lane;
        const char* xs = ring + NSTAGE * SLAB_U4 * 16 + slab * XSLAB_B;
        constexpr int NSTEP = KS * NTW;
        bf16x8 xv[KS][TT];
#pragma unroll
        for (int ks = 0; ks < KS; ++ks)
#pragma unroll
            for (int tt = 0; tt < TT; ++tt) xv[ks][tt] = XS::frag(xs, (wt * TT + tt) * 32 + l32, ks0 + ks, h);
        uint4 af[3];
        af[0] = abase[0];
        if (NSTEP > 1) af[1] = abase[((1 / NTW) * NTP + (1 % NTW)) * 64];
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int j = 0; j < NSTEP; ++j) {
            const int ks = j / NTW, ct = j % NTW;
            if (j + 2 < NSTEP) af[(j + 2) % 3] = abase[(((j + 2) / NTW) * NTP + ((j + 2) % NTW)) * 64];
            const bf16x8 av = as_bf16x8(af[j % 3]);
            if (ct + 1 < NTW || full) {
#pragma unroll
                for (int tt = 0; tt < TT; ++tt)
                    acc[tt][ct] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(av, xv[ks][tt], acc[tt][ct], 0, 0, 0);
            }
            __builtin_amdgcn_sched_barrier(0);
        }
    };

    constexpr int D = NSTAGE - 1;                               // prefetch distance in steps
    const int n_chunks = n_slabs / SPC;
    if constexpr (SPC == 1) {
#pragma unroll
        for (int u = 0; u < D; ++u)
            if (u < n_slabs) { issue_basis(u, u); issue_x(u, u); }
        if (pads) wait_vmem_times<NV_MIN + NX_MIN>(min(D - 1, n_slabs - 1)); else wait_vmem_times<NV_ALL + NX_MIN>(min(D - 1, n_slabs - 1));       // stage 0 has landed, and the tables before it
    } else {
        // in the order of the loop's steps, which D of them would have been in front of it: a slab of X goes out behind the basis of step SPC * c - SPC + D
        if (SPC > D) issue_x(0, 0);
#pragma unroll
        for (int t = -D; t < 0; ++t) {
            if (t + D < n_slabs) issue_basis(t + D, t + D);
            if (t == -SPC) issue_x(0, 0);
        }
        wait_vmem<0>();
    }
    __syncthreads();

    // ---- accumulators start at -(mu^T V_kept): centring folded into the product ------
    {
        const float* negc = reinterpret_cast<const float*>(work) + kEncNegcOff / 4 + ct0 * 32 + 16 * h;
#pragma unroll
        for (int ct = 0; ct < NTW; ++ct) {
            f32x16 c;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const float4 v = *reinterpret_cast<const float4*>(negc + ct * 32 + 4 * q);
                c[4 * q] = v.x; c[4 * q + 1] = v.y; c[4 * q + 2] = v.z; c[4 * q + 3] = v.w;
            }
#pragma unroll
            for (int tt = 0; tt < TT; ++tt) acc[tt][ct] = c;
        }
    }
    constexpr int UNROLL = SPC == 1 ? NSTAGE : enc_common(NSTAGE, 2 * SPC);
    for (int s0 = 0; s0 < n_slabs; s0 += UNROLL) {
#pragma unroll
        for (int u = 0; u < UNROLL; ++u) {
            const int s = s0 + u;
            if (s < n_slabs) {
                // stage (u + D) % NSTAGE was read in step s - 1; the barrier that ended it frees it, and so the other X slab at a slab's end
                if (s + D < n_slabs) issue_basis(s + D, (u + D) % NSTAGE);
                if constexpr (SPC == 1) {
                    if (s + D < n_slabs) issue_x(s + D, (u + D) % NSTAGE);
                    compute(u, u, 0);
                    const int later = min(D - 1, n_slabs - 2 - s);
                    if (pads) wait_vmem_times<NV_MIN + NX_MIN>(later); else wait_vmem_times<NV_ALL + NX_MIN>(later);   // stage of step s + 1 has landed
                } else {
                    const bool more = s / SPC + 1 < n_chunks;
                    if (u % SPC == 0 && more) issue_x(s / SPC + 1, (u / SPC + 1) & 1);
                    compute(u % NSTAGE, (u / SPC) & 1, (u % SPC) * KS);
                    // the basis of step s + 1 has landed and, in front of a new slab of X, that: what is younger may be in flight
                    if (!(more && s + D < n_slabs)) wait_vmem<0>();
                    else if (pads) wait_vmem_dyn(enc_in_flight(u, D, SPC, NV_MIN, NX_MIN));      // (constants: the loop is unrolled)
                    else wait_vmem_dyn(enc_in_flight(u, D, SPC, NV_ALL, NX_MIN));
                }
                __syncthreads();
            }
        }
    }

    encode_epilogue<NTW, TT, false>(acc, ct0, n_ct, wt * TT, TOK_WG, TOK_WG, NTP, NTH, P, tr, a, tok_tile0, work, smem);
}

// One kernel per variant (WC waves across coordinates, NTW coordinate tiles per wave, NW waves per
// workgroup): plans of up to 320 padded coordinates fit 4-wave workgroups with 256 registers per lane,
// two per compute unit (one hides the other's memory waits and epilogue); wider plans get the compute
// unit to themselves, as 8 waves of 256 registers.  A batched launch serves only the jobs
// whose plan uses its variant.
// (must agree with the host's variant table)
template <int WC, int NTW, int NW> constexpr int enc_wgs_per_cu() {
    return NW != 4 ? 1 : (WC == 2 && NTW == 3 ? 3 : 2);
}

template <int NTW, typename XT, int TT, int TOK, int AHEAD, bool BULK>
__device__ __forceinline__ void encode_register_tile(const PlanEnc& P, const TileRef& tr, const KernelArgs& a, uint4* work, bool once);

template <typename XT, int WC, int NTW, int NW>
__global__ void __launch_bounds__(NW * 64, (enc_wgs_per_cu<WC, NTW, NW>())) kvtc_encode_kernel(const KernelArgs a) {
    extern __shared__ uint4 smem[];
    uint32_t* tile_start = reinterpret_cast<uint32_t*>(smem);
    uint4* work = smem + kJobTableBytes / 16 + 1;
    const TileTable table = build_tile_table<true, NW * 64>(a, NW * 10000 + WC * 100 + NTW, tile_start, reinterpret_cast<uint32_t*>(work));
    const TileRange mine = my_tiles(table.total);
    const bool once = table.pass;
    for (uint32_t tile = mine.first; tile < mine.end; tile += mine.step) {
        const TileRef tr = find_tile(a, tile_start, tile);
        const PlanEnc P = load_plan_enc<false>(a.plans + tr.plan);
        if constexpr (WC == 8)
            encode_register_tile<NTW, XT, enc_tt(NTW * WC, NW, WC), 32 * enc_tt(NTW * WC, NW, WC), 4, true>(P, tr, a, work, once);
        else if (enc_once<XT, NTW * WC>() && once) encode_tile<NTW, WC, XT, NW, enc_once<XT, NTW * WC>()>(P, tr, a, work);
        else encode_tile<NTW, WC, XT, NW, false>(P, tr, a, work);
    }
}

// Short jobs: a workgroup per tile of 64 tokens, a wave per coordinate tile (NTW = 2: per two), one kernel for plans of every
// width up to 10 (20) tiles -- the waves a plan does not need help to fetch X.  A launch of a few such tiles is bound by how
// fast a compute unit can draw the plan's basis (half a megabyte at 256 coordinates) through itself, and each fragment is used by one
// wave only, so the fragments go straight to registers, 16 KiB of them in flight per wave (16 k-steps ahead), instead of through an LDS
// ring shared by barriers; X comes in chunks of 256 (fp32: 128) features, asynchronously, with one barrier per chunk.  The sums run over the
// features in the bulk kernel's order: a token's record is the same bits whichever kernel codes it.
// 64 caches of 16 tokens with a basis each (32 MB of bases): 60 us in two launches of ring kernels before, 14 in one; 48 tokens of one
// tensor: 18 -> 14.  (Both have their tiles' groups shared out now, further down: 10 and 8.)
// Tiles of 128 tokens, a workgroup to a compute unit, which draw half as much of the basis: 17000 and 32768 tokens of 240 coordinates 25.7 -> 22.6 and 29.1 -> 28.0 us,
// of 192 22.8 -> 22.4 and 26.4 -> 26.5, fp32 of 240 31.6 -> 31.9 and 36.3 -> 38.4, heads of 128 features 6.4 -> 7.7: the gain is for one width of one type.
// (A chunk is 512 bytes of a token in either type, so that two workgroups' chunks fit a compute unit's LDS: with 1 KiB in fp32 only one
// did, and launches of more tiles than compute units ran a second round: 20000 tokens of 240 coordinates 38 us, now 31.)
template <typename XT> constexpr int short_feat() { return 512 / (int)sizeof(XT); }
template <int NTW> constexpr int short_ahead() { return NTW == 1 ? 16 : 4; }   // k-steps of fragments in flight
constexpr int kShortThreads = 640;

// BULK: the same as the bulk kernels' tile of plans of more than 20 tiles, those shared out evenly among 8 waves (NTW of them or one fewer).  By way of LDS
// the basis of 1024 coordinates came into a compute unit at 26 bytes a cycle, 1300 cycles for a k-step whose matrix instructions take 512; it comes
// twice as fast so.  1024 of 4096 features, two sections of 32768 tokens, both ways: 1268 -> 1164 us, with X (once: an input of
// encode_pass_bytes and more) not kept by the caches 1136; 1024 of 1024, 65536 tokens 165 -> 146; 4096 of 8192 in four sections, 1000 tokens, both ways
// 1080 -> 915.
template <int NTW, typename XT, int TT, int TOK, int AHEAD, bool BULK>
__device__ __forceinline__ void encode_register_tile(const PlanEnc& P, const TileRef& tr, const KernelArgs& a, uint4* work, bool once) {
    constexpr int FEAT = short_feat<XT>(), STEPS = FEAT / 16;
    constexpr int UNROLL = AHEAD > STEPS ? AHEAD / STEPS : 1;        // chunks after which a fragment is in the same register again
    constexpr int EB = (int)sizeof(XT), ROW_B = FEAT * EB, COLS = ROW_B / 16, ROWS_DMA = 1024 / ROW_B;
    constexpr int ROWS = 32 * TT, CHUNK_B = TOK * ROW_B;
    static_assert(UNROLL * STEPS % AHEAD == 0, "a fragment's register is known at compile time");
    int tid = (int)threadIdx.x;
    asm volatile("" : "+v"(tid));            // (lane addresses are worked out here, not kept through a loop over tiles)
    const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), n_waves = (int)blockDim.x >> 6;
    const int l32 = lane & 31, h = lane >> 5;
    const int ntp = BULK ? 8 * NTW : P.enc_ntw * P.enc_wc;
    const int p = P.p, T = tr.n_tokens, tok_tile0 = tr.tile * TOK;
    const int n_steps = p / 16, n_chunks = (p + FEAT - 1) / FEAT;
    const int nt = (P.r + 31) / 32;
    const int ct0 = BULK ? wave * (nt / 8) + min(wave, nt % 8) : wave * NTW;
    const int n_ct = BULK ? nt / 8 + (wave < nt % 8 ? 1 : 0) : min(max(nt - ct0, 0), NTW);      // (a wave without a tile only helps)
    const bool full = !BULK || n_ct >= NTW;
    uint4* smem = work + enc_aux_bytes(ntp) / 16;

    // the plan's tables and chunk 0 of X -> LDS
    {
        const uint32_t aux = lds_offset(work);
        if (wave == 0) dma4_async(P.blk, (uint32_t)lane * 4u, aux + kEncBlkOff);
        if (wave == 1) dma4_async(P.grp, (uint32_t)lane * 4u, aux + kEncGrpOff);
        if (wave * 64 < ntp * 8 && tid < ntp * 8) dma16_async(P.negc, (uint32_t)tid * 16u, aux + kEncNegcOff + (uint32_t)wave * 1024u);
    }
    const int blk_lg = a.x_blk_log2;
    const int64_t blk_jump_b = a.x_blk_jump * EB;
    const uint32_t lds_x = lds_offset(smem);
    auto issue_x = [&](int c) {
        for (int i = wave; i < ROWS / ROWS_DMA; i += n_waves) {
            const int row = i * ROWS_DMA + lane / COLS;
            // 16-byte columns of a row are permuted so that the 8 lanes (rows) served together by a 128-bit read meet 8 bank groups
            const int col = (lane % COLS) ^ (row & 7);
            int f = c * FEAT + col * (16 / EB);
            f = f < p ? f : 0;                                       // behind the last feature: read something, it is not used
            const int t = min(tok_tile0 + row, T - 1);               // rows past the end re-read the last token
            const char* src = reinterpret_cast<const char*>(a.x) + ((tr.x_row0 + t) * a.ld_x + f) * EB + (blk_lg ? (int64_t)(f >> blk_lg) * blk_jump_b : (int64_t)0);
            const uint32_t to = __builtin_amdgcn_readfirstlane(lds_x + (uint32_t)((c & 1) * CHUNK_B + i * 1024));
            if (BULK && once) dma16_async_once(src, to); else dma16_async(src, to);
        }
    };
    issue_x(0);

    // fragments of the wave's tiles, AHEAD k-steps of them in registers (past the end the last ones again, so that the number of
    // loads in flight is always the same; waves without a tile load the first one's)
    u32x4 af[AHEAD][NTW];
    typedef const char __attribute__((address_space(1))) * global_ptr;
    typedef const u32x4 __attribute__((address_space(1))) * global_u4;
    const uint64_t vg = (uint64_t)uniform_ptr(P.v_enc + (n_ct > 0 ? ct0 : 0) * 64);
    auto fetch = [&](int step, int slot) {
        const global_ptr src = (global_ptr)(vg + (uint64_t)(uint32_t)min(step, n_steps - 1) * (uint64_t)(uint32_t)(ntp * 1024));      // a scalar address
#pragma unroll
        for (int i = 0; i < NTW; ++i) af[slot][i] = *(global_u4)(src + (uint32_t)(lane * 16) + (NTW <= 2 || BULK ? i : min(i, max(n_ct - 1, 0))) * 1024);      // (two tiles to a wave are whole pairs)
    };
#pragma unroll
    for (int k = 0; k < AHEAD; ++k) fetch(k, k);
    asm volatile("" ::: "memory");
    wait_vmem<AHEAD * NTW>();                                        // everything older than the fragments has landed
    __syncthreads();

    f32x16 acc[TT][NTW];
    {
        const float* negc = reinterpret_cast<const float*>(work) + kEncNegcOff / 4 + (n_ct > 0 ? ct0 : 0) * 32 + 16 * h;
#pragma unroll
        for (int ct = 0; ct < NTW; ++ct) {
            f32x16 c;
#pragma unroll
            for (int q = 0; q < 16; ++q) c[q] = negc[ct * 32 + q];
#pragma unroll
            for (int tt = 0; tt < TT; ++tt) acc[tt][ct] = c;
        }
    }
    // a k-step's piece of a row: the permutation touches the column's lowest 3 bits, so four lane addresses serve all k-steps (fp32: two,
    // the other column of a pair is one bit away: four are two registers too many)
    constexpr int XOFF = EB == 2 ? 4 : 2;
    uint32_t xoff[XOFF];
#pragma unroll
    for (int j = 0; j < XOFF; ++j) {
        const int col = EB == 2 ? 2 * j + h : 4 * j + 2 * h;
        xoff[j] = (uint32_t)(l32 * ROW_B + (col ^ (l32 & 7)) * 16);
    }
    auto xfrag = [&](const char* x, int tt, int ks) {
        const char* r = x + tt * 32 * ROW_B;
        if constexpr (EB == 2) {
            return as_bf16x8(*reinterpret_cast<const uint4*>(r + xoff[ks & 3] + (ks >> 2) * 128));
        } else {
            const float4 u = *reinterpret_cast<const float4*>(r + xoff[ks & 1] + (ks >> 1) * 128);
            const float4 w = *reinterpret_cast<const float4*>(r + (xoff[ks & 1] ^ 16u) + (ks >> 1) * 128);
            bf16x8 v;                                                // round to bf16, nearest even
            v[0] = (__bf16)u.x; v[1] = (__bf16)u.y; v[2] = (__bf16)u.z; v[3] = (__bf16)u.w;
            v[4] = (__bf16)w.x; v[5] = (__bf16)w.y; v[6] = (__bf16)w.z; v[7] = (__bf16)w.w;
            return v;
        }
    };
    bf16x8 xv[2][TT];                                                // of this k-step and of the next
    auto step = [&](const char* x, int c, int slot0, int ks, bool last) {      // slot0: where the chunk's first fragment is
#pragma unroll
        for (int tt = 0; tt < TT; ++tt)
            if (!last) xv[(ks + 1) & 1][tt] = xfrag(x, tt, ks + 1);
#pragma unroll
        for (int ct = 0; ct < NTW; ++ct)
            if (ct + 1 < NTW || full) {
#pragma unroll
                for (int tt = 0; tt < TT; ++tt)
                    acc[tt][ct] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, af[(slot0 + ks) % AHEAD][ct]), xv[ks & 1][tt], acc[tt][ct], 0, 0, 0);
            }
        fetch(c * STEPS + ks + AHEAD, (slot0 + ks) % AHEAD);
        __builtin_amdgcn_sched_barrier(0);
    };
    const int n_full = p / FEAT;
    for (int c0 = 0; c0 < n_full; c0 += UNROLL) {
#pragma unroll
        for (int u = 0; u < UNROLL; ++u) {
            const int c = c0 + u;
            if (c >= n_full) break;
            const char* x = reinterpret_cast<const char*>(smem) + (c & 1) * CHUNK_B;
            const bool more = c + 1 < n_chunks;
            if (more) issue_x(c + 1);                                // its half was read in chunk c - 1; the barrier that ended it frees it
#pragma unroll
            for (int tt = 0; tt < TT; ++tt) xv[0][tt] = xfrag(x, tt, 0);
#pragma unroll
            for (int ks = 0; ks < STEPS; ++ks) step(x, c, u * STEPS, ks, ks + 1 == STEPS);
            asm volatile("" ::: "memory");
            if (more) wait_vmem<(STEPS * NTW < 63 ? STEPS * NTW : 63)>();                      // the next chunk is older than this one's fragment loads: it has landed
            __syncthreads();
        }
    }
    if (n_full < n_chunks) {                                         // 64 features are left, or (bf16) 128 or 192
        const char* x = reinterpret_cast<const char*>(smem) + (n_full & 1) * CHUNK_B;
        const int left = n_steps - n_full * STEPS;
        auto rest = [&](int slot0) {
#pragma unroll
            for (int g = 0; g < STEPS / 4 - 1; ++g)
                if (4 * g < left) {
#pragma unroll
                    for (int tt = 0; tt < TT; ++tt) xv[0][tt] = xfrag(x, tt, 4 * g);
#pragma unroll
                    for (int ks = 4 * g; ks < 4 * g + 4; ++ks) step(x, n_full, slot0, ks, ks == 4 * g + 3);
                }
        };
        static_assert(UNROLL <= 2, "the register of the rest's first fragment: one of two");
        if (UNROLL == 2 && (n_full & 1)) rest(STEPS); else rest(0);
        __syncthreads();
    }
    wait_vmem<0>();                                                  // the fragments fetched past the end
    encode_epilogue<NTW, TT, !BULK>(acc, ct0, n_ct, 0, ROWS, TOK, ntp, (int)blockDim.x, P, tr, a, tok_tile0, work, smem);
}

// A share of the groups of a tile of 32 tokens.  A launch of a few tiles is bound by what one compute unit can draw (half a megabyte of basis at 256 coordinates, and
// X) and by the round trips it takes to do that.  Groups are quantised each for themselves and own their bytes of a record, so where there are compute
// units enough, workgroups of their own code a tile's groups, a coordinate tile to a wave, and each draws a share of the basis; all of X, which is small, is asked for at
// once, so that the main loop has no barrier, and AHEAD k-steps of fragments.  Sums and roundings are the bulk kernels', and so are the bits.  One tensor of 48
// tokens, 240 coordinates: 12.9 us as a tile of 64 tokens of the short-job kernel, 12.3 in three shares of that tile, 7.8 so; of 528 coordinates 20.3 and 9.9; an
// append step of 64 tensors with 16 tokens each 13.3 and 9.7 (10.3 in up to three shares, for four).
template <typename XT, int AHEAD>
__device__ __forceinline__ void encode_part_tile(const PlanEnc& P, const EncPart& part, const TileRef& tr, const KernelArgs& a, uint4* work) {
    constexpr int FEAT = short_feat<XT>(), STEPS = FEAT / 16;
    constexpr int EB = (int)sizeof(XT), ROW_B = FEAT * EB, COLS = ROW_B / 16, ROWS_DMA = 1024 / ROW_B;
    constexpr int ROWS = kEncPartTile, CHUNK_B = ROWS * ROW_B;
    static_assert(AHEAD % STEPS == 0 || STEPS % AHEAD == 0, "a round of the main loop is whole chunks, or within one");
    const int tid = (int)threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), n_waves = (int)blockDim.x >> 6;
    const int l32 = lane & 31, h = lane >> 5;
    const int ntp = P.enc_ntw * P.enc_wc;
    const int p = P.p, T = tr.n_tokens, tok_tile0 = tr.tile * kEncPartTile, n_valid = min(T - tok_tile0, ROWS);
    const int n_steps = p / 16, n_chunks = (p + FEAT - 1) / FEAT;
    const int ct0 = min(part.ct0 + wave, part.ct1 - 1), n_ct = part.ct0 + wave < part.ct1 ? 1 : 0;      // (a wave without a tile only helps)
    uint4* smem = work + enc_aux_bytes(ntp) / 16;
    {
        const uint32_t aux = lds_offset(work);
        if (wave == 0) dma4_async(P.blk, (uint32_t)lane * 4u, aux + kEncBlkOff);
        if (wave == 1) dma4_async(P.grp, (uint32_t)lane * 4u, aux + kEncGrpOff);
        for (int w = wave; w * 64 < ntp * 8; w += n_waves)
            if (w * 64 + lane < ntp * 8) dma16_async(P.negc, (uint32_t)(w * 64 + lane) * 16u, aux + kEncNegcOff + (uint32_t)w * 1024u);
    }
    const uint32_t lds_x = lds_offset(smem);
    for (int i = wave; i < n_chunks * (ROWS / ROWS_DMA); i += n_waves) {
        const int c = i / (ROWS / ROWS_DMA), row = i % (ROWS / ROWS_DMA) * ROWS_DMA + lane / COLS;
        const int col = (lane % COLS) ^ (row & 7);                   // (permuted as in encode_register_tile)
        int f = c * FEAT + col * (16 / EB);
        f = f < p ? f : 0;                                           // behind the last feature: read something, it is not used
        if (i % (ROWS / ROWS_DMA) * ROWS_DMA >= n_valid) continue;   // (rows past the end are whatever the LDS holds: nothing of theirs is used)
        const int t = min(tok_tile0 + row, T - 1);
        const char* src = reinterpret_cast<const char*>(a.x) + ((tr.x_row0 + t) * a.ld_x + f) * EB + (a.x_blk_log2 ? (int64_t)(f >> a.x_blk_log2) * a.x_blk_jump * EB : (int64_t)0);
        dma16_async(src, __builtin_amdgcn_readfirstlane(lds_x + (uint32_t)(i * 1024)));
    }
    u32x4 af[AHEAD];
    typedef const char __attribute__((address_space(1))) * global_ptr;
    typedef const u32x4 __attribute__((address_space(1))) * global_u4;
    const uint64_t vg = (uint64_t)uniform_ptr(P.v_enc + ct0 * 64);
    auto fetch = [&](int step, int slot) {
        const global_ptr src = (global_ptr)(vg + (uint64_t)(uint32_t)min(step, n_steps - 1) * (uint64_t)(uint32_t)(ntp * 1024));      // a scalar address
        af[slot] = *(global_u4)(src + (uint32_t)(lane * 16));
    };
    asm volatile("" ::: "memory");
#pragma unroll
    for (int k = 0; k < AHEAD; ++k) fetch(k, k);
    asm volatile("" ::: "memory");
    wait_vmem<AHEAD>();                                              // everything older than the fragments has landed
    __syncthreads();

    f32x16 acc[1][1];
    {
        const float* negc = reinterpret_cast<const float*>(work) + kEncNegcOff / 4 + ct0 * 32 + 16 * h;
#pragma unroll
        for (int q = 0; q < 16; ++q) acc[0][0][q] = negc[q];
    }
    auto xfrag = [&](const char* x, int ks) {
        const char* r = x + l32 * ROW_B;
        if constexpr (EB == 2) {
            return as_bf16x8(*reinterpret_cast<const uint4*>(r + (((2 * ks + h) ^ (l32 & 7)) * 16)));
        } else {
            const float4 u = *reinterpret_cast<const float4*>(r + (((4 * ks + 2 * h) ^ (l32 & 7)) * 16));
            const float4 w = *reinterpret_cast<const float4*>(r + (((4 * ks + 2 * h + 1) ^ (l32 & 7)) * 16));
            bf16x8 v;                                                // round to bf16, nearest even
            v[0] = (__bf16)u.x; v[1] = (__bf16)u.y; v[2] = (__bf16)u.z; v[3] = (__bf16)u.w;
            v[4] = (__bf16)w.x; v[5] = (__bf16)w.y; v[6] = (__bf16)w.z; v[7] = (__bf16)w.w;
            return v;
        }
    };
    // one round: AHEAD steps, and (MORE) the fragments of as many after them
    const char* x = reinterpret_cast<const char*>(smem);
    auto round = [&](int s0, auto more_tag) {
        constexpr bool MORE = decltype(more_tag)::value;
        const int k0 = AHEAD % STEPS == 0 ? 0 : s0 % STEPS;
#pragma unroll
        for (int g = 0; g < AHEAD / 4; ++g) {                        // (features come in multiples of 64: four k-steps)
            if (!MORE && s0 + 4 * g >= n_steps) continue;
            const char* xc = x + (s0 / STEPS + 4 * g / STEPS) * CHUNK_B;
            bf16x8 xv[4];
#pragma unroll
            for (int k = 0; k < 4; ++k) xv[k] = xfrag(xc, k0 + (4 * g + k) % STEPS);
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                acc[0][0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, af[4 * g + k]), xv[k], acc[0][0], 0, 0, 0);
                if constexpr (MORE) fetch(s0 + 4 * g + k + AHEAD, 4 * g + k);
            }
            __builtin_amdgcn_sched_barrier(0);
        }
    };
    int s0 = 0;
    for (; s0 + AHEAD < n_steps; s0 += AHEAD) round(s0, std::true_type());
    round(s0, std::false_type());                                    // (nothing to come: of 64 steps, 32 ahead, a third of all the fragments were fetched for nothing)
    wait_vmem<0>();                                                  // the fragments fetched past the end
    __syncthreads();
    encode_epilogue<1, 1, true, true>(acc, ct0, n_ct, 0, n_valid, ROWS, ntp, (int)blockDim.x, P, tr, a, tok_tile0, work, smem, part);
}

// the lane's number, worked out where it is used and not kept through a loop
__device__ __forceinline__ uint32_t lane_id() {
    uint32_t lane = __builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u));
    asm volatile("" : "+v"(lane));
    return lane;
}

// A batch whose jobs all together are few enough tiles for one round of this kernel -- the host knows from the size of the stream buffer, the
// jobs' lengths are on the device -- is coded by this launch alone.  The tiles of all jobs are numbered through; every wave finds its
// workgroup's by a prefix sum over the jobs' tiles, a job per lane and round (bounded by the load and six lane exchanges).  Workgroups go
// round-robin over the eight XCDs, each of which takes an eighth of the tiles, neighbours: the tiles of a job share an L2 and its basis.
// (With a launch per bulk variant, which found no job, in front of it: an append step of 64 tensors 21.8 us, then 16.4 (13.5 with groups shared out); a head of 4096
// tokens in fp32, encode and decode, 24.0, now 17.9, two of it by the decode's tiles.)
// KEEP: the lane's number, and with it the addresses of its jobs, may be kept through the loop over tiles.  In fp32 there are no registers for them:
// with them, and with `upto` left as it is for rounds that a list does not have, up to 18 went to scratch memory, four of them inside the loop over
// chunks.  (12000 tokens, us, kept and not: fp32, 240 coordinates 22.2 and 19.5; bf16, 160 coordinates, six waves, 13.4 and 15.4.)
template <bool KEEP, int TILE = kEncShortTile>
struct ShortTable {
    uint32_t tiles[kShortTableJobs / 64], upto[kShortTableJobs / 64];       // of the lane's job in each round: its tiles; those of the jobs up to it
    uint32_t total;
    __device__ __forceinline__ explicit ShortTable(const KernelArgs& a) {
        const uint32_t lane = KEEP ? (uint32_t)threadIdx.x & 63u : lane_id();
#pragma unroll
        for (int k = 0; k < kShortTableJobs / 64; ++k) {
            const uint32_t j = 64u * k + lane;
            tiles[k] = upto[k] = 0u;
            if (64 * k < a.n_jobs && j < (uint32_t)a.n_jobs) {
                const int n = a.jobs[j].n_tokens;                    // (what else is wrong with a job is seen at its tiles)
                tiles[k] = n > 0 && n <= a.enc_max_tokens ? (uint32_t)(n + TILE - 1) / TILE : 0u;
            }
        }
        total = 0u;
#pragma unroll
        for (int k = 0; k < kShortTableJobs / 64; ++k) {
            if (64 * k >= a.n_jobs) break;
            upto[k] = total + wave_inclusive_scan(tiles[k]);
            total = (uint32_t)__builtin_amdgcn_readlane((int)upto[k], 63);
        }
    }
    // job and tile inside it of the tile with this number; false: there is none
    __device__ __forceinline__ bool find(const KernelArgs& a, uint32_t number, TileRef& tr) const {
        tr.job = tr.tile = 0;
        if (number >= total) return false;
#pragma unroll
        for (int k = 0; k < kShortTableJobs / 64; ++k) {
            if (64 * k >= a.n_jobs) break;
            const uint64_t beyond = __ballot(upto[k] > number);
            if (beyond != 0ull) {
                const int l = __builtin_ctzll(beyond);
                tr.job = 64 * k + l;
                tr.tile = (int)(number - (uint32_t)__builtin_amdgcn_readlane((int)(upto[k] - tiles[k]), l));
                break;
            }
        }
        return true;
    }
};

// the lowest job that cannot be coded -> *status, as the bulk launches report it; one wave
__device__ inline void report_bad_job(const KernelArgs& a) {
    const int lane = (int)threadIdx.x & 63;
    for (int base = 0; base < a.n_jobs; base += 64) {
        const int j = base + lane;
        const uint64_t bad = __ballot(j < a.n_jobs && !job_ok(a, j, a.jobs[j < a.n_jobs ? j : 0]));
        if (bad != 0ull) {
            if (lane == 0) *a.status = (uint32_t)(base + __builtin_ctzll(bad)) + 1u;
            return;
        }
    }
}

// Workgroup `number`'s tile of one tensor or of short jobs, or, TABLE, the tile that tr names; false: none for this kernel.
// A job that is not short, not of this kernel's plans or not valid is left alone (the bulk launches in front of this one, or the last
// workgroup, report it).
template <int NTW, bool TABLE, int TILE = kEncShortTile>
__device__ __forceinline__ bool short_tile(const KernelArgs& a, uint32_t number, TileRef& tr, PlanEnc& P) {
    if constexpr (!TABLE) tr = TileRef{0, a.single.plan, a.single.n_tokens, a.single.x_row0, 0ull, (int32_t)number};
    if (TABLE || a.jobs) {
        if constexpr (!TABLE) {
            // the first tiles of all jobs come first: they spread over the XCDs, and workgroups that find no tile wait behind them
            tr.tile = (int)number / a.n_jobs;
            tr.job = (int)number - tr.tile * a.n_jobs;
        }
        const Words4And2 v = sload_x4_x2(a.jobs + tr.job, a.offsets + tr.job);
        tr.plan = (int32_t)v.four[0];
        tr.n_tokens = (int32_t)v.four[1];
        tr.x_row0 = (int64_t)(((uint64_t)v.four[3] << 32) | v.four[2]);
        tr.offset = ((uint64_t)v.two[1] << 32) | v.two[0];
        if (tr.plan < 0 || tr.plan >= a.n_plans || tr.n_tokens <= tr.tile * TILE || (!TABLE && tr.n_tokens > a.enc_short_max)) return false;
    }
    P = load_plan_enc<true>(a.plans + tr.plan);
    if (NTW != 0 && P.enc_short != NTW) return false;
    if (TABLE || a.jobs) {
        // (one branch for the wave, which only this tells the compiler: as a choice per lane it cost the main loop of the wide form 3 %)
        if (!TABLE && __builtin_expect(tr.n_tokens > kEncShortTile, 0) &&
            __builtin_amdgcn_readfirstlane((int)bulk_takes_mid_jobs(a, enc_key(P), (uint32_t)(a.enc_cus * P.enc_wgs))) != 0)
            return false;
        const uint64_t bytes = (uint64_t)tr.n_tokens * (uint64_t)P.rec_dwords * 4ull;
        if (tr.offset > a.cap || bytes > a.cap - tr.offset) return false;
    }
    return true;
}
template <int NTW, typename XT, int AHEAD = short_ahead<NTW>()>
__device__ __forceinline__ void short_tile_code(const PlanEnc& P, const TileRef& tr, const KernelArgs& a, uint4* smem) {
    if (tr.n_tokens - tr.tile * kEncShortTile <= 32) encode_register_tile<NTW, XT, 1, kEncShortTile, AHEAD, false>(P, tr, a, smem, false);
    else encode_register_tile<NTW, XT, 2, kEncShortTile, AHEAD, false>(P, tr, a, smem, false);
}

// By parts: a.enc_split workgroups to a tile, each a share of its plan's groups.
template <typename XT, int AHEAD>
__device__ __forceinline__ void part_code(const PlanEnc& P, const TileRef& tr, const KernelArgs& a, int part, uint4* smem) {
    const PlanDev __attribute__((address_space(4)))* pd = (const PlanDev __attribute__((address_space(4)))*)(uintptr_t)uniform_ptr(a.plans + tr.plan);
    if (part >= pd->enc_parts) return;
    const EncPart ep(pd->enc_part[2 * part], pd->enc_part[2 * part + 1]);
    encode_part_tile<XT, AHEAD>(P, ep, tr, a, smem);
}
// (registers for four waves a SIMD where two workgroups of eight are to share a compute unit)
#define KVTC_SHORT_BOUNDS(NTW) __launch_bounds__(kShortThreads) __attribute__((amdgpu_waves_per_eu((NTW) == 1 ? 4 : 3)))
template <int NTW, typename XT>
__global__ void KVTC_SHORT_BOUNDS(NTW) kvtc_encode_short_kernel(const KernelArgs a) {
    extern __shared__ uint4 smem[];
    TileRef tr;
    PlanEnc P;
    if (short_tile<NTW, false>(a, blockIdx.x, tr, P)) short_tile_code<NTW, XT>(P, tr, a, smem);
}
// EITHER: by parts where the jobs, whose lengths only the device knows, then are one round of workgroups.  With the launch's waves and registers, 16 k-steps ahead (1); of plans
// whose shares are of up to four coordinate tiles, with the four waves and 32 k-steps of the parts, and the short jobs' tiles by one to three to a wave (2).  (An append step of
// 64 tensors at 16x with room for four: 12.0 us as the short-job kernel, 10.5 (1), 9.3 (2), 9.2 in a launch of its own that does not count; of 32 to 96 tokens 15.3, 15.7, 15.5 and 16.8.)
template <int NTW, typename XT, int EITHER>
__global__ void __launch_bounds__(EITHER == 2 ? 256 : kShortThreads) __attribute__((amdgpu_waves_per_eu(EITHER == 2 ? 2 : NTW == 1 && !(EITHER == 1 && sizeof(XT) == 4) ? 4 : 3))) kvtc_encode_small_batch_kernel(const KernelArgs args) {
    extern __shared__ uint4 smem[];
    if (blockIdx.x + 1u == gridDim.x) {
        if (threadIdx.x < 64) report_bad_job(args);
        return;
    }
    if constexpr (EITHER != 0) {
        uint32_t tiles = 0u;                                         // of the lane's jobs
        for (uint32_t j = threadIdx.x & 63u; j < (uint32_t)args.n_jobs; j += 64u) {
            const int n = args.jobs[j].n_tokens;
            tiles += n > 0 && n <= args.enc_max_tokens ? (uint32_t)(n + kEncPartTile - 1) / kEncPartTile : 0u;
        }
        const uint32_t split = (uint32_t)args.enc_split, shares = (uint32_t)__builtin_amdgcn_readlane((int)wave_inclusive_scan(tiles), 63) * split;
        if (shares <= (uint32_t)args.enc_part_most) {
            const uint32_t per_xcd = (shares + 7u) / 8u, i = blockIdx.x / 8u, number = (blockIdx.x & 7u) * per_xcd + i;
            if (i >= per_xcd) return;
            const ShortTable<false, kEncPartTile> t(args);
            TileRef tr;
            PlanEnc P;
            if (t.find(args, number / split, tr) && short_tile<0, true, kEncPartTile>(args, 0u, tr, P)) part_code<XT, EITHER == 2 ? 32 : 16>(P, tr, args, (int)(number % split), smem);
            return;
        }
    }
    // One tile a workgroup, unless jobs overlap in the stream buffer, which is not allowed but ends all the same.  (The arguments are read
    // again for every tile, or the compiler keeps more of them through the loop than there are registers.)
    for (uint32_t i = blockIdx.x / 8u;; i += (gridDim.x - 1u) / 8u) {
        struct Words { uint64_t w[sizeof(KernelArgs) / 8]; } words;
        uint64_t where = (uint64_t)__builtin_amdgcn_kernarg_segment_ptr();
        asm volatile("" : "+s"(where));
#pragma unroll
        for (size_t w = 0; w < sizeof(KernelArgs) / 8; ++w) words.w[w] = reinterpret_cast<const uint64_t __attribute__((address_space(4)))*>(where)[w];
        const KernelArgs a = __builtin_bit_cast(KernelArgs, words);
        TileRef tr;
        PlanEnc P;
        const ShortTable<sizeof(XT) == 2> t(a);
        const uint32_t per_xcd = (t.total + 7u) / 8u;
        if (i >= per_xcd || !t.find(a, (blockIdx.x & 7u) * per_xcd + i, tr)) return;
        const bool last = i + (gridDim.x - 1u) / 8u >= per_xcd;       // (seen at the table of the next one it was half a microsecond)
        if (short_tile<EITHER == 2 ? 0 : NTW, true>(a, 0u, tr, P)) short_tile_code<NTW, XT, EITHER != 2 || NTW == 1 ? short_ahead<NTW>() : NTW == 2 ? 16 : 8>(P, tr, a, smem);
        if (last) return;
    }
}

// k-steps of fragments on their way: with up to four waves a SIMD's registers are one wave's, and 32 are; with more waves 16; and hardly more than there are, which are
// fetched all the same and keep a small call waiting.  (One token of 64, 128 and 320 features, us, 32 ahead whatever there are, 8, 8 and 16, and the short-job kernel:
// 4.4, 4.6 and 5.1; 3.5, 3.8 and 4.5; 4.0, 4.2 and 5.0.)
constexpr int kPartThreads = 640;
inline int part_ahead(int waves, int p) { return p <= 8 * 16 ? 8 : waves > 4 || p <= 32 * 16 ? 16 : 32; }
template <typename XT, int AHEAD>
__global__ void __launch_bounds__(AHEAD == 32 ? 256 : kPartThreads) kvtc_encode_parts_kernel(const KernelArgs a) {
    extern __shared__ uint4 smem[];
    const TileRef tr{0, a.single.plan, a.single.n_tokens, a.single.x_row0, 0ull, (int32_t)(blockIdx.x / (uint32_t)a.enc_split)};
    const PlanEnc P = load_plan_enc<true>(a.plans + tr.plan);
    part_code<XT, AHEAD>(P, tr, a, (int)(blockIdx.x % (uint32_t)a.enc_split), smem);
}
template <typename XT, int AHEAD>
__global__ void __launch_bounds__(AHEAD == 32 ? 256 : kPartThreads) kvtc_encode_small_batch_parts_kernel(const KernelArgs a) {
    extern __shared__ uint4 smem[];
    if (blockIdx.x + 1u == gridDim.x) {
        if (threadIdx.x < 64) report_bad_job(a);
        return;
    }
    const uint32_t split = (uint32_t)a.enc_split;
    for (uint32_t i = blockIdx.x / 8u;; i += (gridDim.x - 1u) / 8u) {
        TileRef tr;
        PlanEnc P;
        const ShortTable<false, kEncPartTile> t(a);
        const uint32_t per_xcd = (t.total * split + 7u) / 8u, number = (blockIdx.x & 7u) * per_xcd + i;
        if (i >= per_xcd || !t.find(a, number / split, tr)) return;
        const bool last = i + (gridDim.x - 1u) / 8u >= per_xcd;
        if (short_tile<0, true, kEncPartTile>(a, 0u, tr, P)) part_code<XT, AHEAD>(P, tr, a, (int)(number % split), smem);
        if (last) return;
    }
}

// (waves across coordinates, coordinate tiles per wave, waves per workgroup); no short-job kernel serves the plans of the last two, so
// these, on 64-token tiles, code jobs of any length
#define KVTC_ENC_VARIANTS(X)                                                                           \
    X(1, 2, 4) X(1, 4, 4) X(2, 3, 4) X(2, 4, 4) X(2, 5, 4) X(4, 3, 8) X(4, 4, 8) X(4, 5, 8) X(8, 3, 8) X(8, 4, 8)

// key = 10000 * NW + 100 * WC + NTW
hipError_t launch_encode(const KernelArgs& a, kvtc_dtype dtype, int key, int grid, size_t lds_bytes, hipStream_t stream) {
    const void* fn = nullptr;
    int threads = 0;
    switch (key) {
#define KVTC_X(WC, NTW, NW)                                                                                    \
    case (NW) * 10000 + (WC) * 100 + (NTW):                                                                    \
        fn = dtype == KVTC_BF16 ? reinterpret_cast<const void*>(&kvtc_encode_kernel<uint16_t, WC, NTW, NW>)    \
                                : reinterpret_cast<const void*>(&kvtc_encode_kernel<float, WC, NTW, NW>);      \
        threads = (NW) * 64;                                                                                   \
        break;
        KVTC_ENC_VARIANTS(KVTC_X)
#undef KVTC_X
        default: return hipErrorInvalidValue;
    }
    hipError_t e = allow_full_lds(fn);
    if (e != hipSuccess) return e;
    KernelArgs args = a;
    void* params[] = {&args};
    return hipLaunchKernel(fn, dim3(grid), dim3(threads), params, lds_bytes, stream);
}

// `grid` workgroups of `waves` waves, one per 64-token tile: those of a single tensor, or of a batch the tiles a short job may have
// times the jobs; ntw: coordinate tiles per wave (the plans' enc_short).
hipError_t launch_encode_short(const KernelArgs& a, kvtc_dtype dtype, int ntw, int waves, int grid, size_t lds_bytes, hipStream_t stream) {
    const void* fn = nullptr;
#define KVTC_X(NTW, XT, EITHER) reinterpret_cast<const void*>(&kvtc_encode_small_batch_kernel<NTW, XT, EITHER>)
#define KVTC_Y(NTW, XT) (a.enc_table ? KVTC_X(NTW, XT, 0) : reinterpret_cast<const void*>(&kvtc_encode_short_kernel<NTW, XT>))
    if (a.enc_part_most != 0 && dtype == KVTC_BF16 && waves == 4) fn = ntw == 1 ? KVTC_X(1, uint16_t, 2) : ntw == 2 ? KVTC_X(2, uint16_t, 2) : KVTC_X(3, uint16_t, 2);
    else if (a.enc_part_most != 0) fn = ntw != 1 ? nullptr : dtype == KVTC_BF16 ? KVTC_X(1, uint16_t, 1) : KVTC_X(1, float, 1);
    else if (ntw == 1) fn = dtype == KVTC_BF16 ? KVTC_Y(1, uint16_t) : KVTC_Y(1, float);
    else if (ntw == 2) fn = dtype == KVTC_BF16 ? KVTC_Y(2, uint16_t) : KVTC_Y(2, float);
#undef KVTC_X
#undef KVTC_Y
    if (!fn || waves < 2 || waves * 64 > kShortThreads) return hipErrorInvalidValue;
    hipError_t e = allow_full_lds(fn);
    if (e != hipSuccess) return e;
    KernelArgs args = a;
    void* params[] = {&args};
    return hipLaunchKernel(fn, dim3(grid), dim3(64 * waves), params, lds_bytes, stream);
}

// `grid` workgroups of `waves` waves: a.enc_split for every tile of a tensor or of a batch, as for launch_encode_short; max_p: features of a token, the most of any plan
hipError_t launch_encode_parts(const KernelArgs& a, kvtc_dtype dtype, int waves, int max_p, int grid, size_t lds_bytes, hipStream_t stream) {
    const void* fn = nullptr;
#define KVTC_X(XT, AHEAD) (a.enc_table ? reinterpret_cast<const void*>(&kvtc_encode_small_batch_parts_kernel<XT, AHEAD>) : reinterpret_cast<const void*>(&kvtc_encode_parts_kernel<XT, AHEAD>))
    switch (part_ahead(waves, max_p)) {
        case 8: fn = dtype == KVTC_BF16 ? KVTC_X(uint16_t, 8) : KVTC_X(float, 8); break;
        case 16: fn = dtype == KVTC_BF16 ? KVTC_X(uint16_t, 16) : KVTC_X(float, 16); break;
        default: fn = dtype == KVTC_BF16 ? KVTC_X(uint16_t, 32) : KVTC_X(float, 32);
    }
#undef KVTC_X
    if (waves < 2 || waves * 64 > kPartThreads || a.enc_split < 1) return hipErrorInvalidValue;
    hipError_t e = allow_full_lds(fn);
    if (e != hipSuccess) return e;
    KernelArgs args = a;
    void* params[] = {&args};
    return hipLaunchKernel(fn, dim3(grid), dim3(64 * waves), params, lds_bytes, stream);
}
int encode_part_waves_most() { return kPartThreads / 64; }
// LDS bytes of a tile of a plan of p features, or 0 where X does not fit
int encode_part_lds_bytes(int p, int ntp, int n_groups, int rec_dwords, kvtc_dtype dtype) {
    const int feat = dtype == KVTC_BF16 ? short_feat<uint16_t>() : short_feat<float>();
    const int main_b = (p + feat - 1) / feat * kEncPartTile * 512;
    const int epi_b = kEncPartTile * (2 * ntp * 8 + n_groups * 8 + (rec_dwords + 1) * 4);
    const int b = enc_aux_bytes(ntp) + (main_b > epi_b ? main_b : epi_b);
    return b <= kLdsBudget ? b : 0;
}

// Coordinate tiles per wave of the short-job kernel for a plan of ntp tiles (0 = none), waves, and LDS bytes.
int encode_short_ntw(int ntp) { return ntp <= 10 ? 1 : (ntp <= 20 ? 2 : 0); }
int encode_short_waves(int ntp) {
    const int n = (ntp + encode_short_ntw(ntp) - 1) / encode_short_ntw(ntp);
    return n < 4 ? 4 : n;
}
int encode_short_lds_bytes(int ntp, int n_groups, int rec_dwords, kvtc_dtype dtype) {
    const int main_b = 2 * kEncShortTile * (dtype == KVTC_BF16 ? short_feat<uint16_t>() * 2 : short_feat<float>() * 4);
    const int epi_b = kEncShortTile * (2 * ntp * 8 + n_groups * 8 + (rec_dwords + 1) * 4);
    return enc_aux_bytes(ntp) + (main_b > epi_b ? main_b : epi_b);
}

// Bytes of a call's features from which on the variant reads them without keeping them.  (The caches keep some of an fp32 input of a little more than
// their size from one call to the next: two tensors of 35000 tokens at 40x, 287 MB, 63 us and 81 without keeping it, of 41000, 336 MB, 84.4 and
// 83.7; bf16: of 67000, 274 MB, 53.9 and 55.5, of 75000, 307 MB, 71 and 64.  bf16 of 4 tiles: its ring by lines has the basis one k-step ahead, which
// shows in launches of one round of tiles or two.  64 tensors of 128 coordinates, one plan and 64, kept and not: of 2100 tokens, 275 MB, 78 88 and 89 102, of 3000 97 97
// and 102.5 106 (375 MB; in another run 100 99 and 111 107), of 5000 171.6 163 and 174 167; one tensor of 140000 82 87, of 180000, 351 MB, 96 92, of 200000 113 107.)
uint64_t encode_pass_bytes(int ntp, kvtc_dtype dtype) {
    const int eb = dtype == KVTC_BF16 ? 2 : 4;
    return ntp > 20 || enc_can_pass(ntp, eb) ? (eb == 4 ? 320ull : ntp == 4 ? 340ull : 256ull) << 20 : ~0ull;
}

int encode_tok_wg(int ntw, int wc, int nw) { return 32 * enc_tt(ntw * wc, nw, wc) * (nw / wc); }

// LDS bytes encode_tile needs for a variant (main loop slabs vs epilogue images).
int encode_lds_bytes(int ntw, int wc, int nw, int n_groups, int rec_dwords, kvtc_dtype dtype) {
    const int ntp = ntw * wc;
    const int eb = dtype == KVTC_BF16 ? 2 : 4;
    const int tok_wg = 32 * enc_tt(ntp, nw, wc) * (nw / wc);
    const int ring_b = enc_ring_bytes(ntp, eb, nw, wc, false), ring_once_b = enc_ring_bytes(ntp, eb, nw, wc, true);
    const int main_b = wc == 8 ? 2 * tok_wg * 512 : (ring_b > ring_once_b ? ring_b : ring_once_b);
    const int epi_b = tok_wg * (2 * ntp * 8 + n_groups * 8 + (rec_dwords + 1) * 4);
    return enc_aux_bytes(ntp) + (main_b > epi_b ? main_b : epi_b);
}

}  // namespace kvtc
