// Fused decode kernel for gfx950, the mirror of the encode kernel: records are unpacked
// and dequantised straight into bf16 matrix-core operands, back-projected with V_kept and
// un-centred, one launch.  (Paper, Section "Method", mode "Decompression"; eq. 3.)
//
// X_hat = D_hat V_kept^T with the 32x32x16 bf16 MFMA: M = tokens, N = features,
// K = kept coordinates.  In the prologue a lane owns one token: its dequantised coordinates ARE
// its A operand (16 consecutive coordinates = one block of the record = two k-step fragments),
// built once per tile and kept in registers while the wave sweeps the feature tiles.
// V_kept is pre-swizzled into B fragments per 32-feature tile, moved global -> LDS without
// register staging (ring of slabs) and shared by the four wavefronts.  The accumulator then has
// features across lanes and tokens across registers.  Feature tiles come in pairs that
// interleave the even and the odd features of a 64-feature span, so a lane packs its two
// results into one dword (bf16) or one dwordx2 (fp32) and every store instruction writes whole
// 128-byte lines of two token rows -- no transposition through LDS (measured on MI355X: such
// dword stores reach the same 5.7 TB/s as 16-byte stores of whole lines, while pieces of
// 32 bytes per row reach 1.6 TB/s).
#include <hip/hip_runtime.h>
#include <type_traits>
#include "kvtc_dev.h"
#include "kvtc_numeric.h"

namespace kvtc {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x2_d __attribute__((ext_vector_type(2)));

__device__ __forceinline__ bf16x8 as_bf16x8_d(uint4 v) { return __builtin_bit_cast(bf16x8, v); }

// Work-area layout in LDS (behind the job table): [block table of the tile's plan, 256 B][record
// image][basis ring].  The ring has two stages; a stage is one 32-feature slab of B fragments
// followed by that tile's 32 entries of mu (kMuU4 * 16 bytes with padding).
constexpr int kDecStages = 2;
constexpr int kMuU4 = 16;
constexpr int kAuxBytes = 256;

__device__ __forceinline__ uint32_t pack_bf16x2(float lo, float hi) {
    typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
    bf16x2 v;
    v[0] = (__bf16)lo;
    v[1] = (__bf16)hi;
    return __builtin_bit_cast(uint32_t, v);
}

// Where the records of a tile sit in the LDS image.  Transfers move 16 bytes per lane (the
// global->LDS path handles a lane at a time, so narrower pieces cost the same and carry less):
//   * records of a whole number of 16-byte pieces, the tile starting on a 16-byte boundary of the
//     stream (it does unless jobs with other record sizes precede it): each row gets an odd number of pieces (one or
//     two of padding), which spreads the rows that 32 lanes unpack side by side over the banks
//     (two lanes per bank at worst);
//   * other record sizes: the tile's bytes are copied as they are, starting from the 16-byte
//     boundary below the tile's first byte (`skew` dwords before it); the row stride is then rd
//     dwords, which is not a multiple of four -- again two lanes per bank at worst.
struct RecImage {
    uint32_t stride_dw;     // LDS dwords from one row to the next
    uint32_t skew_dw;       // LDS dwords before row 0
    uint32_t pieces_row;    // padded scheme: pieces per row, padding included; 0 = verbatim copy
};
__device__ __forceinline__ RecImage rec_image(int rd, uint64_t tile_byte0) {
    RecImage im;
    if ((rd & 3) == 0 && (tile_byte0 & 15u) == 0u) {
        const uint32_t m = (uint32_t)rd >> 2;
        im.pieces_row = (m & 1u) ? m + 2u : m + 1u;
        im.stride_dw = 4u * im.pieces_row;
        im.skew_dw = 0u;
    } else {
        im.pieces_row = 0u;
        im.stride_dw = (uint32_t)rd;
        im.skew_dw = (uint32_t)(tile_byte0 & 15u) >> 2;
    }
    return im;
}

// Records of one workgroup tile (and the block table of its plan), global -> LDS, asynchronously
// and without register staging.  Only the tile's valid rows are fetched; rows past the end of the
// tensor are never read (the unpacking redirects them to the last valid row).  Returns the number
// of transfers this wave issued; the caller owns the wait (vmcnt) and the barrier that publishes
// the image.
template <int NT = kThreads>
__device__ __forceinline__ int issue_records(const KernelArgs& a, const TileRef& t, const PlanDec& P, uint32_t lds_work) {
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int rd = P.rec_dwords, tok_wg = P.dec_tok_wg;
    const int tok0 = t.tile * tok_wg;
    const uint32_t n_valid = (uint32_t)min(tok_wg, t.n_tokens - tok0);
    const uint64_t byte0 = t.offset + (uint64_t)tok0 * (uint64_t)rd * 4ull;
    const RecImage im = rec_image(rd, byte0);
    const uint8_t* src = reinterpret_cast<const uint8_t*>(a.stream_buf) + (byte0 & ~15ull);
    const uint32_t lds_rec = lds_work + kAuxBytes;
    int n = 0;
    if (wave == 0) {
        dma4_async(P.blk, (uint32_t)lane * 4u, lds_work);
        ++n;
    }
    if (im.pieces_row != 0u) {
        const uint32_t m = (uint32_t)rd >> 2;
        const uint32_t total = n_valid * im.pieces_row;          // LDS slots, padding included
        const uint32_t magic = 0xffffffffu / im.pieces_row + 1u;
        for (uint32_t l0 = (uint32_t)wave * 64u; l0 < total; l0 += NT) {
            const uint32_t l = l0 + (uint32_t)lane;
            if (l < total) {
                const uint32_t row = __umulhi(l, magic);
                const uint32_t col = l - row * im.pieces_row;
                dma16_async(src, (row * m + min(col, m - 1u)) * 16u, lds_rec + l0 * 16u);    // padding repeats the last piece
            }
            ++n;
        }
    } else {
        const uint32_t total = (im.skew_dw * 4u + n_valid * (uint32_t)rd * 4u + 15u) >> 4;   // pieces
        for (uint32_t l0 = (uint32_t)wave * 64u; l0 < total; l0 += NT) {
            const uint32_t l = l0 + (uint32_t)lane;
            if (l < total) dma16_async(src, l * 16u, lds_rec + l0 * 16u);
            ++n;
        }
    }
    return n;
}

// A record's block (its width, group and first bit as in the block table): the dwords its 16 codes lie in and its header; then its values as bf16
// pairs (a block without bits gives zeros).  Codes of up to 8 bits (kNarrow) come four to a 32-bit window, wider ones two.  Reading and converting
// are apart, so that the reads of the next block travel under the conversions of this one (in turn, each window waited for its own read).
template <bool kNarrow> struct RecBlock {
    static constexpr int PER = kNarrow ? 4 : 2, N = 16 / PER;      // codes per window, windows
    uint32_t bits, pos0, hdr, lo[N], hi[N];
    __device__ __forceinline__ void read(const uint32_t* row, uint32_t info) {
        bits = info & 0xffu;
        pos0 = (info >> 16) * 16u;
        hdr = row[(info >> 8) & 0xffu];
#pragma unroll
        for (int k = 0; k < N; ++k) {
            const uint32_t dw = (pos0 + (uint32_t)(PER * k) * bits) >> 5;
            lo[k] = row[dw];
            hi[k] = row[dw + 1];
        }
    }
    __device__ __forceinline__ void values(uint32_t (&q)[8]) const {
        const uint32_t head = bits != 0u ? hdr : 0u;
        const float shift = (float)__builtin_bit_cast(_Float16, (uint16_t)head);
        const float scale = (float)__builtin_bit_cast(_Float16, (uint16_t)(head >> 16));
#pragma unroll
        for (int k = 0; k < N; ++k) {
            const uint32_t w = __builtin_amdgcn_alignbit(hi[k], lo[k], (pos0 + (uint32_t)(PER * k) * bits) & 31u);
#pragma unroll
            for (int m = 0; m < PER; m += 2) {
                const float d0 = __fmaf_rn((float)__builtin_amdgcn_ubfe(w, m * bits, bits), scale, shift);
                const float d1 = __fmaf_rn((float)__builtin_amdgcn_ubfe(w, (m + 1) * bits, bits), scale, shift);
                q[(PER * k + m) / 2] = pack_bf16x2(d0, d1);
            }
        }
    }
};


// The earlier sections' sum for accumulator register i of token tile tt: the lane's two features (rows past the end: the last row's).
__device__ __forceinline__ float2 load_part(const char* sb, uint32_t lrow, int tt, int i, uint32_t sld, uint32_t lane_col, uint32_t last_row) {
    const uint32_t row = min(lrow + (uint32_t)(tt * 32 + 8 * (i / 4) + i % 4), last_row);
    return *reinterpret_cast<const float2*>(sb + ((size_t)row * sld + 2u * lane_col));
}

// Bytes of a call's output from which on it passes the caches by (non-temporal stores; whole tiles only; ~0: never).  cls: the kernel class; least_tiles:
// the narrowest of the launch's plans, as it runs; bases: bytes of all their bases; single: one tensor's call.  Output that nobody finds in a cache again
// pushes the bases out of the L2s, 4 MB each, that every workgroup reads them from; but stores that pass the last-level cache, 256 MB, by go no faster
// than HBM, and what is left of the output there is found by who reads or writes it next.  So it pays where matrix work or many bases are in the way,
// and not where the stores are all there is.  us, kept and past the caches, one buffer again and again / buffers in turn:
//   wide plans, both types: 400 coordinates, one tensor of 70000 tokens (137 MB) 92 88 / 94 89; never slower
//   bf16, 7 to 10 tiles: 240 coordinates, 137 MB 63 56 / 64 56, 312 MB 114 89 / 112 91; 64 tensors and plans of 4000 190 121
//   bf16, 5 and 6 tiles: 160, one tensor, 195 MB 51 57 / 54.5 56, 253 MB 61 65 / 66 66, 390 MB 115 111 / 114 110; batches, 4 of 18000 54 53 / 52 48,
//     31 of 4000 73 62 / 66 61; 64 plans, 150 MB 60 61 / 61 58, 500 MB 179 111
//   bf16, 3 and 4 tiles: 80, one tensor, 585 MB 130 143 / 130 142, 781 MB 167 175 / 168 176, 878 MB 207 208 / 205 206; 2 of 100000 (390 MB) 118 102 / 114
//     103, but 8 of 32000 (500 MB) 113 125 / 114 121, and before there were such stores 118 / 118; 2 of 140000 135 134 / 136 136; 31 of 12000 (726 MB) 162 170 / 165 171, 128 179 169 / 178 169
//   bf16, up to 2 tiles: 64, 234 MB 41 57 / 53 58, 600 MB 129 134 / 128 135, 1.2 GB 254 248 / 254 252 (16: 283 298 / 281 288 at 1.4), 2 GB 424 413 / 422 417
//   bf16, up to 4 tiles, many plans: 64, 16 plans (2 MB of bases) 300 MB 73 70 / 72 70, 64 plans 500 MB 150 107
//   fp32, 5 to 10 tiles: 160 to 240, 312 MB 95 116 / 94 111, 898 MB 254 275 / 255 280, 1 GB 254 256 / 253 256 (240: 271 260 / 272 261), 1.1 GB 307 290 / 297 286;
//     8 plans of 240 (4 MB) 300 MB 98 101 / 102 102; 16 (8 MB) 109 99 / 109 102
//   fp32, up to 4 tiles: 64, 470 MB 117 132 / 123 136, 1.6 GB 333 342 / 326 338, 4 GB 828 830 / 837 859; 64 plans (8 MB) 300 MB 97 98 / 93 92, 500 MB 158 135
#if KVTC_DECODE_PART == 0
uint64_t decode_pass_bytes(int cls, int least_tiles, kvtc_dtype dtype, uint64_t bases, bool single) {
    const bool bf16 = dtype == KVTC_BF16, many = bf16 ? bases >= (2u << 20) : bases > (4u << 20);
    uint64_t mib = 129;
    if (cls <= 4) mib = !bf16 ? (many ? 384 : 0) : many ? 256 : least_tiles <= 2 ? 1536 : 840;
    else if (cls <= 10) mib = !bf16 ? (many ? 256 : 1024) : single && least_tiles <= 6 ? 256 : 129;
    return mib ? mib << 20 : ~0ull;
}
#endif

// The results of a pair of feature tiles (acc0: the even, acc1: the odd features of 64-feature span `span`) to the output.  `fast`: every row of
// the tile is one of the tensor's, and with STREAM the output is to pass the caches by.  (Stores of either kind side by side, chosen per tile, cost the
// 16x cache 4 %: tiles that are neither take the form that looks after the rows' end, whose addresses are half of the sweep's vector instructions.)
template <int TT, typename OT, int ACC, bool STREAM>
__device__ __forceinline__ void store_pair(const KernelArgs& a, const TileRef& tr, const f32x16 (&acc0)[TT], const f32x16 (&acc1)[TT], char* obase, int span,
                                           uint32_t lane_row, uint32_t lane_col, uint32_t last_row, int tok_tile0, bool fast) {
    const uint32_t ldb = (uint32_t)a.ld_x * (uint32_t)sizeof(OT);
    // the 64-feature span span of the token's features; with a blocked layout (heads or layers apart in
    // memory) every whole block before it adds the gap between blocks
    char* ob = obase + (size_t)(span) * (64 * sizeof(OT)) +
               (a.x_blk_log2 ? (size_t)(((span) * 64) >> a.x_blk_log2) * ((size_t)a.x_blk_jump * sizeof(OT)) : (size_t)0);
    // (through an empty asm so that the 16*TT offsets are recomputed here -- three vector
    // instructions each -- instead of being hoisted out of the sweep into registers the
    // accumulators need)
    uint32_t lrow = lane_row;
    asm volatile("" : "+v"(lrow));
    if constexpr (ACC == 1) {
        // a further section of a sectioned plan: its part of the product is ADDED to what the earlier
        // sections left in the fp32 output (hardware float adds in memory, nothing returned).  Rows past
        // the tensor's end are skipped, not redirected: adding the last row's values twice would be wrong.
        static_assert(sizeof(OT) == 4, "sections are summed in fp32");
#pragma unroll
        for (int k = 0; k < 16 * TT; ++k) {
            const int tt = k / 16, i = k % 16;
            const uint32_t row = lrow + (uint32_t)(tt * 32 + 8 * (i / 4) + i % 4);
            if (row <= last_row) {
                float* dst = reinterpret_cast<float*>(ob + (__umul24(row, ldb) + lane_col));
                unsafeAtomicAdd(dst, acc0[tt][i]);
                unsafeAtomicAdd(dst + 1, acc1[tt][i]);
            }
        }
    } else if constexpr (ACC == 2) {
        // the last section of a sectioned plan, bf16 output: the earlier sections' fp32 sum (rows of a.dec_sum_ld
        // floats, features contiguous) plus this section's part, rounded to bf16 once and stored at the caller's layout
        static_assert(sizeof(OT) == 2, "the final rounding is to bf16");
        const char* sb = reinterpret_cast<const char*>(a.dec_sum) +
                         ((size_t)(tr.x_row0 + tok_tile0) * (size_t)a.dec_sum_ld + (size_t)(span) * 64) * sizeof(float);
        const uint32_t sld = (uint32_t)a.dec_sum_ld * (uint32_t)sizeof(float);
        constexpr int N = TT == 4 ? 16 : 1;                // sums read at a time: the wide kernel has registers for a tile's
#pragma unroll
        for (int k0 = 0; k0 < 16 * TT; k0 += N) {
            float2 part[N];
#pragma unroll
            for (int k = k0; k < k0 + N; ++k) part[k - k0] = load_part(sb, lrow, k / 16, k % 16, sld, lane_col, last_row);
#pragma unroll
            for (int k = k0; k < k0 + N; ++k) {
                const int tt = k / 16, i = k % 16;
                const uint32_t row = min(lrow + (uint32_t)(tt * 32 + 8 * (i / 4) + i % 4), last_row);
                *reinterpret_cast<uint32_t*>(ob + (__umul24(row, ldb) + lane_col)) = pack_bf16x2(part[k - k0].x + acc0[tt][i], part[k - k0].y + acc1[tt][i]);
            }
        }
    } else if (fast) {
        // no row past the end: a row's address is a scalar and the lane's offset the same for all
        typedef char __attribute__((address_space(1))) * global_ptr;
        typedef std::conditional_t<sizeof(OT) == 2, uint32_t, f32x2_d> V;
        typedef V __attribute__((address_space(1))) * global_v;
        const uint64_t rows = (uint64_t)uniform_ptr(ob);
        const uint32_t lane_off = __umul24(lrow, ldb) + lane_col;          // row < 256, ldb <= 2^23
#pragma unroll
        for (int k = 0; k < 16 * TT; ++k) {
            const int tt = k / 16, i = k % 16;
            const global_v dst = (global_v)((global_ptr)(rows + (uint64_t)(uint32_t)(tt * 32 + 8 * (i / 4) + i % 4) * (uint64_t)ldb) + lane_off);
            V v;
            if constexpr (sizeof(OT) == 2) v = pack_bf16x2(acc0[tt][i], acc1[tt][i]); else v = f32x2_d{acc0[tt][i], acc1[tt][i]};
            if constexpr (STREAM) __builtin_nontemporal_store(v, dst); else *dst = v;
        }
    } else {
#pragma unroll
        for (int k = 0; k < 16 * TT; ++k) {
            const int tt = k / 16, i = k % 16;
            const uint32_t row = min(lrow + (uint32_t)(tt * 32 + 8 * (i / 4) + i % 4), last_row);
            char* dst = ob + (__umul24(row, ldb) + lane_col);              // row < 256, ldb <= 2^23
            if constexpr (sizeof(OT) == 2) *reinterpret_cast<uint32_t*>(dst) = pack_bf16x2(acc0[tt][i], acc1[tt][i]);
            else *reinterpret_cast<float2*>(dst) = make_float2(acc0[tt][i], acc1[tt][i]);
        }
    }
}

// One workgroup tile.  The work area holds the tile's block table and record image, landed and
// published.  With `prefetch` the ring does not overlap them: the first basis slab is requested
// before unpacking, and the records of the workgroup's next tile (if any) are requested during
// the first step of the feature sweep.
template <int NCT, int TT, typename OT, int ACC, bool SHARE>
__device__ __forceinline__ void decode_tile(const PlanDec& P, const TileRef& tr, const KernelArgs& a, uint4* work, uint4* ring,
                                            bool prefetch, bool has_next, const TileRef& next, const PlanDec& Pn, int first_span, bool streamed) {
    constexpr int TOK_W = 32 * TT;
    constexpr int TOK_WG = 4 * TOK_W;
    constexpr int SLAB_U4 = 2 * NCT * 64;          // one 32-feature tile of V_kept
    constexpr int STAGE_U4 = SLAB_U4 + kMuU4;
    constexpr int NV = (SLAB_U4 + kThreads - 1) / kThreads;     // transfer rounds of the workgroup per slab; with an odd tile count the last one is half a round (waves 0 and 1)
    static_assert(SLAB_U4 % 128 == 0, "whole wave transfers");
    static_assert(kDecStages == 2, "the wait counts below are written out for a ring of two slabs");

    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l32 = lane & 31, h = lane >> 5;
    const int T = tr.n_tokens;
    const int tok_tile0 = tr.tile * TOK_WG;
    const int rd = P.rec_dwords;
    const int n_valid = min(TOK_WG, T - tok_tile0);
    const RecImage im = rec_image(rd, tr.offset + (uint64_t)tok_tile0 * (uint64_t)rd * 4ull);
    const int n_ft = P.p / 32;                                 // even: p is a multiple of 64

    // basis slab of feature tile ft -> ring stage; wave 0 also moves the tile's mu entries
    const uint4* vg = P.v_dec;
    const uint32_t lds_ring = lds_offset(ring);
    auto issue_slab = [&](int ft, int stage) {
        const uint4* vsrc = vg + (size_t)ft * STAGE_U4;
        const uint32_t dst = lds_ring + (uint32_t)(stage * STAGE_U4) * 16u;
#pragma unroll
        for (int i = 0; i < NV; ++i)
            if ((i + 1) * kThreads <= SLAB_U4 || i * kThreads + wave * 64 < SLAB_U4)
                dma16_async(vsrc + i * kThreads, (uint32_t)tid * 16u, dst + (uint32_t)(i * kThreads + wave * 64) * 16u);
        if (wave == 0 && lane < kMuU4) dma16_async(vsrc + SLAB_U4, (uint32_t)lane * 16u, dst + (uint32_t)SLAB_U4 * 16u);
    };
    if (prefetch) issue_slab(0, 0);

    // ---- each lane unpacks its blocks from the record image ------------------------------
    // A lane owns one token (l32) and, per 32-coordinate tile, the 16-coordinate block of its half h.
    const uint32_t* blk = reinterpret_cast<const uint32_t*>(work);
    const uint32_t* rec = blk + kAuxBytes / 4 + im.skew_dw;
    bf16x8 aop[TT][2 * NCT];
    // codes of up to 8 bits (all that calibration produces) come four to a 32-bit window, wider
    // ones two; the choice is made once per plan
    auto unpack = [&](auto narrow_tag) {
        const uint32_t* row[TT];
#pragma unroll
        for (int tt = 0; tt < TT; ++tt)
            row[tt] = rec + (uint32_t)min(wave * TOK_W + tt * 32 + l32, n_valid - 1) * im.stride_dw;   // tail rows: the last token's record
        uint32_t info[NCT];
#pragma unroll
        for (int c = 0; c < NCT; ++c) info[c] = blk[2 * c + h];
        RecBlock<decltype(narrow_tag)::value> b[2];              // this item's and the next one's
        b[0].read(row[0], info[0]);
#pragma unroll
        for (int k = 0; k < NCT * TT; ++k) {
            const int c = k / TT, tt = k % TT;
            if (k + 1 < NCT * TT) b[(k + 1) & 1].read(row[(k + 1) % TT], info[(k + 1) / TT]);
            __builtin_amdgcn_sched_barrier(0);
            uint32_t q[8];                                      // the block's 16 values as bf16 pairs
            b[k & 1].values(q);
            // (through an empty asm: the conversions are done here, block by block, instead of all the
            // fp32 values staying live until the end of the unpacking)
            asm volatile("" : "+v"(q[0]), "+v"(q[1]), "+v"(q[2]), "+v"(q[3]), "+v"(q[4]), "+v"(q[5]), "+v"(q[6]), "+v"(q[7]));
            aop[tt][2 * c] = __builtin_bit_cast(bf16x8, make_uint4(q[0], q[1], q[2], q[3]));
            aop[tt][2 * c + 1] = __builtin_bit_cast(bf16x8, make_uint4(q[4], q[5], q[6], q[7]));
        }
    };
    if (P.code_bits_max <= 8) unpack(std::true_type()); else unpack(std::false_type());
    if (!prefetch) {
        __syncthreads();          // record image is dead; the ring reuses its space
        issue_slab(0, 0);
    }
    wait_vmem<0>();
    __syncthreads();              // slab 0 is published (and, with prefetch, the record image is dead)

    // ---- sweep the feature tiles --------------------------------------------------------
    // Output addressing.  Accumulator register i of token tile tt holds row tt*32 + 8*(i/4) + 4*h + i%4
    // of this wave's tokens; the lane's two features of a pair of tiles are adjacent in memory.
    // Rows past the end of the tensor are redirected to the last token's row (they hold its values),
    // so no store is ever predicated off and the number of memory operations per step is fixed.
    constexpr int NST = 16 * TT;                               // stores per pair of feature tiles
    char* obase = reinterpret_cast<char*>(const_cast<void*>(a.x)) + (size_t)(tr.x_row0 + tok_tile0) * (size_t)a.ld_x * sizeof(OT);
    const uint32_t lane_row = (uint32_t)(wave * TOK_W + 4 * h);
    const uint32_t lane_col = (uint32_t)(2 * l32 * (int)sizeof(OT));
    const uint32_t last_row = (uint32_t)(n_valid - 1);
    const bool fast = n_valid == TOK_WG && (TT == 1 || (!SHARE && streamed));

    // One 32-feature tile: the accumulators start from mu and sweep the coordinates.
    auto tile_step = [&](int stage, f32x16 (&acc)[TT]) {
        const uint4* bbase = ring + stage * STAGE_U4 + lane;
        f32x16 start;                                           // (one copy of mu for all token tiles)
        {
            const float m = reinterpret_cast<const float*>(ring + stage * STAGE_U4 + SLAB_U4)[l32];
#pragma unroll
            for (int i = 0; i < 16; ++i) start[i] = m;
        }
        constexpr int NSTEP = 2 * NCT;
        uint4 bf[3];
        bf[0] = bbase[0];
        bf[1] = bbase[64];
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int ks = 0; ks < NSTEP; ++ks) {
            if (ks + 2 < NSTEP) bf[(ks + 2) % 3] = bbase[(ks + 2) * 64];
            const bf16x8 bv = as_bf16x8_d(bf[ks % 3]);
#pragma unroll
            for (int tt = 0; tt < TT; ++tt)
                acc[tt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(aop[tt][ks], bv, ks == 0 ? start : acc[tt], 0, 0, 0);
            __builtin_amdgcn_sched_barrier(0);
        }
    };

    // Waits: the slab of the next step must have landed before the barrier publishes it.  Memory
    // operations complete in issue order, so it is enough that no more operations are in flight
    // than this wave issued after that slab's transfers (the next tile's records in the first
    // step, the stores in odd steps).
    for (int f0 = 0; f0 < n_ft; f0 += 2) {
        f32x16 acc0[TT], acc1[TT];
        issue_slab(f0 + 1, 1);
        int n_rec = 0;
        if (f0 == 0 && has_next) n_rec = issue_records(a, next, Pn, lds_offset(work));
        tile_step(0, acc0);
        if (f0 == 0) wait_vmem_dyn(n_rec); else wait_vmem<0>();
        __syncthreads();

        const bool more = f0 + 2 < n_ft;
        if (more) issue_slab(f0 + 2, 0);
        tile_step(1, acc1);
        {
            store_pair<TT, OT, ACC, (TT > 1)>(a, tr, acc0, acc1, obase, SHARE ? f0 / 2 + first_span : f0 / 2, lane_row, lane_col, last_row, tok_tile0, fast);
        }
        // (the adds are a data-dependent number of operations, so after them the wait is for everything)
        if (more && ACC == 0) wait_vmem<NST>(); else wait_vmem<0>();
        __syncthreads();
    }
}

// One kernel per register class (TT token tiles per wave, plans of up to CLS coordinate tiles): up to 4 tiles
// three workgroups share a compute unit, up to 10 two (wider plans: the wide kernels below).  Inside a class every tile runs the
// code of its own plan's width (a switch over the widths built for the class -- their register needs are
// alike, so the class allocates what its widest member needs and no more), which makes a batch whose plans
// differ in width ONE launch per class: separate launches per width each ended with compute units idle
// while their last tiles finished (the 32-layer cache at 16x has plans of 7, 8 and 9 tiles: 1.39 ms in
// three launches, against 16 full rounds of tiles in one).  A batched launch serves only the jobs whose
// plan belongs to its class.  The tile loop is persistent.  With a non-zero a.dec_ring_off the ring sits
// behind the record image and each tile's records are fetched during the previous tile's sweep; with
// offset 0 they share the space and the records are fetched at the tile's start.
// (must agree with the host's class table)
template <int TT, int CLS> constexpr int dec_wgs_per_cu() { return CLS <= 4 ? 3 : (CLS <= 10 ? 2 : 1); }

// The widths built for each class; a plan's tile count is rounded up to the next of them at plan creation.
template <int CLS, int TT, typename OT, int ACC, bool SHARE>
__device__ __forceinline__ void decode_tile_of_class(const PlanDec& P, const TileRef& tr, const KernelArgs& a, uint4* work, uint4* ring,
                                                     bool prefetch, bool has_next, const TileRef& next, const PlanDec& Pn, int first_span, bool streamed) {
#define KVTC_W(N) case N: decode_tile<N, TT, OT, ACC, SHARE>(P, tr, a, work, ring, prefetch, has_next, next, Pn, first_span, streamed); break;
    if constexpr (CLS == 4) {
        switch (P.dec_nct) { KVTC_W(2) default: decode_tile<4, TT, OT, ACC, SHARE>(P, tr, a, work, ring, prefetch, has_next, next, Pn, first_span, streamed); break; }
    } else if constexpr (CLS == 10) {
        switch (P.dec_nct) { KVTC_W(6) KVTC_W(7) KVTC_W(8) KVTC_W(9) default: decode_tile<10, TT, OT, ACC, SHARE>(P, tr, a, work, ring, prefetch, has_next, next, Pn, first_span, streamed); break; }
    }
#undef KVTC_W
}

template <typename OT, int TT, int CLS, int ACC = 0>
__global__ void __launch_bounds__(kThreads, (dec_wgs_per_cu<TT, CLS>())) kvtc_decode_kernel(const KernelArgs a) {
    extern __shared__ uint4 smem[];
    uint32_t* tile_start = reinterpret_cast<uint32_t*>(smem);
    uint4* work = smem + kJobTableBytes / 16 + 1;
    const TileTable table = build_tile_table<false>(a, TT * 100 + CLS, tile_start, reinterpret_cast<uint32_t*>(work));
    const uint32_t total = table.total;
    const bool prefetch = a.dec_ring_off != 0u;
    uint4* ring = work + a.dec_ring_off / 16u;
    // Few tiles: every token tile is given to `parts` workgroups, each of which unpacks it again and sweeps its own share
    // of the features, so that a launch of a few tiles spreads over the chip instead of a lone workgroup walking all
    // features (48 tokens of 1024 features: 27 us -> 10).  Features are independent of each other: the results are the same bits.
    // (A copy of the sweep of its own: the two more scalars it carries cost the 16x cache 1 % when every sweep carried them.)
    const uint32_t parts = total ? gridDim.x / total : 0u;
    if (parts > 1u) {
        const uint32_t tile = blockIdx.x / parts, part = blockIdx.x % parts;
        if (tile >= total) return;
        const TileRef tr = find_tile(a, tile_start, tile);
        PlanDec P = load_plan_dec(a.plans + tr.plan);
        P.dec_tok_wg = 4 * 32 * TT;          // this variant's tile (the descriptor holds the bulk variant's)
        const uint32_t pairs = (uint32_t)P.p / 64u, n = min(parts, pairs);
        if (part >= n) return;
        const uint32_t begin = part * pairs / n;
        P.p = (int32_t)(64u * ((part + 1u) * pairs / n - begin));          // a plan that has only these features
        P.v_dec += (size_t)(2u * begin) * (size_t)(2 * P.dec_nct * 64 + kMuU4);
        issue_records(a, tr, P, lds_offset(work));
        wait_vmem<0>();
        __syncthreads();
        decode_tile_of_class<CLS, TT, OT, ACC, true>(P, tr, a, work, ring, prefetch, false, tr, P, (int)begin, false);
        return;
    }
    const TileRange mine = my_tiles(total);
    uint32_t tile = mine.first;
    if (tile >= mine.end) return;
    TileRef tr = find_tile(a, tile_start, tile);
    PlanDec P = load_plan_dec(a.plans + tr.plan);
    const bool streamed = TT > 1 && table.pass;
    P.dec_tok_wg = 4 * 32 * TT;
    issue_records(a, tr, P, lds_offset(work));
    wait_vmem<0>();
    __syncthreads();
    for (;;) {
        const uint32_t next = tile + mine.step;
        const bool has_next = next < mine.end;
        TileRef trn = tr;
        PlanDec Pn = P;
        if (has_next) {
            trn = find_tile(a, tile_start, next);
            Pn = load_plan_dec(a.plans + trn.plan);
            Pn.dec_tok_wg = 4 * 32 * TT;
        }
        decode_tile_of_class<CLS, TT, OT, ACC, false>(P, tr, a, work, ring, prefetch, has_next && prefetch, trn, Pn, 0, streamed);
        if (!has_next) break;
        tile = next;
        tr = trn;
        P = Pn;
        if (!prefetch) {
            issue_records(a, tr, P, lds_offset(work));
            wait_vmem<0>();
            __syncthreads();
        }
    }
}

// Wide plans (more than 320 coordinates).  Their operands do not fit the registers of a wave beside accumulators for more than one
// token tile, and with one token tile per basis fragment the LDS bandwidth is used up by fragments.  So here the roles are turned
// round: a workgroup of 8 waves unpacks its tile's records ONCE into matrix operands in LDS (32 * TT tokens x all coordinates, up to 144 KiB),
// and each wave sweeps feature pairs of its own, its basis fragments streaming from the L2 straight into registers, DEPTH k-steps ahead and on
// across the pairs.  A fragment serves TT token tiles, an operand read from LDS two feature tiles; the sweep has no barrier, so a
// wave's stores run under the other waves' matrix work.  TT = 4 up to 576 coordinates, 2 beyond (the operands must fit).  One kernel
// serves all widths of a class: the number of k-steps is a loop bound.  Measured against the register-operand form (a wave's operands in
// registers, the basis through an LDS ring): 16 tensors of 32768 tokens at 480-528 coordinates 740 -> 665 us, 1024 coordinates of 4096 features
// 402 -> 352, the same with the earlier section's sum added 832 -> 426 (it now travels under the last k-steps), one tensor of 100 tokens at
// 8x 25 -> 16.  What bounds it: the basis at 12 TB/s from the L2s (TT = 2), the unpacking that nothing overlaps (TT = 4).
template <int TT, int ACC> constexpr int wide_depth() { return TT == 4 || ACC == 2 ? 4 : 8; }       // (fewer where the earlier sum needs registers)
constexpr int kWideThreads = 512;

template <int TT, typename OT, int ACC>
__device__ __forceinline__ void decode_wide_tile(const PlanDec& P, const TileRef& tr, const KernelArgs& a, uint4* work, int q_begin, int q_end, bool streamed) {
    constexpr int DEPTH = wide_depth<TT, ACC>(), TOK = 32 * TT, ITEMS = (TT == 4 ? 18 * 4 : 32 * 2) / 8;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l32 = lane & 31, h = lane >> 5;
    const int nct = P.dec_nct, n_ks = 2 * nct;
    const int tok_tile0 = tr.tile * TOK, n_valid = min(TOK, tr.n_tokens - tok_tile0);
    uint4* ops = work + kAuxBytes / 16;                          // [k-step][token tile][lane]

    // ---- records -> operands: through registers, because the operands take the records' place ----
    __syncthreads();                                             // the tile before has been swept
    issue_records<kWideThreads>(a, tr, P, lds_offset(work));
    wait_vmem<0>();
    __syncthreads();
    {
        const RecImage im = rec_image(P.rec_dwords, tr.offset + (uint64_t)tok_tile0 * (uint64_t)P.rec_dwords * 4ull);
        const uint32_t* blk = reinterpret_cast<const uint32_t*>(work);
        const uint32_t* rec = blk + kAuxBytes / 4 + im.skew_dw;
        const int n_items = (nct * TT - wave + 7) / 8;           // (unpacking the class's most items instead cost plans of 19 to 24 tiles, which have 5 or 6 of the 8, 1 to 2 % of a small call)
        uint32_t q[ITEMS][8], info[ITEMS];
#pragma unroll
        for (int k = 0; k < ITEMS; ++k) info[k] = blk[2 * min((wave + 8 * k) / TT, nct - 1) + h];
        auto unpack = [&](auto narrow_tag) {
            RecBlock<decltype(narrow_tag)::value> b[2];          // this item's and the next one's
            auto read = [&](int k) {
                const int tt = (wave + 8 * k) % TT;
                b[k & 1].read(rec + (uint32_t)min(tt * 32 + l32, n_valid - 1) * im.stride_dw, info[k]);      // tail rows: the last token's record
            };
            read(0);
#pragma unroll
            for (int k = 0; k < ITEMS; ++k) {
                if (k >= n_items) break;
                if (k + 1 < ITEMS && k + 1 < n_items) read(k + 1);
                __builtin_amdgcn_sched_barrier(0);
                b[k & 1].values(q[k]);
                asm volatile("" : "+v"(q[k][0]), "+v"(q[k][1]), "+v"(q[k][2]), "+v"(q[k][3]), "+v"(q[k][4]), "+v"(q[k][5]), "+v"(q[k][6]), "+v"(q[k][7]));
            }
        };
        if (P.code_bits_max <= 8) unpack(std::true_type()); else unpack(std::false_type());
        __syncthreads();
#pragma unroll
        for (int k = 0; k < ITEMS; ++k) {
            const int item = wave + 8 * k, c = item / TT, tt = item % TT;
            if (c >= nct) continue;
            ops[(2 * c * TT + tt) * 64 + lane] = make_uint4(q[k][0], q[k][1], q[k][2], q[k][3]);
            ops[((2 * c + 1) * TT + tt) * 64 + lane] = make_uint4(q[k][4], q[k][5], q[k][6], q[k][7]);
        }
        __syncthreads();
    }

    // ---- sweep the wave's feature pairs ----
    int q = q_begin + wave;
    if (q >= q_end) return;
    typedef const char __attribute__((address_space(1))) * global_ptr;
    typedef const u32x4 __attribute__((address_space(1))) * global_u4;
    typedef const float __attribute__((address_space(1))) * global_f;
    const uint32_t stage_b = (uint32_t)(n_ks * 64 + kMuU4) * 16u;
    const uint64_t v0 = (uint64_t)uniform_ptr(P.v_dec);
    u32x4 bf[DEPTH][2];
    auto fetch = [&](int pair, int step, int slot) {
        const global_ptr src = (global_ptr)(v0 + (uint64_t)(uint32_t)(2 * pair) * (uint64_t)stage_b + (uint64_t)(uint32_t)step * 1024ull);      // a scalar address
        bf[slot][0] = *(global_u4)(src + (uint32_t)(lane * 16));
        bf[slot][1] = *(global_u4)(src + stage_b + (uint32_t)(lane * 16));
    };
    auto mu = [&](int pair, int odd) {
        return *(global_f)((global_ptr)(v0 + (uint64_t)(uint32_t)(2 * pair + odd) * (uint64_t)stage_b + (uint64_t)(uint32_t)(n_ks * 1024)) + (uint32_t)(l32 * 4));
    };
    float m0 = mu(q, 0), m1 = mu(q, 1);
#pragma unroll
    for (int j = 0; j < DEPTH; ++j) fetch(q, j, j);
    bf16x8 af[2][TT];                                            // operands of this k-step and of the next (the first again behind the last)
    const uint4* mine = ops + lane;
#pragma unroll
    for (int tt = 0; tt < TT; ++tt) af[0][tt] = as_bf16x8_d(mine[tt * 64]);

    char* obase = reinterpret_cast<char*>(const_cast<void*>(a.x)) + (size_t)(tr.x_row0 + tok_tile0) * (size_t)a.ld_x * sizeof(OT);
    const uint32_t lane_row = (uint32_t)(4 * h), lane_col = (uint32_t)(2 * l32 * (int)sizeof(OT)), last_row = (uint32_t)(n_valid - 1);
    const bool fast = n_valid == TOK && streamed;
    for (; q < q_end; q += 8) {
        const int qn = q + 8 < q_end ? q + 8 : q;
        f32x16 acc0[TT], acc1[TT];
#pragma unroll
        for (int tt = 0; tt < TT; ++tt)
#pragma unroll
            for (int i = 0; i < 16; ++i) { acc0[tt][i] = m0; acc1[tt][i] = m1; }
        m0 = mu(qn, 0);
        m1 = mu(qn, 1);
        // DEPTH k-steps from s on; their successors' fragments are requested as they go
        auto block = [&](int s) {
            const bool wrap = s + DEPTH >= n_ks;
            const int fq = wrap ? qn : q, fs0 = wrap ? s + DEPTH - n_ks : s + DEPTH;
#pragma unroll
            for (int j = 0; j < DEPTH; ++j) {
                const uint4* next = j + 1 < DEPTH ? mine + (s + j + 1) * (TT * 64) : mine + (wrap ? 0 : (s + DEPTH) * (TT * 64));
#pragma unroll
                for (int tt = 0; tt < TT; ++tt) af[(j + 1) & 1][tt] = as_bf16x8_d(next[tt * 64]);
                const bf16x8 b0 = __builtin_bit_cast(bf16x8, bf[j][0]), b1 = __builtin_bit_cast(bf16x8, bf[j][1]);
#pragma unroll
                for (int tt = 0; tt < TT; ++tt) {
                    acc0[tt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(af[j & 1][tt], b0, acc0[tt], 0, 0, 0);
                    acc1[tt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(af[j & 1][tt], b1, acc1[tt], 0, 0, 0);
                }
                fetch(fq, fs0 + j, j);
                __builtin_amdgcn_sched_barrier(0);
            }
        };
        if constexpr (ACC == 2 && TT == 2) {
            // the earlier sections' sums travel under the last k-steps
            for (int s = 0; s + DEPTH < n_ks; s += DEPTH) block(s);
            const char* sb = reinterpret_cast<const char*>(a.dec_sum) + ((size_t)(tr.x_row0 + tok_tile0) * (size_t)a.dec_sum_ld + (size_t)q * 64) * sizeof(float);
            const uint32_t sld = (uint32_t)a.dec_sum_ld * (uint32_t)sizeof(float);
            float2 part[TT][16];
            uint32_t lrow = lane_row;
            asm volatile("" : "+v"(lrow));
            if (last_row + 1u == (uint32_t)TOK) {                // (as in store_pair: scalar row addresses where no row lies past the end)
                typedef const f32x2_d __attribute__((address_space(1))) * global_f2;
                const uint64_t rows = (uint64_t)uniform_ptr(sb);
                const uint32_t lane_off = lrow * sld + 2u * lane_col;                      // below 64 rows of 2^23 bytes
#pragma unroll
                for (int tt = 0; tt < TT; ++tt)
#pragma unroll
                    for (int i = 0; i < 16; ++i) {
                        const f32x2_d v = *(global_f2)((global_ptr)(rows + (uint64_t)(uint32_t)(tt * 32 + 8 * (i / 4) + i % 4) * (uint64_t)sld) + lane_off);
                        part[tt][i] = make_float2(v[0], v[1]);
                    }
            } else {
#pragma unroll
                for (int tt = 0; tt < TT; ++tt)
#pragma unroll
                    for (int i = 0; i < 16; ++i) part[tt][i] = load_part(sb, lrow, tt, i, sld, lane_col, last_row);
            }
            __builtin_amdgcn_sched_barrier(0);
            block(n_ks - DEPTH);
#pragma unroll
            for (int tt = 0; tt < TT; ++tt)
#pragma unroll
                for (int i = 0; i < 16; ++i) { acc0[tt][i] = part[tt][i].x + acc0[tt][i]; acc1[tt][i] = part[tt][i].y + acc1[tt][i]; }
            store_pair<TT, OT, 0, true>(a, tr, acc0, acc1, obase, q, lane_row, lane_col, last_row, tok_tile0, fast);
        } else {
            for (int s = 0; s < n_ks; s += DEPTH) block(s);
            store_pair<TT, OT, ACC, true>(a, tr, acc0, acc1, obase, q, lane_row, lane_col, last_row, tok_tile0, fast);
        }
    }
    wait_vmem<0>();                                              // the fragments fetched past the last pair
}

template <typename OT, int TT, int CLS, int ACC>
__global__ void __launch_bounds__(kWideThreads, 1) kvtc_decode_wide_kernel(const KernelArgs a) {
    extern __shared__ uint4 smem[];
    uint32_t* tile_start = reinterpret_cast<uint32_t*>(smem);
    uint4* work = smem + kJobTableBytes / 16 + 1;
    const TileTable table = build_tile_table<false, kWideThreads>(a, TT * 100 + CLS, tile_start, reinterpret_cast<uint32_t*>(work));
    const uint32_t total = table.total;
    // few tiles: several workgroups share a tile's features, as above, but no fewer than four pairs each (a wave per SIMD)
    const uint32_t parts = total ? gridDim.x / total : 0u;
    TileRange mine = my_tiles(total);
    uint32_t part = 0u;
    if (parts > 1u) {
        mine = TileRange{blockIdx.x / parts, total, total};
        part = blockIdx.x % parts;
    }
    for (uint32_t tile = mine.first; tile < mine.end; tile += mine.step) {
        const TileRef tr = find_tile(a, tile_start, tile);
        PlanDec P = load_plan_dec(a.plans + tr.plan);
        const uint32_t pairs = (uint32_t)P.p / 64u, n = min(max(parts, 1u), max(pairs / 4u, 1u));
        if (part >= n) return;
        decode_wide_tile<TT, OT, ACC>(P, tr, a, work, (int)(part * pairs / n), (int)((part + 1u) * pairs / n), table.pass);
    }
}

// (token tiles per wave, class): the bulk kernels, then the same classes with one token tile per wave (128-token
// workgroup tiles) for single tensors short enough to run all their tiles at once -- a workgroup without a
// neighbour is bound by its own instruction stream, and this halves it.
// The wide kernels: (token tiles, class = the widest plan in coordinate tiles).
// The file is compiled once per part, each holding some of the kernels: the parts compile side by side.
#define KVTC_DEC_PART_0(X, W) X(2, 4) X(1, 4)
#define KVTC_DEC_PART_1(X, W) X(2, 10)
#define KVTC_DEC_PART_2(X, W) X(1, 10)
#define KVTC_DEC_PART_3(X, W) W(4, 18)
#define KVTC_DEC_PART_4(X, W) W(2, 32)

#define KVTC_CAT2(A, B) A##B
#define KVTC_CAT(A, B) KVTC_CAT2(A, B)

// The kernel of a key (100 * TT + CLS) if this part holds it, else null.
const void* KVTC_CAT(decode_kernel_part_, KVTC_DECODE_PART)(int key, kvtc_dtype dtype, int accumulate) {
    switch (key) {
#define KVTC_X(TT, CLS)                                                                                        \
    case (TT) * 100 + (CLS):                                                                                   \
        if (dtype == KVTC_BF16)                                                                                \
            return accumulate == 2 ? reinterpret_cast<const void*>(&kvtc_decode_kernel<uint16_t, TT, CLS, 2>)  \
                                   : reinterpret_cast<const void*>(&kvtc_decode_kernel<uint16_t, TT, CLS>);    \
        return accumulate == 1 ? reinterpret_cast<const void*>(&kvtc_decode_kernel<float, TT, CLS, 1>)         \
                               : reinterpret_cast<const void*>(&kvtc_decode_kernel<float, TT, CLS>);
#define KVTC_W(TT, CLS)                                                                                            \
    case (TT) * 100 + (CLS):                                                                                       \
        if (dtype == KVTC_BF16)                                                                                    \
            return accumulate == 2 ? reinterpret_cast<const void*>(&kvtc_decode_wide_kernel<uint16_t, TT, CLS, 2>) \
                                   : reinterpret_cast<const void*>(&kvtc_decode_wide_kernel<uint16_t, TT, CLS, 0>); \
        return accumulate == 1 ? reinterpret_cast<const void*>(&kvtc_decode_wide_kernel<float, TT, CLS, 1>)        \
                               : reinterpret_cast<const void*>(&kvtc_decode_wide_kernel<float, TT, CLS, 0>);
        KVTC_CAT(KVTC_DEC_PART_, KVTC_DECODE_PART)(KVTC_X, KVTC_W)
#undef KVTC_X
#undef KVTC_W
        default: return nullptr;
    }
}

#if KVTC_DECODE_PART == 0

#define KVTC_DEC_PARTS(X) X(0) X(1) X(2) X(3) X(4)
#define KVTC_X(P) const void* decode_kernel_part_##P(int key, kvtc_dtype dtype, int accumulate);
KVTC_DEC_PARTS(KVTC_X)
#undef KVTC_X

hipError_t launch_decode(const KernelArgs& a, kvtc_dtype dtype, int key, int grid, size_t lds_bytes, hipStream_t stream) {
    const void* fn = nullptr;
#define KVTC_X(P) if (!fn) fn = decode_kernel_part_##P(key, dtype, a.dec_accumulate);
    KVTC_DEC_PARTS(KVTC_X)
#undef KVTC_X
    if (!fn) return hipErrorInvalidValue;
    hipError_t e = allow_full_lds(fn);
    if (e != hipSuccess) return e;
    KernelArgs args = a;
    void* params[] = {&args};
    return hipLaunchKernel(fn, dim3(grid), dim3(key % 100 > 10 ? kWideThreads : kThreads), params, lds_bytes, stream);
}

// Bytes of the block table + record image and of the basis ring of a decode variant (the host
// lays them out: side by side when both fit, else sharing the space).
int decode_rec_bytes(int tt, int rec_dwords) {
    const int tok_wg = 4 * 32 * tt;
    return kAuxBytes + (tok_wg * (rec_dwords + 8) * 4 + 16 + 1023) / 1024 * 1024;      // padded rows or skew + one piece; whole 64-piece transfers
}
// The same of a wide kernel: block table, then the record image of 32 * tt tokens or the operands that take its place.
int decode_wide_bytes(int tt, int nct, int rec_dwords) {
    const int rec = (32 * tt * (rec_dwords + 8) * 4 + 16 + 1023) / 1024 * 1024, ops = tt * 2 * nct * 1024;
    return kAuxBytes + (rec > ops ? rec : ops);
}
int decode_ring_bytes(int nct) { return kDecStages * (2 * nct * 64 + kMuU4) * 16; }
int decode_stage_u4(int nct) { return 2 * nct * 64 + kMuU4; }

#endif  // KVTC_DECODE_PART == 0

}  // namespace kvtc
