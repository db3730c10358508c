// Device-side descriptors and the job -> tile scheduling shared by the encode and
// decode kernels.  Internal to the library.
#pragma once
#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>
#include <atomic>
#include <mutex>
#include <utility>
#include <vector>
#include "../../include/kvtc.h"

namespace kvtc {

constexpr int kThreads = 256;          // 4 wavefronts, one per SIMD of a compute unit
constexpr int kMaxJobs = 1024;         // jobs per batched launch (tile table lives in LDS)
constexpr int kLdsBudget = 160 * 1024; // gfx950 LDS per workgroup
constexpr int kJobTableBytes = (kMaxJobs + 1) * 4;
constexpr int kEncShortTile = 64;      // tokens per workgroup tile of the encode kernel for short jobs
constexpr int kShortTableJobs = 512;   // jobs of a batch that the short-job kernel codes alone, at most
constexpr int kEncPartTile = 32;       // tokens per workgroup tile of the encode by parts
constexpr int kEncParts = 4;           // workgroups that share the groups of a tile of a few tokens, at most
constexpr int kDecShortTile = 128;     // the same for decode (one token tile per wave)

// Lets a kernel use the whole LDS of a compute unit as dynamic shared memory.  The attribute
// sticks to the (device, function) pair, so it is set on the first launch there only.
inline hipError_t allow_full_lds(const void* fn) {
    static std::mutex m;
    static std::vector<std::pair<int, const void*>> done;
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    std::lock_guard<std::mutex> lock(m);
    for (const auto& d : done)
        if (d.first == dev && d.second == fn) return hipSuccess;
    e = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, kLdsBudget);
    if (e == hipSuccess) done.emplace_back(dev, fn);
    return e;
}

// Compute units of the current device, asked for once per device (any number of threads may).
inline int compute_units() {
    static std::atomic<int> known[64];
    int dev = 0, n = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return 256;
    n = known[dev].load(std::memory_order_relaxed);
    if (n == 0) {
        if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n <= 0) n = 256;
        known[dev].store(n, std::memory_order_relaxed);
    }
    return n;
}

// Everything a kernel needs to know about a plan.  Lives in device memory and is read
// through wave-uniform (scalar) loads.
struct PlanDev {
    int32_t p, r, n_groups, n_blocks;       // n_blocks = r / 16
    int32_t rec_dwords;                     // R / 4
    int32_t enc_ntw, enc_wc;                // encode variant: coefficient tiles per wave, waves across coefficients
    int32_t dec_nct, dec_tt;                // decode variant: coefficient tiles, token tiles per wave
    int32_t enc_tok_wg, dec_tok_wg;         // tokens per workgroup tile
    int32_t enc_lds[2];                     // encode: dynamic LDS bytes needed (without the job table), per element dtype
    int32_t dec_rec_lds, dec_ring_lds;      // decode: bytes of the record image, of the basis ring + mu
    int32_t code_bits_max;                  // widest code of the plan
    int32_t enc_wgs, dec_wgs;               // workgroups per compute unit the variant is built for (1..3)
    int32_t enc_nw, enc_short;              // encode: waves per workgroup (4 or 8); coordinate tiles per wave of the kernel for short jobs (64-token tiles), 0 = none
    int32_t dec_cls, enc_parts;             // decode: the kernel class that serves the plan = the widest plan of the class, in coordinate tiles (dec_nct: the width the plan runs at, one of those built for the class); encode: shares of whole groups that workgroups of their own can code, 0 = none
    const uint4* v_enc;    // [p/16][32*ntp/32][64] MFMA A fragments of V_kept^T (encode)
    const uint4* v_dec;    // [p/32][2*nct*64 + 16] MFMA B fragments of V_kept^T (decode), then the tile's 32 mu entries; tiles 2k, 2k+1 = even, odd features of span k
    const float* negc;     // [32*ntp]  -(mu^T V_kept), zero in the padding
    const float* mu;       // [p]
    const uint32_t* blk;   // [64] per 16-coordinate block: bits | group << 8 | halfword offset << 16; 0 = padding
    const uint32_t* grp;   // [n_groups] first block | n blocks << 8 | bits << 16
    uint32_t enc_part[2 * kEncParts];       // of each: first group | last + 1 << 8 | first coordinate tile << 16 | last + 1 << 24; first halfword of its codes | last + 1 << 16
};

struct KernelArgs {
    const PlanDev* plans;      // device array
    int32_t n_plans;
    const kvtc_job* jobs;      // device array, or nullptr -> `single`
    int32_t n_jobs;
    kvtc_job single;
    uint32_t single_tiles;     // of `single`, at the launch's tile size
    const uint64_t* offsets;   // device, [n_jobs + 1], or nullptr (single job at offset 0)
    const void* x;             // feature array (encode: input, decode: output)
    int64_t ld_x;
    float x_pass_from;         // elements of a call's feature array (tokens x features of all its jobs) from which on it is read or written past the caches; infinity: never.  A single tensor's launch: 0 or infinity
    int32_t x_blk_log2;        // 0: a token's features are contiguous.  Else they come in blocks of 2^x_blk_log2 features (a head, a layer) ...
    int64_t x_blk_jump;        // ... and x_blk_jump elements lie between the end of a block and the start of the token's next one
    void* stream_buf;          // record stream (encode: output, decode: input)
    uint64_t cap;              // bytes available in stream_buf
    uint32_t* status;          // device, may be nullptr
    uint32_t dec_ring_off;     // decode: byte offset of the basis ring in the work area; 0 = it shares the record image's space
    int32_t enc_short_max;     // encode: jobs of at most this many tokens whose plan the short-job kernel serves may be left to it (bulk_takes_all); 0 = no job counts as short
    int32_t enc_table;         // encode of a batch: 1 = the short-job launch codes every job (short_table); 0 = it codes the short ones, a workgroup per job and tile
    int32_t enc_split;         // encode by parts: workgroups to a tile (the most of any plan; of one tensor, its plan's)
    int32_t enc_part_most;     // encode by parts or the short-job kernel, as the jobs' lengths have it: shares of tiles, in all, up to which by parts; 0 = the launch has one form
    int32_t enc_max_tokens;    // with enc_table: a job of more tokens cannot lie inside the stream buffer
    int32_t enc_cus;           // encode of a batch: compute units (a bulk launch has this many workgroups times its plans' enc_wgs)
    int32_t dec_short;         // decode: this launch runs the one-token-tile-per-wave variant of every plan (128-token tiles)
    int32_t dec_accumulate;    // decode of a sectioned plan: 1 = fp32 output, add the product to the output instead of storing it (a further section);
                               // 2 = bf16 output, store round(dec_sum + product) (the last section)
    const float* dec_sum;      // mode 2: the earlier sections' fp32 sums, [tokens][dec_sum_ld], features contiguous
    int64_t dec_sum_ld;
};

struct TileRef {
    int32_t job, plan, n_tokens;
    int64_t x_row0;
    uint64_t offset;
    int32_t tile;      // tile index inside the job
};

// The bulk encode variant of a plan, in decimal positions.
template <typename P> __device__ __forceinline__ int enc_key(const P& pl) { return pl.enc_nw * 10000 + pl.enc_wc * 100 + pl.enc_ntw; }

// Whether a job can be coded at all: its plan, its token count, and its own extent inside the buffer (offsets need not be a running
// sum: an append writes each job into its own region).
__device__ __forceinline__ bool job_ok(const KernelArgs& a, int j, const kvtc_job& jb) {
    bool ok = jb.plan >= 0 && jb.plan < a.n_plans && jb.n_tokens >= 0;
    if (ok && a.offsets) {
        const uint64_t off = a.offsets[j], bytes = (uint64_t)jb.n_tokens * (uint64_t)a.plans[jb.plan].rec_dwords * 4ull;
        ok = off <= a.cap && bytes <= a.cap - off;
    }
    return ok;
}

// Which of a batch's jobs the short-job kernel codes: those of at most one of its tiles; and those of up to a.enc_short_max tokens,
// unless a longer job needs their plan's bulk kernel anyway and its launch has room for them, that is, they do not make it run
// another round of tiles.  (The bulk launch then takes them along, where the short-job launch behind it would add its own time;
// another round costs more than that.  16x, jobs of 40000 and 10000 tokens: 57 us together, 65 apart; 63 of 400 and one of 4000: 43 and
// 62; but 8x, 16 of 400 and 16 of 2000, 257 to 320 tiles on 256 places: 86 together, 71 apart.)
// The bulk launches and the short-job launch decide it each for itself, from the same table: `longer` is whether there is such a
// job, `bulk` the tiles of the jobs that the bulk launch takes in any case, `all` those with the jobs in question.
__device__ __forceinline__ bool bulk_takes_all(uint32_t bulk, uint32_t all, uint32_t slots) { return (all + slots - 1u) / slots == (bulk + slots - 1u) / slots; }

// The same for a wave of the short-job kernel: true if the bulk launch of variant `key` takes the jobs of more than one tile along.
__device__ inline bool bulk_takes_mid_jobs(const KernelArgs& a, int key, uint32_t slots) {
    if (a.n_jobs == 1) return false;
    const int lane = (int)threadIdx.x & 63;
    auto ours = [&](int j, const kvtc_job& jb) { return job_ok(a, j, jb) && enc_key(a.plans[jb.plan]) == key; };
    bool longer = false;
    for (int j = lane; j < a.n_jobs; j += 64) {
        const kvtc_job jb = a.jobs[j];
        if (jb.n_tokens > a.enc_short_max) longer |= ours(j, jb);
    }
    if (!__any(longer)) return false;
    uint32_t bulk = 0, all = 0;
    for (int j = lane; j < a.n_jobs; j += 64) {
        const kvtc_job jb = a.jobs[j];
        if (!ours(j, jb)) continue;
        const PlanDev& pl = a.plans[jb.plan];
        if (pl.enc_short != 0 && jb.n_tokens <= kEncShortTile) continue;
        const uint32_t tiles = (uint32_t)((jb.n_tokens + pl.enc_tok_wg - 1) / pl.enc_tok_wg);
        all += tiles;
        if (pl.enc_short == 0 || jb.n_tokens > a.enc_short_max) bulk += tiles;
    }
#pragma unroll
    for (int d = 32; d > 0; d >>= 1) {
        bulk += (uint32_t)__shfl_xor((int)bulk, d, 64);
        all += (uint32_t)__shfl_xor((int)all, d, 64);
    }
    return bulk_takes_all(bulk, all, slots);
}

// Exclusive prefix of the per-thread sums over the workgroup, and the total: inside the waves by lane exchange, then over the waves' totals --
// one barrier, where a scan through LDS took two per doubling (an append step of 64 caches, three such launches: 23.2 us,
// now 22.3).  With it go the minimum of `low` and the OR of two flags.
struct BlockScan { uint32_t before, total, low, flags; };
template <int NT>
__device__ __forceinline__ BlockScan block_scan(uint32_t sum, uint32_t low, uint32_t flags, uint32_t* scratch /*[3 * NT / 64]*/) {
    constexpr int NWAVE = NT / 64;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    uint32_t incl = sum;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        const uint32_t v = (uint32_t)__shfl_up((int)incl, d, 64);
        if (lane >= d) incl += v;
        low = min(low, (uint32_t)__shfl_xor((int)low, d, 64));
    }
    flags = (__any(flags & 1u) ? 1u : 0u) | (__any(flags & 2u) ? 2u : 0u);
    if (lane == 63) {
        scratch[wave] = incl;
        scratch[NWAVE + wave] = low;
        scratch[2 * NWAVE + wave] = flags;
    }
    __syncthreads();
    BlockScan r{incl - sum, 0u, 0xffffffffu, 0u};
#pragma unroll
    for (int w = 0; w < NWAVE; ++w) {
        const uint32_t n = scratch[w];
        if (w < wave) r.before += n;
        r.total += n;
        r.low = min(r.low, scratch[NWAVE + w]);
        r.flags |= scratch[2 * NWAVE + w];
    }
    return r;
}

// Sum over the workgroup, the same number in every thread and every workgroup.
template <int NT>
__device__ __forceinline__ float block_sum(float v, float* scratch /*[NT / 64]*/) {
#pragma unroll
    for (int d = 32; d > 0; d >>= 1) v += __shfl_xor(v, d, 64);
    if ((threadIdx.x & 63) == 0) scratch[threadIdx.x >> 6] = v;
    __syncthreads();
    float sum = 0.0f;
#pragma unroll
    for (int w = 0; w < NT / 64; ++w) sum += scratch[w];
    return sum;
}

// inclusive prefix sum over the 64 lanes, on the vector unit alone
__device__ __forceinline__ uint32_t wave_inclusive_scan(uint32_t v) {
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x111, 0xf, 0xf, false);      // row_shr:1
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x112, 0xf, 0xf, false);
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x114, 0xf, 0xf, false);
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x118, 0xf, 0xf, false);
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x142, 0xa, 0xf, false);      // row_bcast:15 into rows 1 and 3
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x143, 0xc, 0xf, false);      // row_bcast:31 into rows 2 and 3
    return v;
}

// Builds the exclusive prefix of tiles per job in LDS (tile_start[0..n_jobs]) and returns
// the total, and whether the call's feature array goes past the caches (by the tokens of all its valid jobs, whichever launch has them: with whole tiles
// of one launch counted, 512 jobs of 130 tokens, 130 MB, were taken for twice as much; 64 coordinates 35.4 -> 43.2 us).  A job with a bad plan index, a negative token count or a stream that would end
// beyond `cap` gets zero tiles, and so does a job whose plan belongs to another kernel variant
// (variant_key: the variant's parameters in decimal positions) or that the short-job kernel codes; workgroup 0 reports the
// lowest bad job in *status.  (A single tensor's launch has no table: built from one job it was 1 us of a small call.)
struct TileTable { uint32_t total; bool pass; };
template <bool kEncode, int NT = kThreads>
__device__ inline TileTable build_tile_table(const KernelArgs& a, int variant_key, uint32_t* tile_start, uint32_t* scratch /*[7 * NT / 64]*/) {
    if (!a.jobs) return {a.single_tiles, a.x_pass_from == 0.0f};      // the host has checked everything: no table
    const int tid = threadIdx.x;
    const int n_jobs = a.n_jobs;
    const int per = (n_jobs + NT - 1) / NT;
    const int j0 = tid * per;
    uint32_t local[kMaxJobs / NT], mid[kMaxJobs / NT];           // tiles; tiles of a job of more than one short tile that may go either way
    uint32_t sum = 0, mids = 0;
    const bool counts = a.x_pass_from < __builtin_huge_valf();       // (the host knows that a call is too small for it: half a microsecond of every launch)
    float amount = 0.0f;
    uint32_t first_bad = 0xffffffffu;
    uint32_t flags = 0;                                          // 1: a job longer than the short-job launch's limit; 2: one that may go either way
#pragma unroll
    for (int k = 0; k < kMaxJobs / NT; ++k) {
        uint32_t tiles = 0;
        mid[k] = 0;
        const int j = j0 + k;
        if (k < per && j < n_jobs) {
            const kvtc_job jb = a.jobs[j];
            if (job_ok(a, j, jb)) {
                const PlanDev& pl = a.plans[jb.plan];
                if (counts) amount += (float)jb.n_tokens * (float)pl.p;
                // each launch serves the plans of its own kernel variant; other launches take the rest.
                int tw = kEncode ? pl.enc_tok_wg : pl.dec_tok_wg;
                int key = kEncode ? enc_key(pl) : pl.dec_tt * 100 + pl.dec_cls;
                if (!kEncode && a.dec_short) { tw = kDecShortTile; key = 100 + pl.dec_cls; }
                // (no branches: the plan's fields are requested together)
                const uint32_t t = (uint32_t)((jb.n_tokens + tw - 1) / tw);
                const bool here = key == variant_key, shorter = kEncode & (pl.enc_short != 0) & (jb.n_tokens <= a.enc_short_max);
                const bool either = here & shorter & (jb.n_tokens > kEncShortTile);
                tiles = here & !shorter ? t : 0u;
                mid[k] = either ? t : 0u;
                flags |= (here & (jb.n_tokens > a.enc_short_max) ? 1u : 0u) | (either ? 2u : 0u);
            } else if (first_bad == 0xffffffffu) {
                first_bad = (uint32_t)j;
            }
        }
        local[k] = tiles;
        sum += tiles;
        mids += mid[k];
    }
    BlockScan sc = block_scan<NT>(sum, first_bad, flags, scratch);
    const bool pass = counts && __builtin_amdgcn_readfirstlane(block_sum<NT>(amount, reinterpret_cast<float*>(scratch + 6 * NT / 64)) >= a.x_pass_from ? 1 : 0) != 0;
    // lowest bad job -> status (workgroup 0 only; a plain vector store)
    if (a.status && blockIdx.x == 0 && tid == 0 && sc.low != 0xffffffffu) *a.status = sc.low + 1u;
    if (kEncode && __builtin_expect(sc.flags == 3u, 0)) {
        const BlockScan with = block_scan<NT>(sum + mids, 0u, 0u, scratch + 3 * NT / 64);
        if (bulk_takes_all(sc.total, with.total, gridDim.x)) {
            sc = with;
#pragma unroll
            for (int k = 0; k < kMaxJobs / NT; ++k) local[k] += mid[k];
        }
    }
    uint32_t run = sc.before;
#pragma unroll
    for (int k = 0; k < kMaxJobs / NT; ++k) {
        const int j = j0 + k;
        if (k < per && j < n_jobs) tile_start[j] = run;
        run += local[k];
    }
    if (tid == 0) tile_start[n_jobs] = sc.total;
    __syncthreads();
    return {sc.total, pass};
}

// A pointer whose value is the same in every lane, moved into scalar registers.
template <typename T> __device__ __forceinline__ const T* uniform_ptr(const T* p) {
    const uint64_t v = reinterpret_cast<uint64_t>(p);
    const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)v);
    const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)(v >> 32));
    return reinterpret_cast<const T*>(((uint64_t)hi << 32) | lo);
}

// Wave-uniform loads through the scalar unit (read-only data written before the launch: job
// list, stream offsets, plan descriptors).  They count on lgkmcnt, not on vmcnt, so they neither
// wait for nor disturb the vector-memory operations a kernel keeps in flight.
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x8 __attribute__((ext_vector_type(8)));
typedef uint32_t u32x16 __attribute__((ext_vector_type(16)));
// 16 bytes and 8 bytes from two places, one round trip
struct Words4And2 { u32x4 four; u32x2 two; };
__device__ __forceinline__ Words4And2 sload_x4_x2(const void* p4_uniform, const void* p2_uniform) {
    Words4And2 v;
    asm volatile("s_load_dwordx4 %0, %2, 0x0\n\ts_load_dwordx2 %1, %3, 0x0\n\ts_waitcnt lgkmcnt(0)"
                 : "=&s"(v.four), "=&s"(v.two)
                 : "s"(uniform_ptr(reinterpret_cast<const char*>(p4_uniform))), "s"(uniform_ptr(reinterpret_cast<const char*>(p2_uniform))) : "memory");
    return v;
}
template <typename T> __device__ __forceinline__ T* ptr_of(uint32_t lo, uint32_t hi) { return reinterpret_cast<T*>(((uint64_t)hi << 32) | lo); }

// The fields of a plan descriptor the decode kernel uses, in scalar registers.  (Its loads are issued together: one round trip to
// the L2, where a wait behind each of six loads was six.  Small calls are chains of such round trips.  No more is loaded than is used:
// with the descriptor's 24 dwords in one piece the fp32 kernel of ten blocks parked scalars in vector lanes 2011 times, not 876.)
struct PlanDec {
    int32_t p, rec_dwords, dec_nct, dec_tt, dec_tok_wg, code_bits_max;
    const uint4* v_dec;
    const uint32_t* blk;
};
__device__ __forceinline__ PlanDec load_plan_dec(const PlanDev* P) {
    static_assert(offsetof(PlanDev, p) == 0 && offsetof(PlanDev, rec_dwords) == 16 && offsetof(PlanDev, dec_nct) == 28 &&
                  offsetof(PlanDev, dec_tt) == 32 && offsetof(PlanDev, dec_tok_wg) == 40 && offsetof(PlanDev, code_bits_max) == 60, "descriptor layout");
    static_assert(offsetof(PlanDev, v_dec) == 96 && offsetof(PlanDev, blk) == 120, "descriptor layout");
    uint32_t p, rd, tok, cb;
    u32x2 nt, v, k;
    asm volatile("s_load_dword %0, %7, 0x0\n\ts_load_dword %1, %7, 0x10\n\ts_load_dwordx2 %4, %7, 0x1c\n\ts_load_dword %2, %7, 0x28\n\t"
                 "s_load_dword %3, %7, 0x3c\n\ts_load_dwordx2 %5, %7, 0x60\n\ts_load_dwordx2 %6, %7, 0x78\n\ts_waitcnt lgkmcnt(0)"
                 : "=&s"(p), "=&s"(rd), "=&s"(tok), "=&s"(cb), "=&s"(nt), "=&s"(v), "=&s"(k) : "s"(uniform_ptr(reinterpret_cast<const char*>(P))) : "memory");
    PlanDec d;
    d.p = (int32_t)p;
    d.rec_dwords = (int32_t)rd;
    d.dec_nct = (int32_t)nt[0];
    d.dec_tt = (int32_t)nt[1];
    d.dec_tok_wg = (int32_t)tok;
    d.code_bits_max = (int32_t)cb;
    d.v_dec = ptr_of<const uint4>(v[0], v[1]);
    d.blk = ptr_of<const uint32_t>(k[0], k[1]);
    return d;
}

// The fields of a plan descriptor the encode kernels use, in scalar registers; SHORT: with those that only the short-job kernels look at.  (An
// output of the statement is loaded and kept whether or not it is used, and scalar registers are short in the bulk kernels: with one list for
// both, 13 of the 25 dwords that a bulk tile asked for were dead; two tensors of 131072 tokens at 20x, encode and decode, 339.7 us so and 337.3 now.)
struct PlanEnc {
    int32_t p, r, n_groups, rec_dwords, code_bits_max;
    int32_t enc_ntw, enc_wc, enc_wgs, enc_nw, enc_short;     // SHORT
    const uint4* v_enc;
    const float* negc;
    const uint32_t* blk;
    const uint32_t* grp;
};
template <bool SHORT> __device__ __forceinline__ PlanEnc load_plan_enc(const PlanDev* P) {
    static_assert(offsetof(PlanDev, p) == 0 && offsetof(PlanDev, r) == 4 && offsetof(PlanDev, n_groups) == 8 && offsetof(PlanDev, rec_dwords) == 16 && offsetof(PlanDev, enc_ntw) == 20 && offsetof(PlanDev, enc_wc) == 24, "descriptor layout");
    static_assert(offsetof(PlanDev, code_bits_max) == 60 && offsetof(PlanDev, enc_wgs) == 64 && offsetof(PlanDev, enc_nw) == 72 && offsetof(PlanDev, enc_short) == 76 && offsetof(PlanDev, v_enc) == 88 &&
                  offsetof(PlanDev, negc) == 104 && offsetof(PlanDev, blk) == 120 && offsetof(PlanDev, grp) == 128, "descriptor layout");
    const char* from = uniform_ptr(reinterpret_cast<const char*>(P));
    PlanEnc d;
    u32x4 t;
    u32x2 v, c;
    if constexpr (SHORT) {
        u32x8 f;
        u32x4 w;
        uint32_t m;
        asm volatile("s_load_dwordx8 %0, %6, 0x0\n\ts_load_dword %1, %6, 0x3c\n\ts_load_dwordx4 %2, %6, 0x40\n\ts_load_dwordx2 %3, %6, 0x58\n\t"
                     "s_load_dwordx2 %4, %6, 0x68\n\ts_load_dwordx4 %5, %6, 0x78\n\ts_waitcnt lgkmcnt(0)"
                     : "=&s"(f), "=&s"(m), "=&s"(w), "=&s"(v), "=&s"(c), "=&s"(t) : "s"(from) : "memory");
        d.p = (int32_t)f[0];
        d.r = (int32_t)f[1];
        d.n_groups = (int32_t)f[2];
        d.rec_dwords = (int32_t)f[4];
        d.enc_ntw = (int32_t)f[5];
        d.enc_wc = (int32_t)f[6];
        d.code_bits_max = (int32_t)m;
        d.enc_wgs = (int32_t)w[0];
        d.enc_nw = (int32_t)w[2];
        d.enc_short = (int32_t)w[3];
    } else {
        uint32_t g, rd, m;
        u32x2 p;
        asm volatile("s_load_dwordx2 %0, %7, 0x0\n\ts_load_dword %1, %7, 0x8\n\ts_load_dword %2, %7, 0x10\n\ts_load_dword %3, %7, 0x3c\n\t"
                     "s_load_dwordx2 %4, %7, 0x58\n\ts_load_dwordx2 %5, %7, 0x68\n\ts_load_dwordx4 %6, %7, 0x78\n\ts_waitcnt lgkmcnt(0)"
                     : "=&s"(p), "=&s"(g), "=&s"(rd), "=&s"(m), "=&s"(v), "=&s"(c), "=&s"(t) : "s"(from) : "memory");
        d.p = (int32_t)p[0];
        d.r = (int32_t)p[1];
        d.n_groups = (int32_t)g;
        d.rec_dwords = (int32_t)rd;
        d.code_bits_max = (int32_t)m;
        d.enc_ntw = d.enc_wc = d.enc_wgs = d.enc_nw = d.enc_short = 0;
    }
    d.v_enc = ptr_of<const uint4>(v[0], v[1]);
    d.negc = ptr_of<const float>(c[0], c[1]);
    d.blk = ptr_of<const uint32_t>(t[0], t[1]);
    d.grp = ptr_of<const uint32_t>(t[2], t[3]);
    return d;
}

// The tiles of a persistent workgroup: first, first + step, ... below end.  Workgroups are dealt to the
// chip's eight XCDs round-robin (workgroup b runs on XCD b % 8; read back from the hardware's XCC id), and
// each XCD has an L2 of its own.  Every round of gridDim tiles is therefore cut into eight contiguous blocks,
// one per XCD: the workgroups of an XCD then work on the same tensor (or two) at any time and touch one
// basis, not the four that a round spans -- with a basis per tensor the decode of the 32-layer cache
// measured 6 % faster this way (its basis slabs compete for the L2 with 4 GiB of output passing through);
// the whole launch still sweeps memory as one window.  (Wherever the hardware places a workgroup, every
// tile is done exactly once.)
struct TileRange { uint32_t first, end, step; };
__device__ __forceinline__ TileRange my_tiles(uint32_t total) {
    const uint32_t g = gridDim.x, b = blockIdx.x;
    if ((g & 7u) != 0u || total < 2u * g) return TileRange{b, total, g};
    return TileRange{(b & 7u) * (g >> 3) + (b >> 3), total, g};
}

__device__ inline TileRef find_tile(const KernelArgs& a, const uint32_t* tile_start, uint32_t tile) {
    static_assert(sizeof(kvtc_job) == 16 && offsetof(kvtc_job, n_tokens) == 4 && offsetof(kvtc_job, x_row0) == 8, "job layout");
    if (!a.jobs) return TileRef{0, a.single.plan, a.single.n_tokens, a.single.x_row0, 0ull, (int32_t)tile};
    int lo = 0, hi = a.n_jobs;               // invariant: tile_start[lo] <= tile < tile_start[hi]
    while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        if (tile_start[mid] <= tile) lo = mid; else hi = mid;
    }
    lo = __builtin_amdgcn_readfirstlane(lo);
    const Words4And2 v = sload_x4_x2(a.jobs + lo, a.offsets + lo);
    TileRef t;
    t.job = lo;
    t.plan = (int32_t)v.four[0];
    t.n_tokens = (int32_t)v.four[1];
    t.x_row0 = (int64_t)(((uint64_t)v.four[3] << 32) | v.four[2]);
    t.offset = ((uint64_t)v.two[1] << 32) | v.two[0];
    t.tile = __builtin_amdgcn_readfirstlane((int32_t)(tile - tile_start[lo]));
    return t;
}

// LDS byte offset of a pointer into shared memory.
__device__ __forceinline__ uint32_t lds_offset(const void* p) {
    return (uint32_t)(size_t)(const __attribute__((address_space(3))) void*)p;
}

// 16 bytes per lane from global memory straight into LDS, no register staging: lane i's bytes
// land at lds_byte_addr + 16 * i (wave-uniform address; it goes through M0).  Issued behind the
// compiler's back: the compiler neither orders later LDS reads after it nor counts it, so a
// step's transfers can stay in flight while the previous slab is read (the builtin form makes the
// compiler wait for vmcnt(0) before any later LDS read).  The caller owns the wait: wait_vmem<N>()
// before the barrier that publishes the data.
__device__ __forceinline__ void dma16_async(const void* gsrc, uint32_t lds_byte_addr) {
    asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, off"
                 :: "v"(gsrc), "s"(lds_byte_addr) : "memory");
}

// The same with a wave-uniform base (scalar registers) plus a 32-bit per-lane byte offset: the
// per-transfer address arithmetic stays on the scalar unit and costs no vector registers.
// (Values the compiler cannot prove uniform would reach the "s" operands in vector registers, so
// both go through readfirstlane, which folds away when they already are scalar.)
__device__ __forceinline__ void dma16_async(const void* base_uniform, uint32_t lane_byte_off, uint32_t lds_byte_addr) {
    asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1"
                 :: "v"(lane_byte_off), "s"(uniform_ptr(reinterpret_cast<const char*>(base_uniform))),
                    "s"(__builtin_amdgcn_readfirstlane(lds_byte_addr)) : "memory");
}

// The same for data that is read once: the caches are asked not to keep it.
__device__ __forceinline__ void dma16_async_once(const void* gsrc, uint32_t lds_byte_addr) {
    asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, off nt"
                 :: "v"(gsrc), "s"(lds_byte_addr) : "memory");
}
__device__ __forceinline__ void dma16_async_once(const void* base_uniform, uint32_t lane_byte_off, uint32_t lds_byte_addr) {
    asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1 nt"
                 :: "v"(lane_byte_off), "s"(uniform_ptr(reinterpret_cast<const char*>(base_uniform))),
                    "s"(__builtin_amdgcn_readfirstlane(lds_byte_addr)) : "memory");
}

// One dword per lane: lane i's dword lands at lds_byte_addr + 4 * i.
__device__ __forceinline__ void dma4_async(const void* base_uniform, uint32_t lane_byte_off, uint32_t lds_byte_addr) {
    asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dword %0, %1"
                 :: "v"(lane_byte_off), "s"(uniform_ptr(reinterpret_cast<const char*>(base_uniform))),
                    "s"(__builtin_amdgcn_readfirstlane(lds_byte_addr)) : "memory");
}

// s_waitcnt vmcnt(N) only (N <= 63): the N most recent vector-memory operations may stay in flight.
template <int N> __device__ __forceinline__ void wait_vmem() {
    static_assert(N >= 0 && N < 64, "vmcnt is a 6-bit field");
    __builtin_amdgcn_s_waitcnt(0x0F70 | (N & 15) | ((N >> 4) << 14));
}
// s_waitcnt vmcnt(n) with a wave-uniform run-time n; n above 63 waits as for 63.
__device__ __forceinline__ void wait_vmem_dyn(int n) {
#define KVTC_W(N) case N: wait_vmem<N>(); break;
#define KVTC_W8(N) KVTC_W(N) KVTC_W(N + 1) KVTC_W(N + 2) KVTC_W(N + 3) KVTC_W(N + 4) KVTC_W(N + 5) KVTC_W(N + 6) KVTC_W(N + 7)
    switch (n < 0 ? 0 : (n > 63 ? 63 : n)) {
        KVTC_W8(0) KVTC_W8(8) KVTC_W8(16) KVTC_W8(24) KVTC_W8(32) KVTC_W8(40) KVTC_W8(48) KVTC_W8(56)
    }
#undef KVTC_W8
#undef KVTC_W
}
// Wait until at most k * N operations are in flight, k in 0..3 chosen at run time (wave-uniform).
template <int N> __device__ __forceinline__ void wait_vmem_times(int k) {
    if (k <= 0) wait_vmem<0>();
    else if (k == 1) wait_vmem<N>();
    else if (k == 2) wait_vmem<2 * N>();
    else wait_vmem<3 * N>();
}

}  // namespace kvtc
