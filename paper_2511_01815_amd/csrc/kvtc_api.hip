// Host side of the C ABI declared in include/kvtc.h: argument checks, plan compilation
// (swizzling the basis into matrix-core operand fragments, block/group tables), launches,
// and the on-device prefix sum of stream offsets.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdarg>
#include <cstdio>
#include <cstring>
#include <new>
#include <vector>

#include "kvtc_dev.h"
#include "kvtc_numeric.h"
#include "../../include/kvtc_test_hooks.h"

namespace kvtc {
hipError_t launch_encode(const KernelArgs& a, kvtc_dtype dtype, int key, int grid, size_t lds_bytes, hipStream_t stream);
hipError_t launch_decode(const KernelArgs& a, kvtc_dtype dtype, int key, int grid, size_t lds_bytes, hipStream_t stream);
hipError_t launch_encode_short(const KernelArgs& a, kvtc_dtype dtype, int ntw, int waves, int grid, size_t lds_bytes, hipStream_t stream);
int encode_lds_bytes(int ntw, int wc, int nw, int n_groups, int rec_dwords, kvtc_dtype dtype);
hipError_t launch_encode_parts(const KernelArgs& a, kvtc_dtype dtype, int waves, int max_p, int grid, size_t lds_bytes, hipStream_t stream);
int encode_part_waves_most();
int encode_part_lds_bytes(int p, int ntp, int n_groups, int rec_dwords, kvtc_dtype dtype);
int encode_short_ntw(int ntp);
int encode_short_waves(int ntp);
int encode_short_lds_bytes(int ntp, int n_groups, int rec_dwords, kvtc_dtype dtype);
int encode_tok_wg(int ntw, int wc, int nw);
uint64_t encode_pass_bytes(int ntp, kvtc_dtype dtype);
uint64_t decode_pass_bytes(int cls, int least_tiles, kvtc_dtype dtype, uint64_t bases, bool single);
hipError_t launch_fp8_pack(const void* x, kvtc_dtype dtype, int64_t n_tokens, int p, int64_t ld_x, void* out, hipStream_t stream);
hipError_t launch_fp8_unpack(const void* in, int64_t n_tokens, int p, void* x, kvtc_dtype dtype, int64_t ld_x, hipStream_t stream);
hipError_t launch_offsets_append(const uint32_t* rec_dwords, int n_plans, const kvtc_job* jobs, int n_jobs, const uint64_t* region,
                                 const int64_t* n_coded, uint64_t* offsets, hipStream_t stream);
struct RopeArgs {
    void* x;
    int64_t n_tokens, token_stride, head_stride;
    const int32_t* positions;
    int64_t position0;
    int32_t n_heads, d_head, inverse;
    double theta[128];
};
hipError_t launch_rope(const RopeArgs& a, kvtc_dtype dtype, int interleaved, int grid, hipStream_t stream);
hipError_t launch_calib_moments(const void* x, kvtc_dtype dtype, int64_t n_tokens, int p, int64_t ld, int blk_log2, int64_t blk_jump,
                                double* sum, double* gram, hipStream_t stream);
int decode_rec_bytes(int tt, int rec_dwords);
int decode_ring_bytes(int nct);
int decode_wide_bytes(int tt, int nct, int rec_dwords);
int decode_stage_u4(int nct);
}  // namespace kvtc

using namespace kvtc;

struct kvtc_plan {
    PlanDev h;              // host copy of the descriptor (device pointers inside)
    void* blob;             // one device allocation holding everything
    PlanDev* desc_dev;      // the descriptor inside the blob
    size_t record_bytes;
    int enc_s_waves;        // short-job encode kernel (h.enc_short, 0 = none): waves per workgroup ...
    int enc_s_lds[2];       // ... and dynamic LDS bytes per element dtype
    int enc_p_waves;        // the same by parts (h.enc_parts, 0 = none)
    int enc_p_lds[2];       // 0: not of this type
};

// The encode by parts of a set of plans; split = 0: some plan's groups cannot be shared out so.
struct PartVariant {
    int split = -1, waves = 0, lds = 0;                 // workgroups to a tile, waves, LDS bytes: the most of any plan.  (-1: no plan yet)
    void add(const kvtc_plan& plan, kvtc_dtype dtype) {
        const bool can = split != 0 && plan.h.enc_parts != 0 && plan.enc_p_lds[dtype] != 0;
        split = can ? std::max(split, plan.h.enc_parts) : 0;
        waves = std::max(waves, plan.enc_p_waves);
        lds = std::max(lds, plan.enc_p_lds[dtype]);
    }
};

struct kvtc_batch {
    PlanDev* plans_dev;
    int n_plans;
    // the kernel variants the plans use (a launch per variant), with the LDS maxima over each one's plans
    struct EncVariant { int key, wgs, lds[2]; };        // workgroups per compute unit; lds per element dtype
    // workgroups per compute unit; record image, basis ring, record (the widest among the class's plans); the narrowest's coordinate tiles, all their bases' bytes
    struct DecVariant { int key, wgs, rec, ring, rec_dwords, least_tiles; uint64_t bases; };
    std::vector<EncVariant> enc;
    struct ShortVariant { int waves, lds[2]; } enc_short[3];     // short-job kernels by coordinate tiles per wave; waves = 0: no plan uses it
    PartVariant enc_part[2];                            // by parts, per element dtype
    std::vector<DecVariant> dec;
    int max_p;
    int min_rec_dwords;                                 // the shortest record among the plans
    bool all_short;                                     // every plan has a short-job encode kernel
    std::vector<int32_t> ps;                            // the distinct feature counts among the plans
    std::vector<int32_t> rec_dwords;
    uint32_t* rec_dwords_dev;
};

namespace {

thread_local char g_err[256] = "";

kvtc_status fail(kvtc_status st, const char* fmt, ...) {
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(g_err, sizeof(g_err), fmt, ap);
    va_end(ap);
    return st;
}

float bf16_bits_to_float(uint16_t b) { return bits_f32((uint32_t)b << 16); }

// Whether two workgroups of the short-job kernel share a compute unit: up to 8 waves with a coordinate tile each, by their registers, and
// by the LDS they ask for.
bool short_pairs(int ntw, int waves, int lds) { return ntw == 1 && waves <= 8 && 2 * lds <= kLdsBudget; }

// 64-token tiles that each of n_jobs jobs may have and still all run at once on the short-job kernel (`pairs`: two workgroups share a
// compute unit), at least one: a job of no more is a short one.  The bulk tiles are three to four times as large: their launch has
// fewer workgroups than the chip, each walking all features.  One tensor of 4096 tokens at 16x: 42 us on the bulk tile, 21 on this;
// where the tiles need a second round the bulk kernel, which reads the basis less often, is the faster one again.
int short_tiles_per_job(int n_jobs, bool pairs) {
    const int n = compute_units() * (pairs ? 2 : 1) / n_jobs;
    return n < 1 ? 1 : n;
}

// Workgroups of a batch's one short-job launch, or 0 if the batch cannot be shown to fit one round of them: jobs do not overlap in the
// stream buffer, so its size bounds their tokens; each may end in a part of a tile; one workgroup more reports the jobs that are not valid.
int short_table_grid(size_t cap, int min_rec_dwords, int n_jobs, bool pairs) {
    const size_t tiles = cap / ((size_t)min_rec_dwords * 4 * kEncShortTile) + (size_t)n_jobs;
    const size_t grid = (tiles + 7) / 8 * 8 + 1;                     // whole shares for the eight XCDs
    return n_jobs <= kShortTableJobs && grid <= (size_t)compute_units() * (pairs ? 2 : 1) ? (int)grid : 0;
}

// Workgroups by parts that run at once: two to a compute unit of four waves whose LDS allows it.
int part_places(int waves, int lds) { return compute_units() * (waves <= 4 && 2 * lds <= kLdsBudget ? 2 : 1); }

// Tokens of a job, by the stream buffer's size, and shares of tiles, in all, that a batch coded by parts has: at most, if its jobs are equal, and if their last
// tiles are a quarter full on average.  (The jobs' lengths are on the device.)
struct PartShares { size_t each, most, equal, mixed; };
PartShares part_shares(size_t cap, int min_rec_dwords, int n_jobs, int split) {
    const size_t jobs = (size_t)n_jobs, tokens = cap / ((size_t)min_rec_dwords * 4), each = (tokens + jobs - 1) / jobs, whole = tokens / kEncPartTile;
    return {each, (whole + jobs) * split, (each + kEncPartTile - 1) / kEncPartTile * jobs * split, (whole + jobs * 3 / 4) * split};
}
int whole_shares(size_t n) { return (int)((n + 7) / 8 * 8 + 1); }        // for the eight XCDs; one workgroup more reports the jobs that are not valid

// Shares out a plan's groups, in order, over up to kEncParts workgroups so that the largest share has as few coordinate tiles as can be, with as few
// shares as that takes; returns the waves that takes, a coordinate tile to a wave, and at least four, or leaves enc_parts 0 where those are too many.
int share_groups(PlanDev* d, const kvtc_group* groups) {
    const int n = d->n_groups;
    std::vector<int> first(n + 1, 0), half(n + 1, 2 * n);           // a group's first block; the first halfword of its codes
    for (int g = 0; g < n; ++g) {
        first[g + 1] = first[g] + groups[g].n / 16;
        half[g + 1] = half[g] + groups[g].n / 16 * groups[g].bits;
    }
    auto tiles = [&](int g0, int g1) { return (first[g1] + 1) / 2 - first[g0] / 2; };
    // the fewest shares, in order, of at most `most` tiles each; their ends -> cut
    auto shares = [&](int most, int* cut) {
        int k = 0;
        for (int g0 = 0; g0 < n; ++k) {
            int g1 = g0;
            while (g1 < n && tiles(g0, g1 + 1) <= most) ++g1;
            if (g1 == g0 || k == kEncParts) return kEncParts + 1;
            cut[k] = g0 = g1;
        }
        return k;
    };
    int cut[kEncParts], k = kEncParts + 1, most = 0;
    while (most < encode_part_waves_most() && k > kEncParts) k = shares(++most, cut);
    if (k > kEncParts) return 0;
    d->enc_parts = k;
    for (int i = 0; i < k; ++i) {
        const int g0 = i ? cut[i - 1] : 0, g1 = cut[i];
        d->enc_part[2 * i] = (uint32_t)g0 | (uint32_t)g1 << 8 | (uint32_t)(first[g0] / 2) << 16 | (uint32_t)((first[g1] + 1) / 2) << 24;
        d->enc_part[2 * i + 1] = (uint32_t)half[g0] | (uint32_t)(g1 == n ? 2 * d->rec_dwords : half[g1]) << 16;
    }
    return most < 4 ? 4 : most;
}

// Row pitch limit (elements): the kernels address a workgroup tile of up to 256 rows with 32-bit byte offsets.
constexpr int kMaxPitch = 1 << 21;

size_t align_up(size_t v, size_t a) { return (v + a - 1) / a * a; }

// position of coordinate/feature row `rho` of an MFMA tile inside the lane's 16 results:
// the 32x32 accumulator gives lane half hh, register i the row 8*(i/4) + 4*hh + i%4; mapping
// row rho to index 16*hh + i makes each lane own 16 consecutive indices.
int permuted_index(int rho) {
    const int q = rho >> 3, hh = (rho >> 2) & 1, m = rho & 3;
    return 16 * hh + 4 * q + m;
}

bool dtype_ok(kvtc_dtype d) { return d == KVTC_BF16 || d == KVTC_F32; }
size_t elem_size(kvtc_dtype d) { return d == KVTC_BF16 ? 2 : 4; }

__global__ void __launch_bounds__(256) offsets_kernel(const uint32_t* rec_dwords, int n_plans, const kvtc_job* jobs,
                                                     int n_jobs, uint64_t* offsets, uint64_t* offsets_copy /*may be null*/) {
    __shared__ uint64_t s[256];
    __shared__ uint64_t carry;
    const int tid = threadIdx.x;
    if (tid == 0) carry = 0;
    __syncthreads();
    for (int base = 0; base < n_jobs; base += 256) {
        const int j = base + tid;
        uint64_t bytes = 0;
        if (j < n_jobs) {
            const kvtc_job jb = jobs[j];
            if (jb.plan >= 0 && jb.plan < n_plans && jb.n_tokens > 0)
                bytes = (uint64_t)jb.n_tokens * rec_dwords[jb.plan] * 4ull;
        }
        s[tid] = bytes;
        __syncthreads();
        for (int d = 1; d < 256; d <<= 1) {
            const uint64_t v = tid >= d ? s[tid - d] : 0ull;
            __syncthreads();
            s[tid] += v;
            __syncthreads();
        }
        const uint64_t c = carry;
        if (j < n_jobs) {
            offsets[j] = c + s[tid] - bytes;
            if (offsets_copy) offsets_copy[j] = c + s[tid] - bytes;
        }
        __syncthreads();
        if (tid == 255) carry = c + s[255];
        __syncthreads();
    }
    if (tid == 0) {
        offsets[n_jobs] = carry;
        if (offsets_copy) offsets_copy[n_jobs] = carry;
    }
}

// ---- the entry point that allocates nothing ------------------------------------------------------
// Its plan-descriptor table, record-size table and stream offsets -- what kvtc_batch_create and the
// caller's offsets buffer hold for kvtc_encode_batch -- live in this file-scope device array.  Every
// GPU the library runs on holds its own copy (about 17 KB) until the process ends.  The name is a
// host-side stand-in, not a device address: host code only ever uses the per-device pointer that
// hipGetSymbolAddress returned for it.
constexpr int kStaticMaxPlans = 64;
struct StaticScratch {
    PlanDev plans[kStaticMaxPlans];
    uint32_t rec_dwords[kStaticMaxPlans];
    uint64_t offsets[kMaxJobs + 1];
};
static __device__ __align__(256) unsigned char scratch[sizeof(StaticScratch)];

struct PlanPtrs { const PlanDev* p[kStaticMaxPlans]; };

// descriptor of plan i (inside the plan's own device blob) -> table entry i; one thread per dword
// (for a test of the table's count)
__global__ void __launch_bounds__(kThreads) batch_passes_kernel(const KernelArgs a, int variant_key, uint32_t* passes) {
    __shared__ uint32_t tile_start[kMaxJobs + 1], scratch[8 * kThreads / 64];
    const TileTable table = build_tile_table<true>(a, variant_key, tile_start, scratch);
    if (threadIdx.x == 0) *passes = table.pass ? 1u : 0u;
}

__global__ void __launch_bounds__(256) gather_plans_kernel(const PlanPtrs src, int n_plans, StaticScratch* sc) {
    constexpr int kDw = (int)(sizeof(PlanDev) / 4);
    static_assert(sizeof(PlanDev) % 4 == 0, "descriptor is whole dwords");
    for (int i = threadIdx.x; i < n_plans * kDw; i += blockDim.x) {
        const int pl = i / kDw, w = i - pl * kDw;
        reinterpret_cast<uint32_t*>(&sc->plans[pl])[w] = reinterpret_cast<const uint32_t*>(src.p[pl])[w];
    }
    for (int i = threadIdx.x; i < n_plans; i += blockDim.x) sc->rec_dwords[i] = (uint32_t)src.p[i]->rec_dwords;
}

// per-device address of `scratch`, looked up once per device with that device current
hipError_t static_scratch(StaticScratch** out) {
    static std::mutex m;
    static StaticScratch* ptr[64] = {nullptr};
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= 64) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lock(m);
    if (!ptr[dev]) {
        void* p = nullptr;
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return e;
        ptr[dev] = static_cast<StaticScratch*>(p);
    }
    *out = ptr[dev];
    return hipSuccess;
}

// Decode LDS layout for one launch: record image and basis ring side by side when both fit (narrow
// variants: within their share of a compute unit's LDS, so that all their workgroups stay resident), which lets each
// tile's records be fetched during the previous tile's sweep; otherwise they share the space.
struct DecLayout { uint32_t ring_off; size_t lds_bytes; };
DecLayout decode_layout(int rec_b, int ring_b, int wgs_per_cu) {
    const int budget = kLdsBudget / wgs_per_cu - kJobTableBytes - 64;
    if (rec_b + ring_b <= budget) return {(uint32_t)rec_b, (size_t)kJobTableBytes + 64 + rec_b + ring_b};
    return {0u, (size_t)kJobTableBytes + 64 + (rec_b > ring_b ? rec_b : ring_b)};
}

}  // namespace

namespace kvtc {
// for the library's other sources: records the message kvtc_last_error returns on this thread
kvtc_status set_error(kvtc_status st, const char* fmt, ...) {
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(g_err, sizeof(g_err), fmt, ap);
    va_end(ap);
    return st;
}
}  // namespace kvtc

extern "C" {

const char* kvtc_last_error(void) { return g_err; }

uint16_t kvtc_host_f16_round_down(float x) { return f16_round_dir(x, false); }
uint16_t kvtc_host_f16_round_up(float x) { return f16_round_dir(x, true); }
void kvtc_host_group_header(float lo, float hi, int bits, uint16_t* shift16, uint16_t* scale16) {
    const GroupQ q = group_header(lo, hi, bits);
    if (shift16) *shift16 = q.shift16;
    if (scale16) *scale16 = q.scale16;
}
uint32_t kvtc_host_code(float d, uint16_t shift16, uint16_t scale16, int bits) {
    const float sc = f16_bits_to_f32(scale16);
    const float inv = sc > 0.0f ? div_rn(1.0f, sc) : 0.0f;          // as group_header derives it
    return (uint32_t)code_of(d, f16_bits_to_f32(shift16), inv, (float)((1u << bits) - 1u));
}

// v_kept_host: [p] rows of ldv elements, of which the first r are the plan's columns.  dec_zero_mu: the decode side adds
// no mean (a further section of a sectioned plan: the first section's decode has added it already).
static kvtc_status plan_create_impl(kvtc_plan** out, int p, int r, const float* mu_host, const uint16_t* v_kept_host, size_t ldv,
                                    int n_groups, const kvtc_group* groups_host, bool dec_zero_mu, kvtc_stream stream);

kvtc_status kvtc_plan_create(kvtc_plan** out, int p, int r, const float* mu_host, const uint16_t* v_kept_host,
                             int n_groups, const kvtc_group* groups_host, kvtc_stream stream) {
    return plan_create_impl(out, p, r, mu_host, v_kept_host, (size_t)(r > 0 ? r : 0), n_groups, groups_host, false, stream);
}

static kvtc_status plan_create_impl(kvtc_plan** out, int p, int r, const float* mu_host, const uint16_t* v_kept_host, size_t ldv,
                                    int n_groups, const kvtc_group* groups_host, bool dec_zero_mu, kvtc_stream stream) {
    if (out) *out = nullptr;
    if (!out || !mu_host || !v_kept_host || !groups_host) return fail(KVTC_E_ARG, "kvtc_plan_create: null argument");
    if (p <= 0 || p % 64 != 0) return fail(KVTC_E_ARG, "kvtc_plan_create: p=%d must be a positive multiple of 64", p);
    if (r < 16 || r > 1024) return fail(KVTC_E_ARG, "kvtc_plan_create: r=%d outside 16..1024", r);
    if (n_groups < 1 || n_groups > 64) return fail(KVTC_E_ARG, "kvtc_plan_create: n_groups=%d outside 1..64", n_groups);
    long sum = 0, payload_bits = 0;
    for (int g = 0; g < n_groups; ++g) {
        if (groups_host[g].n < 1) return fail(KVTC_E_ARG, "kvtc_plan_create: group %d is empty", g);
        if (groups_host[g].bits < 1 || groups_host[g].bits > 16)
            return fail(KVTC_E_ARG, "kvtc_plan_create: group %d has %d bits (1..16 allowed)", g, groups_host[g].bits);
        sum += groups_host[g].n;
        payload_bits += (long)groups_host[g].n * groups_host[g].bits;
    }
    if (sum != r) return fail(KVTC_E_ARG, "kvtc_plan_create: group sizes sum to %ld, r=%d", sum, r);
    for (int g = 0; g < n_groups; ++g)
        if (groups_host[g].n % 16 != 0)
            return fail(KVTC_E_UNSUPPORTED, "kvtc_plan_create: group %d has %d coordinates; the kernels need multiples of 16",
                        g, groups_host[g].n);

    PlanDev d;
    memset(&d, 0, sizeof(d));
    d.p = p;
    d.r = r;
    d.n_groups = n_groups;
    d.n_blocks = r / 16;
    for (int g = 0; g < n_groups; ++g)
        if (groups_host[g].bits > d.code_bits_max) d.code_bits_max = groups_host[g].bits;
    const long total_bits = 32L * n_groups + payload_bits;
    d.rec_dwords = (int)((total_bits + 31) / 32);
    const int nt = (r + 31) / 32;

    // encode variant: NTW coordinate tiles per wave, WC waves across coordinates, NW waves per workgroup.
    // Up to 320 padded coordinates a 4-wave workgroup keeps its tile (64 tokens per wave across the
    // tokens; 96 in the 8-tile variant, 32 in the 2-tile one) x all its coordinates in 256 registers per lane and two
    // workgroups share a compute unit (three where 168 registers suffice: measured 5 % faster on the
    // 6-tile encode).  Wider plans get 8-wave workgroups (two waves per SIMD at 256 registers): 128-token tiles with four waves
    // across the coordinates up to 640 of them, twice as fast as 4 waves of 512 registers; 64-token tiles with eight waves
    // across up to 1024, the basis straight to their registers (1024 of 4096 features, 32768 tokens: 390 us as 4 waves of 512, 340 with the basis
    // by way of LDS, 285 so; eight waves of two tiles on 128 tokens that way for 448 to 512 coordinates: 4 % slower than these).
    // {waves across coordinates, tiles per wave, workgroups per compute unit, waves per workgroup}, ascending padded width
    static const int enc_tab[][4] = {{1, 2, 2, 4}, {1, 4, 2, 4}, {2, 3, 3, 4}, {2, 4, 2, 4}, {2, 5, 2, 4},
                                     {4, 3, 1, 8}, {4, 4, 1, 8}, {4, 5, 1, 8}, {8, 3, 1, 8}, {8, 4, 1, 8}};
    d.enc_wc = 0;
    for (auto& e : enc_tab)
        if (e[0] * e[1] >= nt) { d.enc_wc = e[0]; d.enc_ntw = e[1]; d.enc_wgs = e[2]; d.enc_nw = e[3]; break; }
    // decode: the widths the kernels are built for, with the register class (= its widest member) that serves each;
    // odd widths where the calibrated plans of the 8B-shaped cache fall (224 = 7, 272 = 9, 528 = 17 tiles): in decode
    // the coordinates are the contraction index, so a tile less is that much less matrix work and basis traffic
    // {token tiles per wave (of the wide kernels, class above 10: per workgroup), coordinate tiles, class, workgroups per compute unit}
    static const int dec_tab[][4] = {{2, 2, 4, 3}, {2, 4, 4, 3}, {2, 6, 10, 2}, {2, 7, 10, 2}, {2, 8, 10, 2}, {2, 9, 10, 2}, {2, 10, 10, 2},
                                     {4, 12, 18, 1}, {4, 14, 18, 1}, {4, 16, 18, 1}, {4, 18, 18, 1}, {2, 20, 32, 1}, {2, 24, 32, 1}, {2, 28, 32, 1}, {2, 32, 32, 1}};
    d.dec_tt = 0;
    for (auto& e : dec_tab)
        if (e[1] >= nt) { d.dec_tt = e[0]; d.dec_nct = e[1]; d.dec_cls = e[2]; d.dec_wgs = e[3]; break; }
    if (d.enc_wc == 0 || d.dec_tt == 0) return fail(KVTC_E_UNSUPPORTED, "kvtc_plan_create: no kernel variant for r=%d", r);
    const int ntp = d.enc_ntw * d.enc_wc;
    d.enc_tok_wg = encode_tok_wg(d.enc_ntw, d.enc_wc, d.enc_nw);
    const bool dec_wide = d.dec_cls > 10;
    d.dec_tok_wg = (dec_wide ? 1 : 4) * 32 * d.dec_tt;
    {
        d.enc_lds[KVTC_BF16] = encode_lds_bytes(d.enc_ntw, d.enc_wc, d.enc_nw, n_groups, d.rec_dwords, KVTC_BF16);
        d.enc_lds[KVTC_F32] = encode_lds_bytes(d.enc_ntw, d.enc_wc, d.enc_nw, n_groups, d.rec_dwords, KVTC_F32);
        d.dec_rec_lds = dec_wide ? decode_wide_bytes(d.dec_tt, d.dec_nct, d.rec_dwords) : decode_rec_bytes(d.dec_tt, d.rec_dwords);
        d.dec_ring_lds = dec_wide ? 0 : decode_ring_bytes(d.dec_nct);
    }
    const int lds_cap = kLdsBudget - kJobTableBytes - 64;
    // the record sizes a plan may have: those whose image of 256 tokens (128 beyond 768 coordinates) fits the LDS, also where
    // the wide kernels would get by with less
    const int dec_limit = decode_rec_bytes(d.dec_nct > 24 ? 1 : 2, d.rec_dwords);
    const int dec_need = std::max(std::max(d.dec_rec_lds, d.dec_ring_lds), dec_limit);
    if (d.enc_lds[0] > lds_cap || d.enc_lds[1] > lds_cap || dec_need > lds_cap)
        return fail(KVTC_E_UNSUPPORTED,
                    "kvtc_plan_create: record of %d bytes with r=%d needs %d/%d/%d bytes of LDS, %d available",
                    d.rec_dwords * 4, r, d.enc_lds[0], d.enc_lds[1], dec_need, lds_cap);

    // the short-job kernel, where it serves the width and its images fit
    int s_waves = 0, s_lds[2] = {0, 0};
    d.enc_short = encode_short_ntw(ntp);
    if (d.enc_short != 0) {
        s_waves = encode_short_waves(ntp);
        s_lds[KVTC_BF16] = encode_short_lds_bytes(ntp, n_groups, d.rec_dwords, KVTC_BF16);
        s_lds[KVTC_F32] = encode_short_lds_bytes(ntp, n_groups, d.rec_dwords, KVTC_F32);
        if (s_lds[0] > kLdsBudget || s_lds[1] > kLdsBudget) d.enc_short = 0;
    }

    const int p_waves = share_groups(&d, groups_host);
    int p_lds[2] = {0, 0};
    if (d.enc_parts != 0) {
        p_lds[KVTC_BF16] = encode_part_lds_bytes(p, ntp, n_groups, d.rec_dwords, KVTC_BF16);
        p_lds[KVTC_F32] = encode_part_lds_bytes(p, ntp, n_groups, d.rec_dwords, KVTC_F32);
    }

    // ---- host images ---------------------------------------------------------------
    const size_t n_venc = (size_t)(p / 16) * ntp * 64 * 8;      // bf16 elements
    const int stage_u4 = decode_stage_u4(d.dec_nct);              // fragments of a 32-feature tile, then its mu entries
    const size_t n_vdec = (size_t)(p / 32) * stage_u4 * 8;
    std::vector<uint16_t> venc, vdec;
    std::vector<float> negc, mu;
    std::vector<uint32_t> blk(64, 0u), grp(64, 0u);      // whole tables: the kernels fetch all 64 entries
    try {
        venc.assign(n_venc, 0);
        vdec.assign(n_vdec, 0);
        negc.assign((size_t)32 * ntp, 0.0f);
        mu.assign(mu_host, mu_host + p);
    } catch (const std::bad_alloc&) {
        return fail(KVTC_E_NOMEM, "kvtc_plan_create: host allocation failed");
    }
    for (int ks = 0; ks < p / 16; ++ks)
        for (int ct = 0; ct < ntp; ++ct)
            for (int lane = 0; lane < 64; ++lane) {
                const int j = 32 * ct + permuted_index(lane & 31);
                if (j >= r) continue;
                uint16_t* dst = &venc[(((size_t)ks * ntp + ct) * 64 + lane) * 8];
                const int f0 = 16 * ks + 8 * (lane >> 5);
                for (int e = 0; e < 8; ++e) dst[e] = v_kept_host[(size_t)(f0 + e) * ldv + j];
            }
    for (int ft = 0; ft < p / 32; ++ft)
        for (int ks = 0; ks < 2 * d.dec_nct; ++ks)
            for (int lane = 0; lane < 64; ++lane) {
                // tiles 2k and 2k+1 hold the even and the odd features of a 64-feature span
                const int f = 64 * (ft >> 1) + 2 * (lane & 31) + (ft & 1);
                const int j0 = 32 * (ks >> 1) + 16 * (lane >> 5) + 8 * (ks & 1);
                uint16_t* dst = &vdec[(((size_t)ft * stage_u4) + (size_t)ks * 64 + lane) * 8];
                for (int e = 0; e < 8; ++e)
                    if (j0 + e < r) dst[e] = v_kept_host[(size_t)f * ldv + j0 + e];
            }
    for (int ft = 0; ft < p / 32; ++ft) {
        float m[32];
        for (int l = 0; l < 32; ++l) m[l] = dec_zero_mu ? 0.0f : mu_host[64 * (ft >> 1) + 2 * l + (ft & 1)];      // the lane order of the tile
        memcpy(&vdec[((size_t)ft * stage_u4 + (size_t)2 * d.dec_nct * 64) * 8], m, sizeof(m));
    }
    for (int j = 0; j < r; ++j) {
        double c = 0.0;
        for (int f = 0; f < p; ++f) c += (double)mu_host[f] * (double)bf16_bits_to_float(v_kept_host[(size_t)f * ldv + j]);
        negc[j] = -(float)c;
    }
    {
        int b = 0;
        long pos = 32L * n_groups;       // bit position of the group's first code
        for (int g = 0; g < n_groups; ++g) {
            const int nb = groups_host[g].n / 16, bits = groups_host[g].bits;
            grp[g] = (uint32_t)b | ((uint32_t)nb << 8) | ((uint32_t)bits << 16);
            for (int k = 0; k < nb; ++k) {
                blk[b + k] = (uint32_t)bits | ((uint32_t)g << 8) | ((uint32_t)(pos / 16) << 16);
                pos += 16L * bits;
            }
            b += nb;
        }
    }

    // ---- one device blob -------------------------------------------------------------
    size_t off = 0;
    const size_t o_desc = off;  off = align_up(off + sizeof(PlanDev), 256);
    const size_t o_venc = off;  off = align_up(off + n_venc * 2, 256);
    const size_t o_vdec = off;  off = align_up(off + n_vdec * 2, 256);
    const size_t o_negc = off;  off = align_up(off + negc.size() * 4, 256);
    const size_t o_mu = off;    off = align_up(off + mu.size() * 4, 256);
    const size_t o_blk = off;   off = align_up(off + blk.size() * 4, 256);
    const size_t o_grp = off;   off = align_up(off + grp.size() * 4, 256);
    char* blob = nullptr;
    if (hipMalloc(reinterpret_cast<void**>(&blob), off) != hipSuccess) {
        (void)hipGetLastError();
        return fail(KVTC_E_NOMEM, "kvtc_plan_create: hipMalloc of %zu bytes failed", off);
    }
    d.v_enc = reinterpret_cast<const uint4*>(blob + o_venc);
    d.v_dec = reinterpret_cast<const uint4*>(blob + o_vdec);
    d.negc = reinterpret_cast<const float*>(blob + o_negc);
    d.mu = reinterpret_cast<const float*>(blob + o_mu);
    d.blk = reinterpret_cast<const uint32_t*>(blob + o_blk);
    d.grp = reinterpret_cast<const uint32_t*>(blob + o_grp);
    hipStream_t st = static_cast<hipStream_t>(stream);
    hipError_t e = hipSuccess;
    auto put = [&](size_t o, const void* src, size_t n) {
        if (e == hipSuccess) e = hipMemcpyAsync(blob + o, src, n, hipMemcpyHostToDevice, st);
    };
    put(o_desc, &d, sizeof(d));
    put(o_venc, venc.data(), n_venc * 2);
    put(o_vdec, vdec.data(), n_vdec * 2);
    put(o_negc, negc.data(), negc.size() * 4);
    put(o_mu, mu.data(), mu.size() * 4);
    put(o_blk, blk.data(), blk.size() * 4);
    put(o_grp, grp.data(), grp.size() * 4);
    if (e == hipSuccess) e = hipStreamSynchronize(st);    // the host images die with this call
    if (e != hipSuccess) {
        (void)hipFree(blob);
        return fail(KVTC_E_HIP, "kvtc_plan_create: upload failed: %s", hipGetErrorString(e));
    }
    kvtc_plan* pl = new (std::nothrow) kvtc_plan;
    if (!pl) {
        (void)hipFree(blob);
        return fail(KVTC_E_NOMEM, "kvtc_plan_create: host allocation failed");
    }
    pl->h = d;
    pl->blob = blob;
    pl->desc_dev = reinterpret_cast<PlanDev*>(blob + o_desc);
    pl->record_bytes = (size_t)d.rec_dwords * 4;
    pl->enc_s_waves = s_waves;
    pl->enc_s_lds[0] = s_lds[0];
    pl->enc_s_lds[1] = s_lds[1];
    pl->enc_p_waves = p_waves;
    pl->enc_p_lds[0] = p_lds[0];
    pl->enc_p_lds[1] = p_lds[1];
    *out = pl;
    return KVTC_OK;
}

void kvtc_plan_destroy(kvtc_plan* plan) {
    if (!plan) return;
    (void)hipFree(plan->blob);
    delete plan;
}

size_t kvtc_record_bytes(const kvtc_plan* plan) { return plan ? plan->record_bytes : 0; }

size_t kvtc_encoded_bytes(const kvtc_plan* plan, int64_t n_tokens) {
    return (plan && n_tokens > 0) ? plan->record_bytes * (size_t)n_tokens : 0;
}

static kvtc_status check_x(const char* who, const void* x, kvtc_dtype dtype, int64_t ld_x, int p) {
    if (!dtype_ok(dtype)) return fail(KVTC_E_ARG, "%s: unknown dtype %d", who, (int)dtype);
    if (ld_x < p) return fail(KVTC_E_ARG, "%s: ld_x=%lld < p=%d", who, (long long)ld_x, p);
    if (ld_x > kMaxPitch) return fail(KVTC_E_ARG, "%s: ld_x=%lld above %d", who, (long long)ld_x, kMaxPitch);
    if ((reinterpret_cast<uintptr_t>(x) & 15u) || ((size_t)ld_x * elem_size(dtype)) % 16 != 0)
        return fail(KVTC_E_ARG, "%s: feature array base and row pitch must be 16-byte aligned", who);
    return KVTC_OK;
}

// A feature layout as the kernels take it: token stride, log2 of the block size (0 = contiguous features), and the
// gap between a block's end and the token's next block.
struct XLayout { int64_t ld; int32_t blk_log2; int64_t blk_jump; };

// Whether the 128 bytes of a row that a kernel asks for or writes at once are always one cache line (a row's offset is a multiple of the pitch; what
// precedes a block in its row is whole pieces of 64 features and gaps between blocks).  The kernels pass the caches by only then: a piece on two
// lines is two parts of lines, and every line would be fetched again or written in parts.  150000 tokens of bf16 with rows of 2064 bytes, us, kept by
// the caches and past them: decode of 64, 128, 240 and 272 coordinates 111, 119, 140 and 142 against 315, 313, 320 and 321; encode of 64, 128 and 240
// 87, 120 and 132 against 106, 133 and 147 (of 272 174 against 151, with rows of 2048 bytes on an odd base 145 against 155).
static bool whole_lines(const void* x, kvtc_dtype dtype, const XLayout& xl) {
    const uint64_t eb = elem_size(dtype);
    return ((reinterpret_cast<uintptr_t>(x) | (uint64_t)xl.ld * eb | (uint64_t)xl.blk_jump * eb) & 127u) == 0;
}

// KernelArgs::x_pass_from of a launch whose variant passes the caches from `from` bytes of the call's features on: a tensor of `elements`, or a batch,
// whose elements are on the device and can't be more than that.
static float pass_from(bool lines, uint64_t from, kvtc_dtype dtype, uint64_t elements, bool batch) {
    const bool may = lines && from / elem_size(dtype) <= elements;
    return !may ? HUGE_VALF : batch ? (float)(from / elem_size(dtype)) : 0.0f;
}
// Bytes of the basis that a decode with this plan reads.
static uint64_t basis_bytes(const PlanDev& h) { return (uint64_t)h.p * (uint64_t)h.dec_nct * 64u; }
// Tokens of a batch at most, by the size of its stream buffer (jobs do not overlap there), times features.
static uint64_t most_elements(size_t stream_bytes, int min_rec_dwords, int max_p) {
    return (uint64_t)(stream_bytes / ((size_t)min_rec_dwords * 4)) * (uint64_t)max_p;
}

// Checks a kvtc_layout for a tensor of p features (n_tokens < 0: unknown, as in a batched call) and converts it.
static kvtc_status check_layout(const char* who, const void* x, kvtc_dtype dtype, const kvtc_layout* lay, int p, int64_t n_tokens,
                                XLayout* out) {
    if (!lay) return fail(KVTC_E_ARG, "%s: null layout", who);
    if (!dtype_ok(dtype)) return fail(KVTC_E_ARG, "%s: unknown dtype %d", who, (int)dtype);
    const int bf = lay->block_features;
    const int64_t ts = lay->token_stride, bs = lay->block_stride;
    if (bf == 0) {
        kvtc_status st = check_x(who, x, dtype, ts, p);
        if (st != KVTC_OK) return st;
        *out = XLayout{ts, 0, 0};
        return KVTC_OK;
    }
    if (bf < 64 || (bf & (bf - 1)) != 0 || p % bf != 0)
        return fail(KVTC_E_ARG, "%s: block_features=%d must be a power of two, at least 64, that divides p=%d", who, bf, p);
    if (ts < bf || ts > kMaxPitch) return fail(KVTC_E_ARG, "%s: token_stride=%lld outside %d..%d", who, (long long)ts, bf, kMaxPitch);
    if (bs < bf) return fail(KVTC_E_ARG, "%s: block_stride=%lld < block_features=%d", who, (long long)bs, bf);
    const size_t eb = elem_size(dtype);
    if ((reinterpret_cast<uintptr_t>(x) & 15u) || ((size_t)ts * eb) % 16 != 0 || ((size_t)bs * eb) % 16 != 0)
        return fail(KVTC_E_ARG, "%s: feature array base, token stride and block stride must be 16-byte aligned", who);
    // blocks inside a token's row, or tokens inside a block's slab: anything else lets elements overlap
    const int nb = p / bf;
    const bool tokens_major = ts >= (int64_t)(nb - 1) * bs + bf;
    const bool blocks_major = n_tokens < 0 ? bs >= ts : bs >= (n_tokens - 1) * ts + bf;
    if (!tokens_major && !blocks_major)
        return fail(KVTC_E_ARG, "%s: strides (token %lld, block %lld) let elements overlap", who, (long long)ts, (long long)bs);
    int lg = 0;
    while ((1 << lg) < bf) ++lg;
    *out = XLayout{ts, lg, bs - bf};
    return KVTC_OK;
}

static kvtc_status encode_single(const char* who, const kvtc_plan* plan, const void* x_dev, kvtc_dtype dtype, int64_t n_tokens,
                                 const kvtc_layout* layout, void* out_dev, size_t out_cap, kvtc_stream stream);
static kvtc_status decode_single(const char* who, const kvtc_plan* plan, const void* in_dev, size_t in_bytes, int64_t n_tokens,
                                 void* x_out_dev, kvtc_dtype dtype, const kvtc_layout* layout, kvtc_stream stream, int accumulate = 0,
                                 const float* sum_dev = nullptr, int64_t sum_ld = 0);

uint64_t kvtc_host_encode_pass_bytes(int tiles, kvtc_dtype dtype) { return encode_pass_bytes(tiles, dtype); }
uint64_t kvtc_host_decode_pass_bytes(int tiles, kvtc_dtype dtype, uint64_t bases, int single) {
    return decode_pass_bytes(tiles <= 4 ? 4 : tiles <= 10 ? 10 : 18, tiles, dtype, bases, single != 0);
}
int kvtc_host_whole_lines(uint64_t x_address, kvtc_dtype dtype, int p, const kvtc_layout* layout) {
    XLayout xl;
    const void* x = reinterpret_cast<const void*>(static_cast<uintptr_t>(x_address));
    return check_layout("kvtc_host_whole_lines", x, dtype, layout, p, -1, &xl) == KVTC_OK ? (int)whole_lines(x, dtype, xl) : -1;
}

kvtc_status kvtc_encode(const kvtc_plan* plan, const void* x_dev, kvtc_dtype dtype, int64_t n_tokens, int64_t ld_x,
                        void* out_dev, size_t out_cap, kvtc_stream stream) {
    const kvtc_layout lay = {ld_x, 0, 0, 0};
    return encode_single("kvtc_encode", plan, x_dev, dtype, n_tokens, &lay, out_dev, out_cap, stream);
}
kvtc_status kvtc_encode_blocked(const kvtc_plan* plan, const void* x_dev, kvtc_dtype dtype, int64_t n_tokens,
                                const kvtc_layout* layout, void* out_dev, size_t out_cap, kvtc_stream stream) {
    return encode_single("kvtc_encode_blocked", plan, x_dev, dtype, n_tokens, layout, out_dev, out_cap, stream);
}
kvtc_status kvtc_decode(const kvtc_plan* plan, const void* in_dev, size_t in_bytes, int64_t n_tokens, void* x_out_dev,
                        kvtc_dtype dtype, int64_t ld_x, kvtc_stream stream) {
    const kvtc_layout lay = {ld_x, 0, 0, 0};
    return decode_single("kvtc_decode", plan, in_dev, in_bytes, n_tokens, x_out_dev, dtype, &lay, stream);
}
kvtc_status kvtc_decode_blocked(const kvtc_plan* plan, const void* in_dev, size_t in_bytes, int64_t n_tokens, void* x_out_dev,
                                kvtc_dtype dtype, const kvtc_layout* layout, kvtc_stream stream) {
    return decode_single("kvtc_decode_blocked", plan, in_dev, in_bytes, n_tokens, x_out_dev, dtype, layout, stream);
}

static kvtc_status encode_single(const char* who, const kvtc_plan* plan, const void* x_dev, kvtc_dtype dtype, int64_t n_tokens,
                                 const kvtc_layout* layout, void* out_dev, size_t out_cap, kvtc_stream stream) {
    if (!plan) return fail(KVTC_E_ARG, "kvtc_encode: null plan");
    if (n_tokens < 0 || n_tokens > 0x7fffffffLL) return fail(KVTC_E_ARG, "kvtc_encode: n_tokens=%lld", (long long)n_tokens);
    if (n_tokens == 0) return KVTC_OK;
    if (!x_dev || !out_dev) return fail(KVTC_E_ARG, "kvtc_encode: null buffer");
    XLayout xl;
    kvtc_status st = check_layout(who, x_dev, dtype, layout, plan->h.p, n_tokens, &xl);
    if (st != KVTC_OK) return st;
    if (reinterpret_cast<uintptr_t>(out_dev) & 15u) return fail(KVTC_E_ARG, "kvtc_encode: out_dev must be 16-byte aligned");
    if (out_cap < plan->record_bytes * (size_t)n_tokens)
        return fail(KVTC_E_SMALL, "kvtc_encode: out_cap=%zu < %zu", out_cap, plan->record_bytes * (size_t)n_tokens);
    KernelArgs a;
    memset(&a, 0, sizeof(a));
    a.plans = plan->desc_dev;
    a.n_plans = 1;
    a.jobs = nullptr;
    a.n_jobs = 1;
    a.single = kvtc_job{0, (int32_t)n_tokens, 0};
    a.offsets = nullptr;
    a.x = x_dev;
    a.ld_x = xl.ld;
    a.x_blk_log2 = xl.blk_log2;
    a.x_blk_jump = xl.blk_jump;
    a.stream_buf = out_dev;
    a.cap = out_cap;
    a.status = nullptr;
    // A tensor short enough for all its 64-token tiles to run at once (one wave of workgroups) runs the short-job kernel.
    const int64_t tiles_short = (n_tokens + kEncShortTile - 1) / kEncShortTile;
    hipError_t e;
    // One shorter still, up to a workgroup for every compute unit, or, where two share one, half as many again, has its tiles' groups shared out as well.  (Tensors of
    // 48, 2700 and 4000 tokens at 16x, us: 12.9, 13.6 and 13.7 on the short-job kernel, 7.8, 8.9 and 12.1 so; of 5400 13.9 and 13.5, at 20x 13.1 and 13.3; fp32 of 4000, one
    // workgroup to a compute unit, 16.3 and 20.8.)
    const int64_t tiles_part = (n_tokens + kEncPartTile - 1) / kEncPartTile;
    if (plan->h.enc_parts != 0 && plan->enc_p_lds[dtype] != 0 &&
        2 * tiles_part * plan->h.enc_parts <= part_places(plan->enc_p_waves, plan->enc_p_lds[dtype]) + compute_units()) {
        a.enc_split = plan->h.enc_parts;
        e = launch_encode_parts(a, dtype, plan->enc_p_waves, plan->h.p, (int)tiles_part * plan->h.enc_parts, (size_t)plan->enc_p_lds[dtype], static_cast<hipStream_t>(stream));
    } else if (plan->h.enc_short != 0 && tiles_short <= short_tiles_per_job(1, short_pairs(plan->h.enc_short, plan->enc_s_waves, plan->enc_s_lds[dtype]))) {
        e = launch_encode_short(a, dtype, plan->h.enc_short, plan->enc_s_waves, (int)tiles_short, (size_t)plan->enc_s_lds[dtype], static_cast<hipStream_t>(stream));
    } else {
        const int64_t tiles = (n_tokens + plan->h.enc_tok_wg - 1) / plan->h.enc_tok_wg;
        a.single_tiles = (uint32_t)tiles;
        a.x_pass_from = pass_from(whole_lines(x_dev, dtype, xl), encode_pass_bytes(plan->h.enc_ntw * plan->h.enc_wc, dtype), dtype, (uint64_t)n_tokens * (uint64_t)plan->h.p, false);
        const int slots = compute_units() * plan->h.enc_wgs;
        const int grid = (int)(tiles < slots ? tiles : slots);
        e = launch_encode(a, dtype, plan->h.enc_nw * 10000 + plan->h.enc_wc * 100 + plan->h.enc_ntw, grid, (size_t)kJobTableBytes + 64 + plan->h.enc_lds[dtype], static_cast<hipStream_t>(stream));
    }
    if (e != hipSuccess) return fail(KVTC_E_HIP, "kvtc_encode: launch failed: %s", hipGetErrorString(e));
    return KVTC_OK;
}

static kvtc_status decode_single(const char* who, const kvtc_plan* plan, const void* in_dev, size_t in_bytes, int64_t n_tokens,
                                 void* x_out_dev, kvtc_dtype dtype, const kvtc_layout* layout, kvtc_stream stream, int accumulate,
                                 const float* sum_dev, int64_t sum_ld) {
    if (!plan) return fail(KVTC_E_ARG, "kvtc_decode: null plan");
    // accumulate: 0 = store; 1 = add into the fp32 output; 2 = bf16 output = round(sum_dev + product)
    if ((accumulate == 1 && dtype != KVTC_F32) || (accumulate == 2 && (dtype != KVTC_BF16 || !sum_dev || sum_ld < plan->h.p)))
        return fail(KVTC_E_ARG, "%s: bad combination of section mode and output type", who);
    if (n_tokens < 0 || n_tokens > 0x7fffffffLL) return fail(KVTC_E_ARG, "kvtc_decode: n_tokens=%lld", (long long)n_tokens);
    if (n_tokens == 0) return KVTC_OK;
    if (!in_dev || !x_out_dev) return fail(KVTC_E_ARG, "kvtc_decode: null buffer");
    XLayout xl;
    kvtc_status st = check_layout(who, x_out_dev, dtype, layout, plan->h.p, n_tokens, &xl);
    if (st != KVTC_OK) return st;
    if (reinterpret_cast<uintptr_t>(in_dev) & 15u) return fail(KVTC_E_ARG, "kvtc_decode: in_dev must be 16-byte aligned");
    if (in_bytes < plan->record_bytes * (size_t)n_tokens)
        return fail(KVTC_E_SMALL, "kvtc_decode: in_bytes=%zu < %zu", in_bytes, plan->record_bytes * (size_t)n_tokens);
    KernelArgs a;
    memset(&a, 0, sizeof(a));
    a.plans = plan->desc_dev;
    a.n_plans = 1;
    a.n_jobs = 1;
    a.single = kvtc_job{0, (int32_t)n_tokens, 0};
    a.x = x_out_dev;
    a.ld_x = xl.ld;
    a.x_blk_log2 = xl.blk_log2;
    a.x_blk_jump = xl.blk_jump;
    a.stream_buf = const_cast<void*>(in_dev);
    a.cap = in_bytes;
    a.dec_accumulate = accumulate;
    a.dec_sum = sum_dev;
    a.dec_sum_ld = sum_ld;
    const int slots = compute_units() * plan->h.dec_wgs;
    // A tensor short enough for all its 128-token tiles to run at once takes the variant with one token
    // tile per wave (same plan data: it depends on the padded width only).  The workgroups beyond a launch's tiles
    // share the tiles' features (at most one workgroup per 64 of them).
    const int64_t spans = plan->h.p / 64;
    const int64_t tiles_short = (n_tokens + kDecShortTile - 1) / kDecShortTile;
    hipError_t e;
    const bool wide = plan->h.dec_cls > 10;
    if (!wide && tiles_short <= slots) {
        const DecLayout lay = decode_layout(decode_rec_bytes(1, plan->h.rec_dwords), plan->h.dec_ring_lds, plan->h.dec_wgs);
        a.dec_ring_off = lay.ring_off;
        a.dec_short = 1;
        a.single_tiles = (uint32_t)tiles_short;
        a.x_pass_from = HUGE_VALF;
        const int grid = (int)(tiles_short * spans < slots ? tiles_short * spans : slots);
        e = launch_decode(a, dtype, 100 + plan->h.dec_cls, grid, lay.lds_bytes, static_cast<hipStream_t>(stream));
    } else {
        const int64_t tiles = (n_tokens + plan->h.dec_tok_wg - 1) / plan->h.dec_tok_wg;
        a.single_tiles = (uint32_t)tiles;
        a.x_pass_from = pass_from(whole_lines(x_out_dev, dtype, xl), decode_pass_bytes(plan->h.dec_cls, plan->h.dec_nct, dtype, basis_bytes(plan->h), true), dtype,
                                  (uint64_t)n_tokens * (uint64_t)plan->h.p, false);
        const int64_t shares = wide ? (spans < 4 ? 1 : spans / 4) : spans;       // workgroups a tile may be shared among
        const int grid = (int)(tiles * shares < slots ? tiles * shares : slots);
        const DecLayout lay = decode_layout(plan->h.dec_rec_lds, plan->h.dec_ring_lds, plan->h.dec_wgs);
        a.dec_ring_off = lay.ring_off;
        e = launch_decode(a, dtype, plan->h.dec_tt * 100 + plan->h.dec_cls, grid, lay.lds_bytes, static_cast<hipStream_t>(stream));
    }
    if (e != hipSuccess) return fail(KVTC_E_HIP, "kvtc_decode: launch failed: %s", hipGetErrorString(e));
    return KVTC_OK;
}

kvtc_status kvtc_batch_create(kvtc_batch** out, const kvtc_plan* const* plans, int n_plans, kvtc_stream stream) {
    if (out) *out = nullptr;
    if (!out || !plans || n_plans < 1) return fail(KVTC_E_ARG, "kvtc_batch_create: null argument or no plans");
    std::vector<PlanDev> h;
    kvtc_batch* b = new (std::nothrow) kvtc_batch;
    if (!b) return fail(KVTC_E_NOMEM, "kvtc_batch_create: host allocation failed");
    b->plans_dev = nullptr;
    b->rec_dwords_dev = nullptr;
    b->n_plans = n_plans;
    b->max_p = 0;
    b->min_rec_dwords = 1 << 30;
    b->all_short = true;
    for (auto& v : b->enc_short) v = {0, {0, 0}};
    try {
    for (int i = 0; i < n_plans; ++i) {
        if (!plans[i]) {
            delete b;
            return fail(KVTC_E_ARG, "kvtc_batch_create: plan %d is null", i);
        }
        h.push_back(plans[i]->h);
        b->rec_dwords.push_back(plans[i]->h.rec_dwords);
        const PlanDev& ph = plans[i]->h;
        b->min_rec_dwords = std::min(b->min_rec_dwords, ph.rec_dwords);
        b->all_short = b->all_short && ph.enc_short != 0;
        for (const kvtc_dtype dt : {KVTC_BF16, KVTC_F32}) b->enc_part[dt].add(*plans[i], dt);
        {
            const int key = ph.enc_nw * 10000 + ph.enc_wc * 100 + ph.enc_ntw;
            kvtc_batch::EncVariant* v = nullptr;
            for (auto& e : b->enc)
                if (e.key == key) v = &e;
            if (!v) {
                b->enc.push_back({key, ph.enc_wgs, {0, 0}});
                v = &b->enc.back();
            }
            for (int dt = 0; dt < 2; ++dt)
                if (ph.enc_lds[dt] > v->lds[dt]) v->lds[dt] = ph.enc_lds[dt];
        }
        if (ph.enc_short != 0) {
            auto& v = b->enc_short[ph.enc_short];
            if (plans[i]->enc_s_waves > v.waves) v.waves = plans[i]->enc_s_waves;
            for (int dt = 0; dt < 2; ++dt)
                if (plans[i]->enc_s_lds[dt] > v.lds[dt]) v.lds[dt] = plans[i]->enc_s_lds[dt];
        }
        {
            const int key = ph.dec_tt * 100 + ph.dec_cls;
            kvtc_batch::DecVariant* v = nullptr;
            for (auto& e : b->dec)
                if (e.key == key) v = &e;
            if (!v) {
                b->dec.push_back({key, ph.dec_wgs, 0, 0, 0, ph.dec_nct, 0});
                v = &b->dec.back();
            }
            if (ph.dec_rec_lds > v->rec) v->rec = ph.dec_rec_lds;
            if (ph.rec_dwords > v->rec_dwords) v->rec_dwords = ph.rec_dwords;
            if (ph.dec_ring_lds > v->ring) v->ring = ph.dec_ring_lds;
            v->least_tiles = std::min(v->least_tiles, ph.dec_nct);
            v->bases += basis_bytes(ph);
        }
        if (ph.p > b->max_p) b->max_p = ph.p;
        {
            bool seen = false;
            for (int v : b->ps) seen = seen || v == ph.p;
            if (!seen) b->ps.push_back(ph.p);
        }
    }
    } catch (const std::bad_alloc&) {
        delete b;
        return fail(KVTC_E_NOMEM, "kvtc_batch_create: host allocation failed");
    }
    hipStream_t st = static_cast<hipStream_t>(stream);
    hipError_t e = hipMalloc(reinterpret_cast<void**>(&b->plans_dev), sizeof(PlanDev) * n_plans);
    if (e == hipSuccess) e = hipMalloc(reinterpret_cast<void**>(&b->rec_dwords_dev), sizeof(uint32_t) * n_plans);
    if (e != hipSuccess) {
        (void)hipGetLastError();
        kvtc_batch_destroy(b);
        return fail(KVTC_E_NOMEM, "kvtc_batch_create: hipMalloc failed");
    }
    e = hipMemcpyAsync(b->plans_dev, h.data(), sizeof(PlanDev) * n_plans, hipMemcpyHostToDevice, st);
    if (e == hipSuccess)
        e = hipMemcpyAsync(b->rec_dwords_dev, b->rec_dwords.data(), sizeof(uint32_t) * n_plans, hipMemcpyHostToDevice, st);
    if (e == hipSuccess) e = hipStreamSynchronize(st);
    if (e != hipSuccess) {
        kvtc_batch_destroy(b);
        return fail(KVTC_E_HIP, "kvtc_batch_create: upload failed: %s", hipGetErrorString(e));
    }
    *out = b;
    return KVTC_OK;
}

void kvtc_batch_destroy(kvtc_batch* batch) {
    if (!batch) return;
    if (batch->plans_dev) (void)hipFree(batch->plans_dev);
    if (batch->rec_dwords_dev) (void)hipFree(batch->rec_dwords_dev);
    delete batch;
}

kvtc_status kvtc_offsets(const kvtc_batch* batch, const kvtc_job* jobs_dev, int n_jobs, uint64_t* offsets_dev,
                         kvtc_stream stream) {
    if (!batch || !offsets_dev || n_jobs < 0 || (n_jobs > 0 && !jobs_dev))
        return fail(KVTC_E_ARG, "kvtc_offsets: null argument or negative job count");
    hipLaunchKernelGGL(offsets_kernel, dim3(1), dim3(256), 0, static_cast<hipStream_t>(stream), batch->rec_dwords_dev,
                       batch->n_plans, jobs_dev, n_jobs, offsets_dev, static_cast<uint64_t*>(nullptr));
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return fail(KVTC_E_HIP, "kvtc_offsets: launch failed: %s", hipGetErrorString(e));
    return KVTC_OK;
}

kvtc_status kvtc_offsets_append(const kvtc_batch* batch, const kvtc_job* jobs_dev, int n_jobs, const uint64_t* region_dev,
                                const int64_t* n_coded_dev, uint64_t* offsets_dev, kvtc_stream stream) {
    if (!batch || !offsets_dev || !region_dev || n_jobs < 0 || (n_jobs > 0 && (!jobs_dev || !n_coded_dev)))
        return fail(KVTC_E_ARG, "kvtc_offsets_append: null argument or negative job count");
    hipError_t e = launch_offsets_append(batch->rec_dwords_dev, batch->n_plans, jobs_dev, n_jobs, region_dev, n_coded_dev, offsets_dev,
                                         static_cast<hipStream_t>(stream));
    if (e != hipSuccess) return fail(KVTC_E_HIP, "kvtc_offsets_append: launch failed: %s", hipGetErrorString(e));
    return KVTC_OK;
}

kvtc_status kvtc_window_split(int64_t ctx, int s, int w, int c, kvtc_split* out) {
    if (!out) return fail(KVTC_E_ARG, "kvtc_window_split: null output");
    if (ctx < 0 || s < 0 || c < 1 || c > w) return fail(KVTC_E_ARG, "kvtc_window_split: need ctx >= 0, s >= 0, 1 <= c <= w (ctx=%lld s=%d w=%d c=%d)", (long long)ctx, s, w, c);
    out->n_sink = ctx < s ? ctx : s;
    const int64_t beyond = ctx - s - (int64_t)(w - c);          // window tokens past the w - c that always stay
    out->n_coded = beyond > 0 ? (beyond / c) * c : 0;
    out->n_window = ctx - out->n_sink - out->n_coded;
    return KVTC_OK;
}

double kvtc_cr_with_window(double ctx, double w, double s, double cr) { return ctx / ((ctx - w - s) / cr + w + s / 2.0); }

kvtc_status kvtc_rope(void* x_dev, kvtc_dtype dtype, int64_t n_tokens, int n_heads, int d_head, int64_t token_stride,
                      int64_t head_stride, const int32_t* positions_dev, int64_t position0, double base, kvtc_rope_pairing pairing,
                      int inverse, kvtc_stream stream) {
    if (n_tokens < 0 || n_tokens > 0x7fffffffLL) return fail(KVTC_E_ARG, "kvtc_rope: n_tokens=%lld", (long long)n_tokens);
    if (n_heads < 1 || d_head < 2 || (d_head & 1) || d_head > 256)
        return fail(KVTC_E_ARG, "kvtc_rope: need n_heads >= 1 and an even d_head in 2..256 (n_heads=%d d_head=%d)", n_heads, d_head);
    if (!dtype_ok(dtype)) return fail(KVTC_E_ARG, "kvtc_rope: unknown dtype %d", (int)dtype);
    if (pairing != KVTC_ROPE_HALF && pairing != KVTC_ROPE_INTERLEAVED) return fail(KVTC_E_ARG, "kvtc_rope: unknown pairing %d", (int)pairing);
    if (!(base > 0.0) || !std::isfinite(base)) return fail(KVTC_E_ARG, "kvtc_rope: base must be positive and finite");
    if (inverse != 0 && inverse != 1) return fail(KVTC_E_ARG, "kvtc_rope: inverse must be 0 or 1");
    if (n_tokens == 0) return KVTC_OK;
    if (!x_dev) return fail(KVTC_E_ARG, "kvtc_rope: null buffer");
    // heads and tokens must not overlap: either tokens-major (a token's heads inside its row) or heads-major (a head's tokens inside its slab)
    const bool tokens_major = head_stride >= d_head && token_stride >= (int64_t)(n_heads - 1) * head_stride + d_head;
    const bool heads_major = token_stride >= d_head && head_stride >= (n_tokens - 1) * token_stride + d_head;
    if (!tokens_major && !heads_major)
        return fail(KVTC_E_ARG, "kvtc_rope: strides (token %lld, head %lld) let elements overlap", (long long)token_stride, (long long)head_stride);
    if (reinterpret_cast<uintptr_t>(x_dev) % elem_size(dtype) != 0) return fail(KVTC_E_ARG, "kvtc_rope: misaligned buffer");
    RopeArgs a;
    memset(&a, 0, sizeof(a));
    a.x = x_dev;
    a.n_tokens = n_tokens;
    a.token_stride = token_stride;
    a.head_stride = head_stride;
    a.positions = positions_dev;
    a.position0 = position0;
    a.n_heads = n_heads;
    a.d_head = d_head;
    a.inverse = inverse;
    for (int j = 0; j < d_head / 2; ++j) a.theta[j] = std::pow(base, -2.0 * (double)j / (double)d_head);
    const int64_t items = n_tokens * (int64_t)(d_head / 2);
    const int64_t want = (items + 255) / 256;
    const int64_t cap = (int64_t)compute_units() * 16;
    hipError_t e = launch_rope(a, dtype, pairing == KVTC_ROPE_INTERLEAVED, (int)(want < cap ? want : cap), static_cast<hipStream_t>(stream));
    if (e != hipSuccess) return fail(KVTC_E_HIP, "kvtc_rope: launch failed: %s", hipGetErrorString(e));
    return KVTC_OK;
}

kvtc_status kvtc_fp8_pack(const void* x_dev, kvtc_dtype dtype, int64_t n_tokens, int p, int64_t ld_x, void* out_dev, size_t out_cap,
                          kvtc_stream stream) {
    if (n_tokens < 0 || n_tokens > 0x7fffffffLL || p <= 0) return fail(KVTC_E_ARG, "kvtc_fp8_pack: n_tokens=%lld p=%d", (long long)n_tokens, p);
    if (n_tokens == 0) return KVTC_OK;
    if (!x_dev || !out_dev) return fail(KVTC_E_ARG, "kvtc_fp8_pack: null buffer");
    kvtc_status st = check_x("kvtc_fp8_pack", x_dev, dtype, ld_x, p);
    if (st != KVTC_OK) return st;
    if (out_cap < (size_t)n_tokens * (size_t)p) return fail(KVTC_E_SMALL, "kvtc_fp8_pack: out_cap=%zu < %zu", out_cap, (size_t)n_tokens * (size_t)p);
    hipError_t e = launch_fp8_pack(x_dev, dtype, n_tokens, p, ld_x, out_dev, static_cast<hipStream_t>(stream));
    if (e != hipSuccess) return fail(KVTC_E_HIP, "kvtc_fp8_pack: launch failed: %s", hipGetErrorString(e));
    return KVTC_OK;
}

kvtc_status kvtc_fp8_unpack(const void* in_dev, size_t in_bytes, int64_t n_tokens, int p, void* x_out_dev, kvtc_dtype dtype,
                            int64_t ld_x, kvtc_stream stream) {
    if (n_tokens < 0 || n_tokens > 0x7fffffffLL || p <= 0) return fail(KVTC_E_ARG, "kvtc_fp8_unpack: n_tokens=%lld p=%d", (long long)n_tokens, p);
    if (n_tokens == 0) return KVTC_OK;
    if (!in_dev || !x_out_dev) return fail(KVTC_E_ARG, "kvtc_fp8_unpack: null buffer");
    kvtc_status st = check_x("kvtc_fp8_unpack", x_out_dev, dtype, ld_x, p);
    if (st != KVTC_OK) return st;
    if (in_bytes < (size_t)n_tokens * (size_t)p) return fail(KVTC_E_SMALL, "kvtc_fp8_unpack: in_bytes=%zu < %zu", in_bytes, (size_t)n_tokens * (size_t)p);
    hipError_t e = launch_fp8_unpack(in_dev, n_tokens, p, x_out_dev, dtype, ld_x, static_cast<hipStream_t>(stream));
    if (e != hipSuccess) return fail(KVTC_E_HIP, "kvtc_fp8_unpack: launch failed: %s", hipGetErrorString(e));
    return KVTC_OK;
}

// The launches of a batched encode: the kernel variants among its plans.
struct EncodeLaunches {
    struct Bulk { int key, wgs, lds; } bulk[16];        // (a variant per row of the plans' table)
    int n_bulk;
    struct Short { int waves, lds; } shrt[3] = {};       // by coordinate tiles per wave; waves = 0: none
    PartVariant part;
    bool all_short;
    int min_rec_dwords, max_p;
    bool lines;                                          // the feature array lies on whole cache lines
};

static kvtc_status launch_encode_jobs(const char* who, const EncodeLaunches& l, KernelArgs& a, kvtc_dtype dtype, hipStream_t st) {
    const bool pairs = l.shrt[2].waves == 0 && short_pairs(1, l.shrt[1].waves, l.shrt[1].lds);
    const int grid = l.all_short ? short_table_grid(a.cap, l.min_rec_dwords, a.n_jobs, pairs) : 0;
    // By parts: where equal jobs would run at once -- with tiles of up to 32 tokens, which the short-job kernel also codes in half the time, one to a compute unit --
    // and so would jobs of mixed lengths; a lone share of many features in one workgroup to a compute unit, or two draw its basis in place of one.  Where jobs
    // may be more than that, the device counts them and codes them by parts or as the short-job kernel does, if the plans and the type have that kernel.  Plans of
    // two coordinate tiles to a wave, one workgroup of which a compute unit has room for, are faster by parts in two rounds as well.
    // (us, the short-job launch and by parts with a workgroup for each share.  At once: 64 tensors at 16x, room for 32 tokens each, all of 31 12.6 and 9.8, 48 and 16 in
    // turn 13.1 and 9.7; 256 heads of 16 to 48 6.4 and 5.6.  Not all at once: 128 of 256 features, 100 and 20 in turn, 7.1 and 9.5; 64 at 16x 15.1 and 16.8; in fp32 of 48 and
    // 16 in turn 17.8 and 18.9; 128 at 40x, one share each, of 64 12.3 and 11.7, of 32 to 96, 312 shares, 12.0 and 13.1 (counted 12.6); 64 of 512 coordinates, 100 and 20 in turn, 20.2 and 18.7.
    // Counted on the device: 64 at 16x, room for 64 tokens each, 16 coded, 12.0, 9.2 and 9.3, of 32 to 96 15.2, 16.8 and 15.5; in fp32 64 of 16 12.8 12.0 11.7, of 48 and 16 in turn 17.8, 18.9 and 17.3.)
    enum { kNot, kParts, kEither } by = kNot;
    const size_t cus = (size_t)compute_units(), places = (size_t)part_places(l.part.waves, l.part.lds);
    const PartShares ps = l.part.split > 0 ? part_shares(a.cap, l.min_rec_dwords, a.n_jobs, l.part.split) : PartShares{};
    const size_t at_once = l.part.split == 1 && l.max_p > 512 ? cus : places;
    const bool fours = dtype == KVTC_BF16 && l.part.waves == 4;        // (short-job kernels of one tile to a wave have ten of them at most)
    if (l.part.split > 0 && a.n_jobs <= kShortTableJobs && ps.equal <= (ps.each > kEncPartTile ? places : std::min(at_once, cus))) {
        const bool either = l.shrt[2].waves == 0 && grid != 0 && (l.part.split > 2 ? dtype == KVTC_BF16 || places == cus : fours && l.max_p > 512);
        if ((either ? ps.most : std::max(ps.equal, ps.mixed)) <= at_once || l.shrt[1].waves == 0) by = kParts;
        else if (either) by = kEither;
    }
    hipError_t e = hipSuccess;
    a.enc_split = l.part.split;
    if (by == kParts) {
        a.enc_table = 1;
        a.enc_max_tokens = (int32_t)(a.cap / ((size_t)l.min_rec_dwords * 4));
        e = launch_encode_parts(a, dtype, l.part.waves, l.max_p, whole_shares(std::min(ps.most, places)), (size_t)l.part.lds, st);
    } else if (by == kEither) {
        a.enc_table = 1;
        a.enc_max_tokens = (int32_t)(a.cap / ((size_t)l.min_rec_dwords * 4));
        const int lds = std::max(l.part.lds, l.shrt[1].lds);
        const int waves = fours ? 4 : std::max(l.part.waves, l.shrt[1].waves);
        a.enc_part_most = fours ? std::min(part_places(4, lds), (int)at_once) : (int)(short_pairs(1, waves, lds) ? cus * 3 / 2 : cus);
        e = launch_encode_short(a, dtype, !fours || l.shrt[1].waves <= 4 ? 1 : l.shrt[1].waves <= 8 ? 2 : 3, waves, std::max(grid, whole_shares((size_t)a.enc_part_most)), (size_t)lds, st);
    } else if (grid != 0) {
        // few tokens in all: one round of the short-job kernel
        a.enc_table = 1;
        a.enc_max_tokens = (int32_t)(a.cap / ((size_t)l.min_rec_dwords * 4));
        for (int ntw = 1; ntw <= 2 && e == hipSuccess; ++ntw)
            if (l.shrt[ntw].waves != 0) e = launch_encode_short(a, dtype, ntw, l.shrt[ntw].waves, grid, (size_t)l.shrt[ntw].lds, st);
    } else {
        // short jobs go to the short-job kernel, the rest to the bulk variants
        const int s_tiles = short_tiles_per_job(a.n_jobs, pairs);
        a.enc_short_max = s_tiles * kEncShortTile;
        a.enc_cus = compute_units();
        for (int k = 0; k < l.n_bulk && e == hipSuccess; ++k) {
            const int key = l.bulk[k].key, ntp = key / 100 % 100 * (key % 100);
            a.x_pass_from = pass_from(l.lines, encode_pass_bytes(ntp, dtype), dtype, most_elements(a.cap, l.min_rec_dwords, l.max_p), true);
            e = launch_encode(a, dtype, l.bulk[k].key, compute_units() * l.bulk[k].wgs, (size_t)kJobTableBytes + 64 + l.bulk[k].lds, st);
        }
        for (int ntw = 1; ntw <= 2 && e == hipSuccess; ++ntw)
            if (l.shrt[ntw].waves != 0) e = launch_encode_short(a, dtype, ntw, l.shrt[ntw].waves, a.n_jobs * s_tiles, (size_t)l.shrt[ntw].lds, st);
    }
    if (e != hipSuccess) return fail(KVTC_E_HIP, "%s: launch failed: %s", who, hipGetErrorString(e));
    return KVTC_OK;
}

static kvtc_status batch_common(const char* who, const kvtc_batch* batch, const kvtc_job* jobs_dev, int n_jobs,
                                const void* x, kvtc_dtype dtype, const kvtc_layout* layout, const uint64_t* offsets_dev,
                                const void* stream_buf, const uint32_t* status_dev, bool* nothing, XLayout* xl) {
    *nothing = false;
    if (!batch) return fail(KVTC_E_ARG, "%s: null batch", who);
    if (n_jobs < 0) return fail(KVTC_E_ARG, "%s: n_jobs=%d", who, n_jobs);
    if (n_jobs == 0) { *nothing = true; return KVTC_OK; }
    if (n_jobs > kMaxJobs) return fail(KVTC_E_UNSUPPORTED, "%s: %d jobs, at most %d per call", who, n_jobs, kMaxJobs);
    if (!jobs_dev || !x || !offsets_dev || !stream_buf || !status_dev) return fail(KVTC_E_ARG, "%s: null buffer", who);
    if (!layout) return fail(KVTC_E_ARG, "%s: null layout", who);
    for (int pv : batch->ps) {                         // the layout must suit every plan of the batch
        kvtc_status st = check_layout(who, x, dtype, layout, pv, -1, xl);
        if (st != KVTC_OK) return st;
    }
    if (reinterpret_cast<uintptr_t>(stream_buf) & 15u) return fail(KVTC_E_ARG, "%s: stream buffer must be 16-byte aligned", who);
    return KVTC_OK;
}

kvtc_status kvtc_encode_batch(const kvtc_batch* batch, const kvtc_job* jobs_dev, int n_jobs, const void* x_base_dev,
                              kvtc_dtype dtype, int64_t ld_x, const uint64_t* offsets_dev, void* out_base_dev,
                              size_t out_cap, uint32_t* status_dev, kvtc_stream stream) {
    const kvtc_layout lay = {ld_x, 0, 0, 0};
    return kvtc_encode_batch_blocked(batch, jobs_dev, n_jobs, x_base_dev, dtype, &lay, offsets_dev, out_base_dev, out_cap, status_dev, stream);
}

kvtc_status kvtc_encode_batch_blocked(const kvtc_batch* batch, const kvtc_job* jobs_dev, int n_jobs, const void* x_base_dev,
                                      kvtc_dtype dtype, const kvtc_layout* layout, const uint64_t* offsets_dev, void* out_base_dev,
                                      size_t out_cap, uint32_t* status_dev, kvtc_stream stream) {
    bool nothing;
    XLayout xl = {0, 0, 0};
    kvtc_status st = batch_common("kvtc_encode_batch", batch, jobs_dev, n_jobs, x_base_dev, dtype, layout, offsets_dev,
                                  out_base_dev, status_dev, &nothing, &xl);
    if (st != KVTC_OK || nothing) return st;
    const int64_t ld_x = xl.ld;
    KernelArgs a;
    memset(&a, 0, sizeof(a));
    a.plans = batch->plans_dev;
    a.n_plans = batch->n_plans;
    a.jobs = jobs_dev;
    a.n_jobs = n_jobs;
    a.offsets = offsets_dev;
    a.x = x_base_dev;
    a.ld_x = ld_x;
    a.x_blk_log2 = xl.blk_log2;
    a.x_blk_jump = xl.blk_jump;
    a.stream_buf = out_base_dev;
    a.cap = out_cap;
    a.status = status_dev;
    EncodeLaunches l;
    l.n_bulk = 0;
    l.all_short = batch->all_short;
    l.min_rec_dwords = batch->min_rec_dwords;
    l.max_p = batch->max_p;
    l.part = batch->enc_part[dtype];
    l.lines = whole_lines(x_base_dev, dtype, xl);
    for (int ntw = 1; ntw <= 2; ++ntw) l.shrt[ntw] = {batch->enc_short[ntw].waves, batch->enc_short[ntw].lds[dtype]};
    for (const auto& v : batch->enc) l.bulk[l.n_bulk++] = {v.key, v.wgs, v.lds[dtype]};
    return launch_encode_jobs("kvtc_encode_batch", l, a, dtype, static_cast<hipStream_t>(stream));
}

kvtc_status kvtc_encode_batch_static(const kvtc_plan* const* plans, int n_plans, const kvtc_job* jobs_dev, int n_jobs,
                                     const void* x_base_dev, kvtc_dtype dtype, int64_t ld_x, void* out_base_dev, size_t out_cap,
                                     uint64_t* offsets_out_dev, uint32_t* status_dev, kvtc_stream stream) {
    const char* who = "kvtc_encode_batch_static";
    if (!plans || n_plans < 1) return fail(KVTC_E_ARG, "%s: null argument or no plans", who);
    if (n_plans > kStaticMaxPlans) return fail(KVTC_E_UNSUPPORTED, "%s: %d plans, at most %d per call", who, n_plans, kStaticMaxPlans);
    if (n_jobs < 0) return fail(KVTC_E_ARG, "%s: n_jobs=%d", who, n_jobs);
    if (n_jobs > kMaxJobs) return fail(KVTC_E_UNSUPPORTED, "%s: %d jobs, at most %d per call", who, n_jobs, kMaxJobs);
    if (n_jobs == 0) return KVTC_OK;
    if (!jobs_dev || !x_base_dev || !out_base_dev || !status_dev) return fail(KVTC_E_ARG, "%s: null buffer", who);
    if (!dtype_ok(dtype)) return fail(KVTC_E_ARG, "%s: unknown dtype %d", who, (int)dtype);
    if ((reinterpret_cast<uintptr_t>(x_base_dev) & 15u) || ((size_t)ld_x * elem_size(dtype)) % 16 != 0 || ld_x <= 0)
        return fail(KVTC_E_ARG, "%s: feature array base and row pitch must be 16-byte aligned", who);
    if (ld_x > kMaxPitch) return fail(KVTC_E_ARG, "%s: ld_x=%lld above %d", who, (long long)ld_x, kMaxPitch);
    if (reinterpret_cast<uintptr_t>(out_base_dev) & 15u) return fail(KVTC_E_ARG, "%s: stream buffer must be 16-byte aligned", who);
    // the kernel variants among the plans and their LDS needs, on the stack
    EncodeLaunches l;
    l.n_bulk = 0;
    l.all_short = true;
    l.min_rec_dwords = 1 << 30;
    l.max_p = 0;
    l.lines = whole_lines(x_base_dev, dtype, XLayout{ld_x, 0, 0});
    l.shrt[1] = l.shrt[2] = {0, 0};
    PlanPtrs ptrs;
    for (int i = 0; i < n_plans; ++i) {
        if (!plans[i]) return fail(KVTC_E_ARG, "%s: plan %d is null", who, i);
        const PlanDev& ph = plans[i]->h;
        if (ld_x < ph.p) return fail(KVTC_E_ARG, "%s: ld_x=%lld < p=%d", who, (long long)ld_x, ph.p);
        ptrs.p[i] = plans[i]->desc_dev;
        const int key = ph.enc_nw * 10000 + ph.enc_wc * 100 + ph.enc_ntw;
        int k = 0;
        while (k < l.n_bulk && l.bulk[k].key != key) ++k;
        if (k == l.n_bulk) l.bulk[l.n_bulk++] = {key, ph.enc_wgs, 0};
        l.bulk[k].lds = std::max(l.bulk[k].lds, ph.enc_lds[dtype]);
        l.min_rec_dwords = std::min(l.min_rec_dwords, ph.rec_dwords);
        l.max_p = std::max(l.max_p, ph.p);
        l.all_short = l.all_short && ph.enc_short != 0;
        l.part.add(*plans[i], dtype);
        if (ph.enc_short != 0) {
            auto& v = l.shrt[ph.enc_short];
            v.waves = std::max(v.waves, plans[i]->enc_s_waves);
            v.lds = std::max(v.lds, plans[i]->enc_s_lds[dtype]);
        }
    }
    for (int i = n_plans; i < kStaticMaxPlans; ++i) ptrs.p[i] = nullptr;
    StaticScratch* sc = nullptr;
    hipError_t e = static_scratch(&sc);
    if (e != hipSuccess) return fail(KVTC_E_HIP, "%s: no address for the static work area: %s", who, hipGetErrorString(e));
    hipStream_t st = static_cast<hipStream_t>(stream);
    // every entry the kernels read is written here first, so nothing of an earlier call is seen
    hipLaunchKernelGGL(gather_plans_kernel, dim3(1), dim3(256), 0, st, ptrs, n_plans, sc);
    hipLaunchKernelGGL(offsets_kernel, dim3(1), dim3(256), 0, st, sc->rec_dwords, n_plans, jobs_dev, n_jobs, sc->offsets, offsets_out_dev);
    e = hipGetLastError();
    if (e != hipSuccess) return fail(KVTC_E_HIP, "%s: launch failed: %s", who, hipGetErrorString(e));
    KernelArgs a;
    memset(&a, 0, sizeof(a));
    a.plans = sc->plans;
    a.n_plans = n_plans;
    a.jobs = jobs_dev;
    a.n_jobs = n_jobs;
    a.offsets = sc->offsets;
    a.x = x_base_dev;
    a.ld_x = ld_x;
    a.stream_buf = out_base_dev;
    a.cap = out_cap;
    a.status = status_dev;
    return launch_encode_jobs(who, l, a, dtype, st);
}

kvtc_status kvtc_test_batch_passes(const kvtc_batch* batch, const kvtc_job* jobs_dev, int n_jobs, const uint64_t* offsets_dev, size_t stream_bytes,
                                   uint64_t elements, uint32_t* passes_dev, kvtc_stream stream) {
    if (!batch || !jobs_dev || !offsets_dev || !passes_dev || n_jobs < 1 || n_jobs > kMaxJobs) return fail(KVTC_E_ARG, "kvtc_test_batch_passes: bad argument");
    KernelArgs a;
    memset(&a, 0, sizeof(a));
    a.plans = batch->plans_dev;
    a.n_plans = batch->n_plans;
    a.jobs = jobs_dev;
    a.n_jobs = n_jobs;
    a.offsets = offsets_dev;
    a.cap = stream_bytes;
    a.x_pass_from = (float)elements;
    hipLaunchKernelGGL(batch_passes_kernel, dim3(1), dim3(kThreads), 0, static_cast<hipStream_t>(stream), a, batch->enc[0].key, passes_dev);
    const hipError_t e = hipGetLastError();
    return e == hipSuccess ? KVTC_OK : fail(KVTC_E_HIP, "kvtc_test_batch_passes: launch failed: %s", hipGetErrorString(e));
}

kvtc_status kvtc_decode_batch(const kvtc_batch* batch, const kvtc_job* jobs_dev, int n_jobs, const void* in_base_dev,
                              size_t in_bytes, const uint64_t* offsets_dev, void* x_out_base_dev, kvtc_dtype dtype,
                              int64_t ld_x, uint32_t* status_dev, kvtc_stream stream) {
    const kvtc_layout lay = {ld_x, 0, 0, 0};
    return kvtc_decode_batch_blocked(batch, jobs_dev, n_jobs, in_base_dev, in_bytes, offsets_dev, x_out_base_dev, dtype, &lay, status_dev, stream);
}

kvtc_status kvtc_decode_batch_blocked(const kvtc_batch* batch, const kvtc_job* jobs_dev, int n_jobs, const void* in_base_dev,
                                      size_t in_bytes, const uint64_t* offsets_dev, void* x_out_base_dev, kvtc_dtype dtype,
                                      const kvtc_layout* layout, uint32_t* status_dev, kvtc_stream stream) {
    bool nothing;
    XLayout xl = {0, 0, 0};
    kvtc_status st = batch_common("kvtc_decode_batch", batch, jobs_dev, n_jobs, x_out_base_dev, dtype, layout, offsets_dev,
                                  in_base_dev, status_dev, &nothing, &xl);
    if (st != KVTC_OK || nothing) return st;
    const int64_t ld_x = xl.ld;
    KernelArgs a;
    memset(&a, 0, sizeof(a));
    a.plans = batch->plans_dev;
    a.n_plans = batch->n_plans;
    a.jobs = jobs_dev;
    a.n_jobs = n_jobs;
    a.offsets = offsets_dev;
    a.x = x_out_base_dev;
    a.ld_x = ld_x;
    a.x_blk_log2 = xl.blk_log2;
    a.x_blk_jump = xl.blk_jump;
    a.stream_buf = const_cast<void*>(in_base_dev);
    a.cap = in_bytes;
    a.status = status_dev;
    for (const auto& v : batch->dec) {
        a.x_pass_from = pass_from(whole_lines(x_out_base_dev, dtype, xl), decode_pass_bytes(v.key % 100, v.least_tiles, dtype, v.bases, false), dtype,
                                  most_elements(in_bytes, batch->min_rec_dwords, batch->max_p), true);
        // Jobs whose 128-token tiles can be shown to run all at once (the stream buffer's size bounds their tokens, and each may end in a
        // part of a tile) take the variant with one token tile per wave, as a single tensor does, where the mean job is no more than one such tile
        // or the tiles, twice as many with twice the basis traffic, are few: one per compute unit; of more plans than there are XCDs fewer, and
        // most of each job's second tile used; all of the narrow class, but for jobs of two tiles.
        // Both sides, us, 256-token tiles and 128-token tiles: a head of 4096 tokens in fp32 11.6 and 8.6; one tensor of 32768 tokens at 16x 28.5 and 27.2, of 34000
        // 31.6 and 36.0, of 40000 at 40x 25.6 and 22.9; 200 of 130 tokens at 40x 26.1 and 27.9; 64 with a plan each, 16x, of 300 tokens 33.1
        // and 29.8, of 500 34.3 and 38.7, 20x in fp32 of 130 tokens 21.0 and 24.3, of 200 23.1 and 24.7.
        const int cus = compute_units(), slots = cus * v.wgs;
        const bool wide = v.key % 100 > 10, many = batch->n_plans > 8;
        const size_t tokens = in_bytes / ((size_t)batch->min_rec_dwords * 4), jobs = (size_t)n_jobs, mean = (tokens + jobs - 1) / jobs;
        const size_t few = v.wgs == 3 && mean > 2 * kDecShortTile ? slots : !many ? cus : mean > 7 * kDecShortTile / 4 ? cus * 3 / 4 : 0;
        a.dec_short = !wide && tokens / kDecShortTile + jobs <= (size_t)slots &&
                      (mean <= kDecShortTile || (mean + kDecShortTile - 1) / kDecShortTile * jobs <= few);
        const DecLayout lay = decode_layout(a.dec_short ? decode_rec_bytes(1, v.rec_dwords) : v.rec, v.ring, v.wgs);
        a.dec_ring_off = lay.ring_off;
        // Where there may be few shares of tiles, 64 features each, no more workgroups than that: every one reads the job table before it knows that it has none.  Two to a
        // tile at least, or the kernel's form for few tiles is not taken.  Of a few more than the compute units some would be two to one and others idle.  (us, all
        // and so: a head of 4096 tokens in fp32, 66 for 768, 7.5 -> 6.7, four tensors of 16 tokens at 16x 8.5 -> 7.4, 90 heads of 64, 270, 8.3 -> 7.0, of 256 features 64 of 33,
        // 320, 8.1 -> 7.8; not so: 128 heads of 64, 384, 6.9 7.1, 16 tensors of 16 at 40x, 288, 6.3 6.7, at 16x in fp32 8.8 10.1; one of 64 features, one workgroup, 5.0 5.4.)
        const size_t shares = (tokens / kDecShortTile + jobs) * (size_t)std::max(batch->max_p / 64, 2), grid = shares <= (size_t)(batch->max_p <= 256 ? cus * 5 / 4 : cus) ? shares : slots;
        hipError_t e = launch_decode(a, dtype, a.dec_short ? 100 + v.key % 100 : v.key, (int)std::min<size_t>(slots, grid), lay.lds_bytes, static_cast<hipStream_t>(stream));
        if (e != hipSuccess) return fail(KVTC_E_HIP, "kvtc_decode_batch: launch failed: %s", hipGetErrorString(e));
    }
    return KVTC_OK;
}

}  // extern "C"

// ---- sectioned plans: more kept coordinates than one record holds ---------------------------------
struct kvtc_wide {
    int p, r;
    std::vector<kvtc_plan*> sections;
    size_t record_bytes;            // over all sections
};

namespace {

constexpr int kSectionCoords = 1024, kSectionGroups = 64;

}  // namespace

extern "C" {

kvtc_status kvtc_wide_create(kvtc_wide** out, int p, int r, const float* mu_host, const uint16_t* v_kept_host, int n_groups,
                             const kvtc_group* groups_host, kvtc_stream stream) {
    if (out) *out = nullptr;
    if (!out || !mu_host || !v_kept_host || !groups_host) return fail(KVTC_E_ARG, "kvtc_wide_create: null argument");
    if (p <= 0 || p % 64 != 0) return fail(KVTC_E_ARG, "kvtc_wide_create: p=%d must be a positive multiple of 64", p);
    if (n_groups < 1 || r < 16) return fail(KVTC_E_ARG, "kvtc_wide_create: r=%d, n_groups=%d", r, n_groups);
    long sum = 0;
    for (int g = 0; g < n_groups; ++g) {
        if (groups_host[g].n < 1 || groups_host[g].n > kSectionCoords)
            return fail(KVTC_E_ARG, "kvtc_wide_create: group %d has %d coordinates (1..%d allowed)", g, (int)groups_host[g].n, kSectionCoords);
        sum += groups_host[g].n;
    }
    if (sum != r) return fail(KVTC_E_ARG, "kvtc_wide_create: group sizes sum to %ld, r=%d", sum, r);
    kvtc_wide* w = new (std::nothrow) kvtc_wide;
    if (!w) return fail(KVTC_E_NOMEM, "kvtc_wide_create: host allocation failed");
    w->p = p;
    w->r = r;
    w->record_bytes = 0;
    // consecutive groups -> sections, greedily: a section takes groups while it stays within 1024 coordinates and 64 groups
    int g0 = 0, j0 = 0;
    while (g0 < n_groups) {
        int g1 = g0, n = 0;
        while (g1 < n_groups && g1 - g0 < kSectionGroups && n + groups_host[g1].n <= kSectionCoords) n += groups_host[g1++].n;
        kvtc_plan* sec = nullptr;
        kvtc_status st = plan_create_impl(&sec, p, n, mu_host, v_kept_host + j0, (size_t)r, g1 - g0, groups_host + g0,
                                          /*dec_zero_mu=*/g0 != 0, stream);
        if (st == KVTC_OK) {
            try { w->sections.push_back(sec); } catch (const std::bad_alloc&) { kvtc_plan_destroy(sec); st = fail(KVTC_E_NOMEM, "kvtc_wide_create: host allocation failed"); }
        }
        if (st != KVTC_OK) {
            kvtc_wide_destroy(w);
            return st;
        }
        w->record_bytes += sec->record_bytes;
        g0 = g1;
        j0 += n;
    }
    *out = w;
    return KVTC_OK;
}

void kvtc_wide_destroy(kvtc_wide* w) {
    if (!w) return;
    for (kvtc_plan* s : w->sections) kvtc_plan_destroy(s);
    delete w;
}

int kvtc_wide_sections(const kvtc_wide* w) { return w ? (int)w->sections.size() : 0; }

size_t kvtc_wide_section_record_bytes(const kvtc_wide* w, int section) {
    return (w && section >= 0 && section < (int)w->sections.size()) ? w->sections[section]->record_bytes : 0;
}

size_t kvtc_wide_record_bytes(const kvtc_wide* w) { return w ? w->record_bytes : 0; }

size_t kvtc_wide_encoded_bytes(const kvtc_wide* w, int64_t n_tokens) {
    if (!w || n_tokens <= 0) return 0;
    size_t pos = 0;
    for (const kvtc_plan* s : w->sections) pos = align_up(pos, 16) + s->record_bytes * (size_t)n_tokens;
    return pos;
}

kvtc_status kvtc_wide_encode(const kvtc_wide* w, const void* x_dev, kvtc_dtype dtype, int64_t n_tokens, const kvtc_layout* layout,
                             void* out_dev, size_t out_cap, kvtc_stream stream) {
    if (!w) return fail(KVTC_E_ARG, "kvtc_wide_encode: null plan");
    if (n_tokens < 0 || n_tokens > 0x7fffffffLL) return fail(KVTC_E_ARG, "kvtc_wide_encode: n_tokens=%lld", (long long)n_tokens);
    if (n_tokens == 0) return KVTC_OK;
    if (!out_dev) return fail(KVTC_E_ARG, "kvtc_wide_encode: null buffer");
    if (out_cap < kvtc_wide_encoded_bytes(w, n_tokens))
        return fail(KVTC_E_SMALL, "kvtc_wide_encode: out_cap=%zu < %zu", out_cap, kvtc_wide_encoded_bytes(w, n_tokens));
    size_t pos = 0;
    for (const kvtc_plan* s : w->sections) {          // a launch per section, each over all tokens
        pos = align_up(pos, 16);
        const size_t bytes = s->record_bytes * (size_t)n_tokens;
        kvtc_status st = encode_single("kvtc_wide_encode", s, x_dev, dtype, n_tokens, layout, static_cast<char*>(out_dev) + pos, bytes, stream);
        if (st != KVTC_OK) return st;
        pos += bytes;
    }
    return KVTC_OK;
}

kvtc_status kvtc_wide_decode(const kvtc_wide* w, const void* in_dev, size_t in_bytes, int64_t n_tokens, void* x_out_dev, kvtc_dtype dtype,
                             const kvtc_layout* layout, float* sum_dev, kvtc_stream stream) {
    if (!w) return fail(KVTC_E_ARG, "kvtc_wide_decode: null plan");
    if (n_tokens < 0 || n_tokens > 0x7fffffffLL) return fail(KVTC_E_ARG, "kvtc_wide_decode: n_tokens=%lld", (long long)n_tokens);
    if (n_tokens == 0) return KVTC_OK;
    if (!in_dev || !x_out_dev) return fail(KVTC_E_ARG, "kvtc_wide_decode: null buffer");
    if (!dtype_ok(dtype)) return fail(KVTC_E_ARG, "kvtc_wide_decode: unknown dtype %d", (int)dtype);
    if (in_bytes < kvtc_wide_encoded_bytes(w, n_tokens))
        return fail(KVTC_E_SMALL, "kvtc_wide_decode: in_bytes=%zu < %zu", in_bytes, kvtc_wide_encoded_bytes(w, n_tokens));
    // the sections' products are summed in fp32: straight in the output when that is fp32; else in the caller's workspace,
    // from which the last section's launch reads the sum of the others, adds its own part and rounds to bf16 once
    XLayout xl;
    kvtc_status st = check_layout("kvtc_wide_decode", x_out_dev, dtype, layout, w->p, n_tokens, &xl);
    if (st != KVTC_OK) return st;
    const kvtc_layout flat = {w->p, 0, 0, 0};
    const size_t n_sec = w->sections.size();
    if (dtype == KVTC_BF16 && n_sec > 1) {
        if (!sum_dev) return fail(KVTC_E_ARG, "kvtc_wide_decode: bf16 output needs the fp32 workspace sum_dev [n_tokens][p]");
        if (reinterpret_cast<uintptr_t>(sum_dev) & 15u) return fail(KVTC_E_ARG, "kvtc_wide_decode: sum_dev must be 16-byte aligned");
    }
    size_t pos = 0;
    for (size_t c = 0; c < n_sec; ++c) {
        const kvtc_plan* s = w->sections[c];
        pos = align_up(pos, 16);
        const size_t bytes = s->record_bytes * (size_t)n_tokens;
        const char* in = static_cast<const char*>(in_dev) + pos;
        if (dtype == KVTC_F32)
            st = decode_single("kvtc_wide_decode", s, in, bytes, n_tokens, x_out_dev, KVTC_F32, layout, stream, c == 0 ? 0 : 1);
        else if (c + 1 == n_sec)
            st = n_sec == 1 ? decode_single("kvtc_wide_decode", s, in, bytes, n_tokens, x_out_dev, KVTC_BF16, layout, stream)
                            : decode_single("kvtc_wide_decode", s, in, bytes, n_tokens, x_out_dev, KVTC_BF16, layout, stream, 2, sum_dev, w->p);
        else
            st = decode_single("kvtc_wide_decode", s, in, bytes, n_tokens, sum_dev, KVTC_F32, &flat, stream, c == 0 ? 0 : 1);
        if (st != KVTC_OK) return st;
        pos += bytes;
    }
    return KVTC_OK;
}

kvtc_status kvtc_calib_moments(const void* x_dev, kvtc_dtype dtype, int64_t n_tokens, int p, const kvtc_layout* layout, double* sum_dev,
                               double* gram_dev, kvtc_stream stream) {
    if (n_tokens < 0 || n_tokens > 0x7fffffffLL) return fail(KVTC_E_ARG, "kvtc_calib_moments: n_tokens=%lld", (long long)n_tokens);
    if (p <= 0 || p % 64 != 0) return fail(KVTC_E_ARG, "kvtc_calib_moments: p=%d must be a positive multiple of 64", p);
    if (!x_dev || !sum_dev || !gram_dev) return fail(KVTC_E_ARG, "kvtc_calib_moments: null buffer");
    if ((reinterpret_cast<uintptr_t>(sum_dev) & 7u) || (reinterpret_cast<uintptr_t>(gram_dev) & 7u))
        return fail(KVTC_E_ARG, "kvtc_calib_moments: outputs must be 8-byte aligned");
    XLayout xl;
    kvtc_status st = check_layout("kvtc_calib_moments", x_dev, dtype, layout, p, n_tokens, &xl);
    if (st != KVTC_OK) return st;
    const hipError_t e = launch_calib_moments(x_dev, dtype, n_tokens, p, xl.ld, xl.blk_log2, xl.blk_jump, sum_dev, gram_dev,
                                              static_cast<hipStream_t>(stream));
    if (e != hipSuccess) return fail(KVTC_E_HIP, "kvtc_calib_moments: launch failed: %s", hipGetErrorString(e));
    return KVTC_OK;
}

}  // extern "C"
