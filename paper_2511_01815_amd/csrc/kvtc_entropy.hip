// Lossless stage over the packed records for gfx950 (declared in include/kvtc.h, "Lossless stage"):
// a static prefix code per byte position of the record.  (Paper, Section "Entropy coding": the
// quantiser's byte array goes through a lossless coder on the GPU; the paper uses a general-purpose
// DEFLATE, this library a byte-wise entropy coder matched to the records' fixed layout.)
//
// Work decomposition: a wavefront owns chunks of 64 tokens; blockIdx.y is the job (tensor) of a batched call, so a
// workgroup's chunks share one table set, which it keeps in LDS.  The code tables are data (256 code lengths per byte
// position and table set, from calibration); canonical codes and the decoding tables are derived from them on the host at
// creation.
//   encode = three launches: (1) code lengths -> len_bits[] and the chunk sizes, written into the container's own
//   directory; (2) a workgroup per job turns the sizes into offsets; (3) the code strings.  In (1) and (3) a chunk is the
//   flat run of its records' bytes, dealt to the lanes in 16-byte pieces (coalesced loads, no staging, no idle lanes
//   whatever the record size): a chunk's bit string is the concatenation of its bytes' codes in that very order, so one
//   prefix sum over the wave places every lane's string.
//   decode = one launch: a lane walks the string of one token, all lanes at the same byte position.  With canonical
//   codes the next 12 bits, read as a number with the first bit on top, are below limit[L] exactly when the code has at most
//   L bits.  Records of up to 128 bytes under complete codes find the length by one lookup, in a table indexed by the complement of
//   those bits as a float, and their strings come through LDS (entropy_decode_staged_kernel).  In the general form a code's length is
//   what a 256-entry table says for the next 8 bits (9 for every longer code) plus a count of comparisons.  Length and bits give the
//   symbol's rank, the rank the symbol; the walk waits for neither.
// Nothing is allocated: the directory lives in the output buffer.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <atomic>
#include <cstring>
#include <memory>
#include <new>
#include <type_traits>
#include <vector>

#include "kvtc_dev.h"

namespace kvtc {
kvtc_status set_error(kvtc_status st, const char* fmt, ...);
}
using namespace kvtc;

struct kvtc_entropy {
    int record_bytes, n_tables;
    void* blob;                 // device: the tables below
    const uint16_t* enc_dev;    // [n_tables][R][256] reversed code | length << 12
    const uint8_t* len_dev;     // [n_tables][R][256] length
    const uint8_t* dec_dev;     // the decoder's tables, one behind the other, each [n_tables][R]: lengths, symbols, offsets
    const uint32_t* lim_dev;    // [n_tables][R][4]
    const uint8_t* log_dev;     // the staged decoder's tables, or nullptr: [n_tables] of kLogRow * R bytes
};

namespace {

constexpr int kMaxLen = 12;
constexpr int kChunk = 64;
constexpr int kMaxRecord = 576;       // bytes
constexpr int kMaxEntropyJobs = 65535;

__host__ __device__ inline uint32_t chunk_image_dwords(int R) { return (uint32_t)(kChunk * R * kMaxLen + 31) / 32u; }   // worst case
__host__ __device__ inline uint64_t header_bytes(int64_t n_chunks) { return 4ull * (uint64_t)(n_chunks + 1) + 2ull * kChunk * (uint64_t)n_chunks; }

// Tables in LDS: the rows of successive byte positions are a dword apart from a multiple of the banks, so that lanes that
// look up like bytes of different positions do not all meet on one bank.
constexpr int kLenRow = 256 + 4, kEncRow = 512 + 4;                          // bytes per byte position
constexpr int kImageDw = 392;         // a wave's part of the bit string: 64 pieces of 16 codes of at most 12 bits, 16 carried bytes, and 16 for zeros beyond them
constexpr int kLdsMost = kLdsBudget - 1024;
constexpr int kMaxLdsRecord = 264;    // bytes: the largest whose code table fits beside 16 waves' images
static_assert(kMaxLdsRecord * kEncRow + 16 * kImageDw * 4 <= kLdsMost && (kMaxLdsRecord + 4) * kEncRow + 16 * kImageDw * 4 > kLdsMost, "the edge");
static_assert(kMaxRecord * kLenRow + 16 * kChunk * 4 <= kLdsMost, "the length table of every record size fits");

// Decoding data of one byte position.  Codes are canonical: those of L bits are first[L] .. first[L] + count[L] - 1.
// Three tables, kDecRow bytes in all, in LDS behind the waves' rows (each from a multiple of 256 bytes on, so that an index is OR-ed in):
// [256] by the next 8 bits of the string, the code's length, 9 for every code of 9 bits or more (10 .. 12 if none is shorter);
// [256] symbols by rank, i.e. ordered by (length, value); [16] at L: first[L] - (number of symbols with shorter codes), modulo
// 256, so that the rank of a code of L bits is its value minus this.  (All lanes look up the same position at a time: rows
// need no padding.)  Records too long for one table in LDS are decoded in segments of kDecSegment bytes.
// In scalar registers, four dwords: ((first[L] + count[L]) << (32 - L)) - 1 for L = 9, 10, 11: a string whose next 32 bits, first
// bit on top, exceed it begins with a code of more than L bits.
// A wave collects kDecBatch dwords of its 64 rows in front of the tables, at a pitch of whole 16-byte pieces.
constexpr int kDecOff = 16, kDecRow = 256 + 256 + kDecOff;
constexpr int kDecSegment = 144, kDecBatch = 16, kDecPitch = 20;
static_assert(kChunk * kDecPitch * 4 % 256 == 0, "tables from a multiple of 256 bytes on");
static_assert(kDecSegment % 16 == 0 && kDecBatch % 2 == 0 && kDecSegment * kDecRow + 16 * kChunk * kDecPitch * 4 <= kLdsMost, "a segment's table and 16 waves' rows fit");

// The staged decoder (entropy_decode_staged_kernel) finds a code's length with one lookup and no comparison.  u, the complement of the string's
// next 12 bits read as a number with the first bit on top, is small where codes are long.  Codes longer than L bits, at most 256 of at most 2^(11 - L)
// such numbers each, take those below a multiple of 2^(12 - L) that is at most 64 * 2^(13 - L), so it is enough to know u to one part in 64: the
// bits of a float, exponent and six of mantissa, where u = 64 is the smallest normal number and everything below lies in the denormals' even steps.
// 448 entries to a position, 32 - length each.  (A code with strings that begin no code has its bounds elsewhere: such tables are not built, and
// the other decoder serves them.)  Behind the length all is as above, with the offsets by 32 - length, 16 + 4 .. 16 + 15.
// LDS: kLogMost rows each of symbols, offsets and lengths, those of the last R rows only, so that a row is a constant of an instruction; then the waves' strings,
// kLogString dwords of every lane's, dword-major: free of conflicts whatever the lanes read.
constexpr int kLogMost = 128, kLogEntries = 448, kLogRow = 256 + kDecOff + kLogEntries;
constexpr int kLogSym = 0, kLogOff = kLogMost * 256, kLogLen = kLogOff + kLogMost * kDecOff;
constexpr int kLogUnit = 32, kLogAhead = 8, kLogString = 17;           // positions decoded from a slot; of those, still to come when the next is requested; its dwords
constexpr int kLogSlot = kLogString * 256;
static_assert((31 + (kLogAhead + kLogUnit - 4) * kMaxLen) / 32 + 2 < kLogString, "the window of a unit's last four codes lies in its slot");
static_assert(kLogSlot >= kChunk * 64 && kLogLen % 256 == 0 && kLogMost * kLogEntries % 256 == 0, "64 bytes of every row fit a slot; slots on multiples of 256");
static_assert(kLogLen >= 32768 && kLogLen - 32768 + kLogMost * kLogEntries <= 65536, "the lengths lie within an instruction's offset of 32768");
__host__ __device__ constexpr size_t log_bytes(int R) { return (size_t)(kLogLen + R * kLogEntries + 255) / 256 * 256; }        // the tables in LDS
static_assert(log_bytes(kLogMost) + 16 * kLogSlot <= kLdsMost, "all of it fits");

struct EntropyArgs {
    const kvtc_entropy_job* jobs;     // device, or nullptr -> `single`
    int32_t n_jobs;
    kvtc_entropy_job single;
    const uint8_t* records;           // encode: input, decode: output
    uint64_t records_cap;
    uint8_t* coded;                   // encode: output, decode: input
    uint64_t coded_total;
    uint64_t* coded_bytes;            // encode: [n_jobs] container lengths
    const uint16_t* enc;
    const uint8_t* len;
    const uint8_t* dec;
    const uint32_t* lim;
    const uint8_t* log;
    int32_t R, n_tables;
    int32_t waves;                    // of a workgroup that take chunks; any others only help to copy its tables
    int32_t chunks_per_wave;          // chunks a wave takes one after the other, so that a workgroup's tables serve several
    int64_t max_tokens;               // the launch covers this many tokens per job; a longer job is left alone
};

// A job as the kernels see it, or ok = false when anything about it is out of range (then the job is left alone).
struct JobView {
    bool ok;
    int64_t T, n_chunks;
    uint32_t* rec;             // the job's records
    uint32_t* chunk_off;       // the container's directory ...
    uint16_t* len_bits;
    uint8_t* payload;          // ... and payload
    uint64_t payload_cap;
    size_t table;              // first byte position of the job's table set
};
__device__ __forceinline__ JobView job_view(const EntropyArgs& a, int j) {
    const kvtc_entropy_job jb = a.jobs ? a.jobs[j] : a.single;
    JobView v;
    v.T = jb.n_tokens;
    v.n_chunks = ((int64_t)jb.n_tokens + kChunk - 1) / kChunk;
    const uint64_t hdr = header_bytes(v.n_chunks);
    const uint64_t rec_bytes = (uint64_t)(jb.n_tokens > 0 ? jb.n_tokens : 0) * (uint64_t)a.R;
    v.ok = jb.table >= 0 && jb.table < a.n_tables && jb.n_tokens >= 0 && (int64_t)jb.n_tokens <= a.max_tokens && (jb.records_off & 3ull) == 0 && (jb.coded_off & 3ull) == 0 &&
           jb.records_off <= a.records_cap && rec_bytes <= a.records_cap - jb.records_off &&
           jb.coded_off <= a.coded_total && jb.coded_cap <= a.coded_total - jb.coded_off && hdr <= jb.coded_cap;
    if (!v.ok) return v;
    v.rec = reinterpret_cast<uint32_t*>(const_cast<uint8_t*>(a.records) + jb.records_off);
    v.chunk_off = reinterpret_cast<uint32_t*>(a.coded + jb.coded_off);
    v.len_bits = reinterpret_cast<uint16_t*>(v.chunk_off + v.n_chunks + 1);
    v.payload = a.coded + jb.coded_off + hdr;
    v.payload_cap = jb.coded_cap - hdr;
    v.table = (size_t)jb.table * a.R;
    return v;
}

// LDS written by some lanes of a wave and read by others of the same wave
__device__ __forceinline__ void wave_fence() {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

struct __attribute__((packed, aligned(4))) Dwords4 { uint32_t w[4]; };      // 16 bytes on any dword boundary
struct __attribute__((packed, aligned(4))) Dwords2 { uint32_t w[2]; };

// A wave's walk over a chunk's bytes: in every step the wave takes 64 pieces of four dwords, a lane one piece.
struct PieceWalk {
    uint32_t dw, n_dw;          // the piece's first dword in the chunk; dwords of the chunk
    uint32_t at;                // that dword's place in its record
    uint32_t per_row, step;     // dwords per record; 256 modulo that
    __device__ __forceinline__ PieceWalk(int64_t T, int64_t chunk, int R) {
        const int64_t left = T - chunk * kChunk;
        per_row = (uint32_t)R / 4u;
        n_dw = (uint32_t)(left < kChunk ? left : kChunk) * per_row;
        dw = (threadIdx.x & 63u) * 4u;
        at = dw % per_row;
        step = 256u % per_row;
    }
    __device__ __forceinline__ void load(const uint32_t* src, uint32_t (&w)[4]) const {
        if (dw + 4u <= n_dw) {
            const Dwords4 v = *reinterpret_cast<const Dwords4*>(src + dw);
#pragma unroll
            for (int j = 0; j < 4; ++j) w[j] = v.w[j];
        } else {
#pragma unroll
            for (int j = 0; j < 4; ++j) w[j] = dw + j < n_dw ? src[dw + j] : 0u;
        }
    }
    __device__ __forceinline__ void next() {
        dw += 256u;
        at += step;
        if (at >= per_row) at -= per_row;
    }
};

// the workgroup's tables, global -> LDS, in 16-byte pieces: rows of 2^log2_row dwords, a dword of padding behind each.  (Dword by dword
// the copy was a quarter of a small call: one 64-token tensor of 128-byte records, encode 28 us, now 20, decode 26, now 19.)
__device__ __forceinline__ void stage_table(const uint32_t* src, int rows, int log2_row, uint32_t* dst) {
    const int n = (rows << log2_row) >> 2;
    const uint4* from = reinterpret_cast<const uint4*>(src);
#pragma unroll 4
    for (int i = threadIdx.x; i < n; i += blockDim.x) {
        const uint4 v = from[i];
        uint32_t* to = dst + 4 * i + (4 * i >> log2_row);
        to[0] = v.x;
        to[1] = v.y;
        to[2] = v.z;
        to[3] = v.w;
    }
}

// (1) bits of every token's code string -> len_bits[]; bytes of every chunk's bit string -> chunk_off[chunk] (sizes for now).
// Bound by the table lookups: one LDS gather per byte (looked up in global memory, with a lane per token and the rows staged
// in LDS, the same 256 MiB took 237 us; now 75).  A token's length is the difference of the running bit count at its last
// dword and at the token's before it.
// LONG: records of whole 16 bytes have pieces within a record: one end at most, and rows at distances that stand in the instructions.  Bound by vector instructions and the
// LDS alike: 256 MiB 75 us, 80 where each dword of a piece was looked at for a record's end; of 64 tensors of 30000 tokens of 32 bytes, encode 53.3 -> 50.6.
template <bool LONG>
__global__ void __launch_bounds__(1024, 2) entropy_size_kernel(const EntropyArgs a) {
    extern __shared__ uint32_t lds[];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), n_waves = a.waves;
    const int R = a.R;
    const JobView v = job_view(a, blockIdx.y);
    const int64_t first = (int64_t)blockIdx.x * n_waves * a.chunks_per_wave;
    if (!v.ok || first >= v.n_chunks) return;
    uint32_t* ends = lds + wave * kChunk;                            // running bit count at the end of every token
    uint32_t* tab32 = lds + n_waves * kChunk;
    stage_table(reinterpret_cast<const uint32_t*>(a.len + v.table * 256), R, 6, tab32);
    const uint8_t* tab = reinterpret_cast<const uint8_t*>(tab32);
    __syncthreads();
    if (wave >= n_waves) return;
    for (int c = 0; c < a.chunks_per_wave; ++c) {
        const int64_t chunk = first + (int64_t)c * n_waves + wave;
        if (chunk >= v.n_chunks) break;
        PieceWalk pw(v.T, chunk, R);
        const uint32_t* src = v.rec + chunk * kChunk * pw.per_row;
        uint32_t token = pw.dw / pw.per_row;
        const uint32_t token_step = 256u / pw.per_row;
        const uint32_t rows_end = pw.per_row * (4u * kLenRow);
        const bool within = LONG && pw.per_row % 4u == 0u;           // every piece within a record
        uint32_t run = 0;                                            // bits of the pieces before this step
        uint32_t w[4];
        pw.load(src, w);
        for (uint32_t d0 = 0; d0 < pw.n_dw; d0 += 256u) {
            const PieceWalk cur = pw;
            const uint32_t tok0 = token;
            uint32_t s[4], row = __umul24(cur.at, 4u * kLenRow), tok = tok0, last = 0u, end_tok[4];
            auto dword_bits = [&](int j, int rows) {                 // an entry's address: the row's, and the byte, by one dot product
                auto entry = [&](int b) {
                    return LONG ? (uint32_t)tab[__builtin_amdgcn_udot4(w[j], 1u << (8 * b), row, false) + (4 * rows + b) * kLenRow]
                                : (uint32_t)(tab + row)[((w[j] >> (8 * b)) & 0xffu) + (4 * rows + b) * kLenRow];
                };
                return entry(0) + entry(1) + entry(2) + entry(3);
            };
            if (within) {
#pragma unroll
                for (int j = 0; j < 4; ++j) last += dword_bits(j, j);
                last = cur.dw < cur.n_dw ? last : 0u;
                asm volatile("; rows of one record");                // (keeps the two forms' reads from being made one, behind registers of addresses)
            } else {
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const uint32_t bits = dword_bits(j, 0);
                    s[j] = cur.dw + j < cur.n_dw ? bits : 0u;
                    row += 4u * kLenRow;
                    end_tok[j] = row == rows_end && cur.dw + j < cur.n_dw ? tok : ~0u;
                    if (row == rows_end) { row = 0u; ++tok; }
                    last += s[j];
                }
            }
            token += token_step + (pw.at + pw.step >= pw.per_row ? 1u : 0u);
            pw.next();
            if (d0 + 256u < pw.n_dw) pw.load(src, w);                // the next step's bytes travel under this step's sums
            const uint32_t incl = wave_inclusive_scan(last);
            if (within) {
                if (cur.at + 4u == pw.per_row && cur.dw < cur.n_dw) ends[tok0] = run + incl;
            } else {
                uint32_t upto = run + incl - last;
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    upto += s[j];
                    if (end_tok[j] != ~0u) ends[end_tok[j]] = upto;
                }
            }
            run += (uint32_t)__builtin_amdgcn_readlane((int)incl, 63);
        }
        wave_fence();
        const int64_t t = chunk * kChunk + lane;
        // the directory has 64 entries per chunk: zero beyond the last token
        v.len_bits[t] = t < v.T ? (uint16_t)(ends[lane] - (lane > 0 ? ends[lane - 1] : 0u)) : (uint16_t)0;
        if (lane == 0) v.chunk_off[chunk] = (run + 31u) / 32u * 4u;
        wave_fence();
    }
}

// (2) sizes -> offsets, in place, one workgroup per job; the container's length -> coded_bytes[job] (all ones for a job
// that was left alone)
__global__ void __launch_bounds__(1024) entropy_scan_kernel(const EntropyArgs a) {
    __shared__ uint32_t sums[2][16];                                 // of the waves' 64 chunks each, in turn
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, n_waves = blockDim.x >> 6;
    const JobView v = job_view(a, blockIdx.x);
    if (!v.ok) {
        if (tid == 0 && a.coded_bytes) a.coded_bytes[blockIdx.x] = ~0ull;
        return;
    }
    uint32_t carry = 0;
    int turn = 0;
    for (int64_t base = 0; base < v.n_chunks; base += blockDim.x, turn ^= 1) {
        const int64_t j = base + tid;
        const uint32_t x = j < v.n_chunks ? v.chunk_off[j] : 0u, incl = wave_inclusive_scan(x);
        if (lane == 63) sums[turn][wave] = incl;
        __syncthreads();
        uint32_t before = carry;
        for (int w = 0; w < n_waves; ++w) {
            const uint32_t s = sums[turn][w];
            before += w < wave ? s : 0u;
            carry += s;
        }
        if (j < v.n_chunks) v.chunk_off[j] = before + incl - x;
    }
    if (tid == 0) {
        v.chunk_off[v.n_chunks] = carry;
        if (a.coded_bytes) a.coded_bytes[blockIdx.x] = header_bytes(v.n_chunks) + carry;
    }
}

// (3) the code strings.  A chunk whose string would end beyond the job's room is left unwritten (the caller sees the
// needed size in coded_bytes).  Per step a wave builds the string of its 64 pieces (1 KiB of records) in LDS, starting at the
// bits the step before left over, and stores the whole 16-byte pieces coalesced: 1.5 KiB of LDS per wave, where the image of a whole
// chunk and its rows took 20 and left a compute unit seven waves.  LDS_TAB: the codes come from the workgroup's copy of the
// table (records of up to kMaxLdsRecord bytes), else from global memory.  Four bytes' codes are
// put together and OR-ed in at once, where a 64-bit buffer emptied behind every second byte made it 16 instructions a byte with nine branches for each lane's 16
// bytes, and everything that is one for the wave stays in scalar registers; a step's 16 lookups are on their way together, and it waits for no store.
// Bound by the LDS (lookups of random bytes meet on banks) and, at 256 MiB in and 226 out, not far from what a copy of as much takes, 100 us.
// 256 MiB of records: 634 us in a chunk image, 163 with the buffer, 136 with dwords stored by and by, the last one or more of a step each by a branch, and
// lookups in three turns, 127 so (nine vector instructions to a byte for eleven).
template <bool LDS_TAB>
__global__ void __launch_bounds__(1024) entropy_write_kernel(const EntropyArgs a) {
    extern __shared__ uint32_t lds[];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), n_waves = a.waves;
    const int R = a.R;
    const JobView v = job_view(a, blockIdx.y);
    const int64_t first = (int64_t)blockIdx.x * n_waves * a.chunks_per_wave;
    if (!v.ok || first >= v.n_chunks) return;
    uint32_t* img = lds + wave * kImageDw;
    constexpr uint32_t kRowB = LDS_TAB ? kEncRow : 512;              // bytes from one byte position's entries to the next's
    const char* tab = reinterpret_cast<const char*>(a.enc + v.table * 256);
    if constexpr (LDS_TAB) {
        uint32_t* tab32 = lds + n_waves * kImageDw;
        stage_table(reinterpret_cast<const uint32_t*>(tab), R, 7, tab32);
        tab = reinterpret_cast<const char*>(tab32);
    }
    if (wave < n_waves)
        for (int i = lane; i < kImageDw; i += 64) img[i] = 0u;
    __syncthreads();
    if (wave >= n_waves) return;
    for (int c = 0; c < a.chunks_per_wave; ++c) {
        const int64_t chunk = first + (int64_t)c * n_waves + wave;
        if (chunk >= v.n_chunks) break;
        const uint32_t begin = __builtin_amdgcn_readfirstlane(v.chunk_off[chunk]), end = __builtin_amdgcn_readfirstlane(v.chunk_off[chunk + 1]);
        if (end < begin || (uint64_t)end > v.payload_cap) continue;
        const uint32_t n_out = (end - begin) / 4u;
        uint32_t* out = reinterpret_cast<uint32_t*>(v.payload + begin);
        PieceWalk pw(v.T, chunk, R);
        const uint32_t* src = v.rec + chunk * kChunk * pw.per_row;
        const uint32_t rows_end = pw.per_row * (4u * kRowB);
        uint32_t carry = 0, written = 0;                             // bits in img[0 .. 3] left by the step before; dwords stored
        uint32_t w[4], ahead[4] = {0u, 0u, 0u, 0u};
        pw.load(src, w);
#pragma unroll
        for (int j = 0; j < 4; ++j) asm volatile("" : "+v"(w[j]));   // (here, so that no step begins by waiting)
        for (uint32_t d0 = 0; d0 < pw.n_dw; d0 += 256u) {
            // all 16 lookups on their way at once.  An entry's address is one dot product: the row's, and twice the byte.
            uint32_t row = __umul24(pw.at, 4u * kRowB), ent[4][4];   // row: of the dword's first byte
            auto lookups = [&](auto wrap_tag) {
#pragma unroll
                for (int j = 0; j < 4; ++j) {
#pragma unroll
                    for (int b = 0; b < 4; ++b)
                        ent[j][b] = *reinterpret_cast<const uint16_t*>(tab + __builtin_amdgcn_udot4(w[j], 2u << (8 * b), row, false) +
                                                                       (decltype(wrap_tag)::value ? b : 4 * j + b) * kRowB);
                    if (decltype(wrap_tag)::value) {
                        row += 4u * kRowB;
                        if (row == rows_end) row = 0u;
                    }
                }
            };
            if (pw.per_row % 4u == 0u) {                             // (a piece is within its record: its rows' distances are in the instructions)
                lookups(std::false_type());
                asm volatile("; rows of one record");                // (keeps the two forms' reads from being made one, behind registers of addresses)
            } else {
                lookups(std::true_type());
            }
            const uint32_t dw = pw.dw;
            pw.next();
            if (d0 + 256u < pw.n_dw) pw.load(src, ahead);            // the next step's bytes travel under this step's string
            __builtin_amdgcn_sched_barrier(0);
            // four bytes' codes together: at most 48 bits
            uint64_t code[4];
            uint32_t len[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                uint32_t two[2], n_two[2];
#pragma unroll
                for (int b = 0; b < 2; ++b) {
                    const uint32_t l0 = ent[j][2 * b] >> 12;
                    two[b] = (ent[j][2 * b] & 0xfffu) | ((ent[j][2 * b + 1] & 0xfffu) << l0);
                    n_two[b] = l0 + (ent[j][2 * b + 1] >> 12);
                }
                code[j] = (uint64_t)two[0] | ((uint64_t)two[1] << n_two[0]);
                len[j] = n_two[0] + n_two[1];
            }
            if (d0 + 256u > pw.n_dw) {
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    if (dw + j >= pw.n_dw) code[j] = 0ull, len[j] = 0u;
            }
            const uint32_t bits = (len[0] + len[1]) + (len[2] + len[3]);
            const uint32_t incl = wave_inclusive_scan(bits);
            uint32_t pos = carry + incl - bits;
            const uint32_t n_bits = carry + (uint32_t)__builtin_amdgcn_readlane((int)incl, 63);
            // shifted to their place and OR-ed in, two dwords at a time whether or not a bit falls into both; into a third for few.  (Not by lanes
            // behind the chunk's last byte, whose zeros would all go to one address, one after the other: 1024000 records of 36 bytes, where a
            // chunk's last step is a quarter full, encoded in 61 us with them and in 45 so; of 100 bytes 99 and 81.)
            if (bits != 0u) {
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const uint32_t shift = pos & 31u;
                    const uint64_t at_place = code[j] << shift;
                    uint32_t* to = img + (pos >> 5);
                    atomicOr(to, (uint32_t)at_place);
                    atomicOr(to + 1, (uint32_t)(at_place >> 32));
                    if (shift + len[j] > 64u) atomicOr(to + 2, (uint32_t)(code[j] >> 32) >> (32u - shift));
                    pos += len[j];
                }
            }
            wave_fence();
            // whole pieces of 16 bytes leave, the one that is not full stays for the next step
            const uint32_t full = (n_bits >> 7) * 4u;                // dwords, at most 384
            const uint4 rest = *reinterpret_cast<const uint4*>(img + full);
            wave_fence();
            // (waited for here: behind the stores it would have to wait for those as well, which have the next step's time so)
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                asm volatile("" : "+v"(ahead[j]));
                w[j] = ahead[j];
            }
            for (uint32_t i0 = 0; i0 <= full; i0 += 256u) {
                const uint32_t i = i0 + 4u * lane;
                if (i > full) break;
                uint4* p = reinterpret_cast<uint4*>(img + i);
                const uint4 q = *p;
                *p = i == 0u ? rest : make_uint4(0u, 0u, 0u, 0u);
                if (i < full && written + i + 4u <= n_out) *reinterpret_cast<Dwords4*>(out + written + i) = Dwords4{{q.x, q.y, q.z, q.w}};
            }
            wave_fence();
            written += full;
            carry = n_bits & 127u;
        }
        if (lane < 4) {                                              // the last piece
            if (32u * (uint32_t)lane < carry && written + lane < n_out) out[written + lane] = img[lane];
            img[lane] = 0u;
        }
        wave_fence();
    }
}

// (3) with the codes in global memory, and more jobs than compute units, whose tables push each other out of the caches: a dword's four lookups at a time, and the string's
// dwords as they become whole.  (The form above and this one, us: 1000 jobs of 128 records of 200 bytes 91 and 84, 700 of 192 of 400 bytes 199 and 193; 64 of 4000 of 400
// bytes, with the other two launches, 640 and 712, one of 64 43 and 46.)
__global__ void __launch_bounds__(1024) entropy_write_global_kernel(const EntropyArgs a) {
    extern __shared__ uint32_t lds[];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), n_waves = blockDim.x >> 6;
    const int R = a.R;
    const JobView v = job_view(a, blockIdx.y);
    const int64_t first = (int64_t)blockIdx.x * n_waves * a.chunks_per_wave;
    if (!v.ok || first >= v.n_chunks) return;
    uint32_t* img = lds + wave * kImageDw;
    constexpr int kRow = 256;                                        // entries from one byte position to the next
    const uint16_t* tab = a.enc + v.table * 256;
    for (int i = lane; i < kImageDw; i += 64) img[i] = 0u;
    wave_fence();
    for (int c = 0; c < a.chunks_per_wave; ++c) {
        const int64_t chunk = first + (int64_t)c * n_waves + wave;
        if (chunk >= v.n_chunks) break;
        const uint32_t begin = __builtin_amdgcn_readfirstlane(v.chunk_off[chunk]), end = __builtin_amdgcn_readfirstlane(v.chunk_off[chunk + 1]);
        if (end < begin || (uint64_t)end > v.payload_cap) continue;
        const uint32_t n_out = (end - begin) / 4u;
        uint32_t* out = reinterpret_cast<uint32_t*>(v.payload + begin);
        PieceWalk pw(v.T, chunk, R);
        const uint32_t* src = v.rec + chunk * kChunk * pw.per_row;
        const uint32_t rows_end = pw.per_row * (4u * kRow);
        uint32_t carry = 0, written = 0;                             // bits in img[0] left by the step before; dwords stored
        uint32_t w[4];
        pw.load(src, w);
        for (uint32_t d0 = 0; d0 < pw.n_dw; d0 += 256u) {
            // four bytes' codes together: at most 48 bits
            uint64_t code[4];
            uint32_t len[4], row = __umul24(pw.at, 4u * kRow), bits = 0;       // the dword's first entry in the table
            auto codes = [&](auto whole_tag) {
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const uint16_t* e = tab + row;
                    uint32_t ent[4], two[2], n_two[2];
#pragma unroll
                    for (int b = 0; b < 4; ++b) ent[b] = e[b * kRow + ((w[j] >> (8 * b)) & 0xffu)];
#pragma unroll
                    for (int b = 0; b < 2; ++b) {
                        const uint32_t l0 = ent[2 * b] >> 12;
                        two[b] = (ent[2 * b] & 0xfffu) | ((ent[2 * b + 1] & 0xfffu) << l0);
                        n_two[b] = l0 + (ent[2 * b + 1] >> 12);
                    }
                    const bool in = decltype(whole_tag)::value || pw.dw + j < pw.n_dw;
                    code[j] = in ? (uint64_t)two[0] | ((uint64_t)two[1] << n_two[0]) : 0ull;
                    len[j] = in ? n_two[0] + n_two[1] : 0u;
                    bits += len[j];
                    row += 4u * kRow;
                    if (row == rows_end) row = 0u;
                }
            };
            if (d0 + 256u <= pw.n_dw) codes(std::true_type()); else codes(std::false_type());
            pw.next();
            if (d0 + 256u < pw.n_dw) pw.load(src, w);                // the next step's bytes travel under this step's string
            const uint32_t incl = wave_inclusive_scan(bits);
            uint32_t pos = carry + incl - bits;
            const uint32_t n_bits = carry + (uint32_t)__builtin_amdgcn_readlane((int)incl, 63);
            if (bits != 0u) {
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const uint32_t shift = pos & 31u;
                    const uint64_t at_place = code[j] << shift;
                    uint32_t* to = img + (pos >> 5);
                    atomicOr(to, (uint32_t)at_place);
                    atomicOr(to + 1, (uint32_t)(at_place >> 32));
                    if (shift + len[j] > 64u) atomicOr(to + 2, (uint32_t)(code[j] >> 32) >> (32u - shift));
                    pos += len[j];
                }
            }
            wave_fence();
            const uint32_t full = n_bits >> 5;                       // at most 384
            const uint32_t rest = img[full];
            wave_fence();
            for (uint32_t i0 = 0; i0 <= full; i0 += 256u) {
                const uint32_t i = i0 + 4u * lane;
                if (i > full) break;
                uint4* p = reinterpret_cast<uint4*>(img + i);
                const uint4 q = *p;
                *p = make_uint4(0u, 0u, 0u, 0u);
                const uint32_t o = written + i;
                if (i + 4u <= full && o + 4u <= n_out) {
                    *reinterpret_cast<Dwords4*>(out + o) = Dwords4{{q.x, q.y, q.z, q.w}};
                } else {
                    const uint32_t qq[4] = {q.x, q.y, q.z, q.w};
#pragma unroll
                    for (int j = 0; j < 4; ++j)
                        if (i + j < full && o + j < n_out) out[o + j] = qq[j];
                }
            }
            wave_fence();
            if (lane == 0) img[0] = rest;
            wave_fence();
            written += full;
            carry = n_bits & 31u;
        }
        if (lane == 0) {                                             // the last, partly filled dword
            if (carry != 0u && written < n_out) out[written] = img[0];
            img[0] = 0u;
        }
        wave_fence();
    }
}

// decode: one wave per chunk, a lane per token.  LDS_TAB: tables in LDS, else in global memory (jobs_wait).  Every read of the container is clamped
// to the job's bytes, so a damaged container gives wrong bytes, never a fault.  A lane decodes eight bytes from a window of four dwords of its
// string in registers (eight codes are at most 96 bits, behind at most 31).  The dwords that the next window may begin in, and those behind,
// are requested when half the codes are taken, and the window is chosen from them at the end: nothing branches, and a wave waits for memory once
// in eight bytes.  (A 64-bit buffer per lane, refilled dword by dword from four that a lane fetched when it had used them up, waited at every
// second byte, because some lane had always just fetched.)  PIECES: a lane keeps eight dwords and requests four more when it has used up as many
// (decode_in_pieces).
// Rows are collected in LDS and stored 64 bytes at a time (stored 16 bytes at a time, straight from the lanes, a line's pieces
// did not meet in the L2: five times the writes to memory, 0.57 ms).
// 256 MiB of records of 128 bytes: 777 us with twelve comparisons per symbol, 326 with three and the buffer, 268 now.  Vector instructions: 21 per symbol (34 with the buffer), half of the cycles; the lanes'
// 24-byte reads come from the L2, a line as often as it is read, because 16 waves' strings do not fit the L1.
typedef uint32_t u32x4_any __attribute__((ext_vector_type(4), aligned(4)));       // on any dword boundary
typedef uint32_t u32x2_any __attribute__((ext_vector_type(2), aligned(4)));
// a byte of a table, at a byte offset that is a multiple of 256 or-ed with an index, plus a constant
template <bool LDS_TAB> __device__ __forceinline__ uint32_t table_byte(const uint8_t* base, uint32_t off, int constant) {
    if constexpr (LDS_TAB) {
        typedef const uint8_t __attribute__((address_space(3))) * lds_ptr;
        return ((lds_ptr)off)[constant];
    } else {
        return base[off + constant];
    }
}
template <bool LDS_TAB, bool PIECES>
__global__ void __launch_bounds__(1024) entropy_decode_kernel(const EntropyArgs a) {
    extern __shared__ uint32_t lds[];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), n_waves = blockDim.x >> 6;
    const int R = a.R;
    const JobView v = job_view(a, blockIdx.y);
    const int64_t first = (int64_t)blockIdx.x * n_waves * a.chunks_per_wave;
    if (!v.ok || first >= v.n_chunks) return;
    uint32_t* out = lds + wave * (kChunk * kDecPitch);
    uint32_t* tab32 = lds + n_waves * (kChunk * kDecPitch);
    const size_t rows = (size_t)a.n_tables * R;
    const uint8_t* g_len = a.dec + v.table * 256;
    const uint8_t* g_sym = a.dec + (rows + v.table) * 256;
    const uint8_t* g_off = a.dec + rows * 512 + v.table * kDecOff;
    // tables at `tab` in LDS, else at g_..: byte offsets of a segment's first row
    const uint32_t seg = (uint32_t)(R < kDecSegment ? R : kDecSegment), tab = LDS_TAB ? lds_offset(tab32) : 0u;
    const uint32_t tab_sym = LDS_TAB ? tab + seg * 256u : 0u, tab_off = LDS_TAB ? tab + seg * 512u : 0u;
    // the limits of four positions at a time, through the scalar unit (constant while the kernel runs)
    typedef const u32x16 __attribute__((address_space(4))) const_u32x16;
    const const_u32x16* lim = (const const_u32x16*)(uintptr_t)uniform_ptr(a.lim + v.table * 4);
    const uint32_t per_row = (uint32_t)R / 4u;
    for (int c = 0; c < a.chunks_per_wave; ++c) {              // the same number of rounds in every wave: there are barriers inside
        const int64_t chunk = first + (int64_t)c * n_waves + wave;
        const bool live = chunk < v.n_chunks;
        int last = 0;                                          // the last dword of the payload, from the chunk's string on, with five behind it
        uint32_t pos = 0;                                      // the lane's next bit, from there
        uint64_t src = 0;                                      // the chunk's string, less the six dwords
        if (live) {
            uint64_t begin = (uint32_t)__builtin_amdgcn_readfirstlane(v.chunk_off[chunk]);
            begin = (begin < v.payload_cap ? begin : v.payload_cap) & ~3ull;
            const uint64_t left = (v.payload_cap - begin) / 4u;
            last = (int)(left < 0x7fffffffull ? left : 0x7fffffffull) - 6;       // (of a shorter payload: in the directory in front of it)
            src = (uint64_t)uniform_ptr(v.payload + begin) - 24u;
            const uint32_t own = v.len_bits[chunk * kChunk + lane];
            pos = wave_inclusive_scan(own) - own;
            if (chunk * kChunk + lane >= v.T) pos = 0u;
        }
        // (lanes behind the last token run along on the first token's string, and their rows are not stored: from the end of the strings on they
        // made the whole wave choose every window the long way.  60 tokens of 36 bytes: 9.2 us there, 8.1 so; of 128: 17.5 and 17.1.)
        uint32_t w0 = 0u, w1 = 0u, w2 = 0u, w3 = 0u;           // the window: dwords pos / 32 and the three behind it
        int at = 0;                                            // dword of the first one at hand
        typedef const char __attribute__((address_space(1))) * global_ptr;
        // PIECES: the eight dwords from `at` on are at hand.  Between two windows pos moves by three dwords at most, two of them behind the request; it
        // asks for four more where fewer than five would be left in front of the window.  (The window's own first dword is carried over.)
        u32x4 lo{}, hi{};
        int behind = 0;                                        // of `hi`: its dwords that lie behind the payload's end
        auto piece = [&](int d) {
            const int from = min(d, last + 2);
            behind = d - from;
            return (u32x4)*reinterpret_cast<const u32x4_any __attribute__((address_space(1)))*>((global_ptr)src + (uint32_t)(from + 6) * 4u);
        };
        auto settle = [&]() {
            while (__builtin_expect(__any(behind > 0), 0)) {
                const bool on = behind > 0;
                hi[0] = on ? hi[1] : hi[0];
                hi[1] = on ? hi[2] : hi[1];
                hi[2] = on ? hi[3] : hi[2];
                behind = min(behind, 3) - 1;                   // far behind the end everything is stray
            }
        };
        uint32_t g0 = 0u, g1 = 0u, g2 = 0u, g3 = 0u, g4 = 0u, g5 = 0u;
        auto request = [&]() {
            if constexpr (PIECES) {
                if ((int)(pos >> 5) - at >= 3) {
                    lo = hi;
                    at += 4;
                    hi = piece(at + 4);
                }
            } else {
                at = min((int)(pos >> 5), last);
                const global_ptr from = (global_ptr)src + (uint32_t)(at + 6) * 4u;
                const u32x4_any four = *reinterpret_cast<const u32x4_any __attribute__((address_space(1)))*>(from);
                const u32x2_any two = *reinterpret_cast<const u32x2_any __attribute__((address_space(1)))*>(from + 16);
                g0 = four[0]; g1 = four[1]; g2 = four[2]; g3 = four[3]; g4 = two[0]; g5 = two[1];
            }
        };
        auto choose = [&]() {                                  // (what lies behind the payload's end is stray, and no code reads it)
            if constexpr (PIECES) {
                settle();
                const int i = (int)(pos >> 5) + 1 - at;        // 0 .. 5
                const bool b0 = (i & 1) != 0, b1 = (i & 2) != 0, b2 = (i & 4) != 0;
                const uint32_t x0 = b2 ? hi[0] : lo[0], x1 = b2 ? hi[1] : lo[1], x2 = b2 ? hi[2] : lo[2], x3 = b2 ? hi[3] : lo[3];
                const uint32_t y0 = b1 ? x2 : x0, y1 = b1 ? x3 : x1, y2 = b1 ? hi[0] : x2, y3 = b1 ? hi[1] : x3;
                w1 = b0 ? y1 : y0;
                w2 = b0 ? y2 : y1;
                w3 = b0 ? y3 : y2;
            } else {
                int d = (int)(pos >> 5) - at;                  // 0 .. 2, but near the payload's end
                while (__builtin_expect(__any(d > 2), 0)) {
                    const bool on = d > 2;
                    g0 = on ? g1 : g0;
                    g1 = on ? g2 : g1;
                    g2 = on ? g3 : g2;
                    g3 = on ? g4 : g3;
                    g4 = on ? g5 : g4;
                    d -= on ? (d > 8 ? d - 2 : 1) : 0;          // far behind the end everything is stray
                }
                const bool one = d == 1, two = d == 2;
                w0 = two ? g2 : (one ? g1 : g0);
                w1 = two ? g3 : (one ? g2 : g1);
                w2 = two ? g4 : (one ? g3 : g2);
                w3 = two ? g5 : (one ? g4 : g3);
            }
        };
        auto first_window = [&]() {
            if constexpr (PIECES) {
                at = (int)(pos >> 5);
                hi = piece(at);
                settle();
                lo = hi;
                w0 = lo[0];
                hi = piece(at + 4);
            } else {
                request();
            }
            choose();
        };
        // the codes of the four bytes of a dword whose rows of the length table begin here: reversed bits and lengths
        auto lengths = [&](uint32_t t_len, const u32x16& L, uint32_t (&rev)[4], uint32_t (&len)[4]) {
#pragma unroll
            for (int pair = 0; pair < 2; ++pair) {
                uint32_t view = __builtin_amdgcn_alignbit(w1, w0, pos);          // the next 32 bits
#pragma unroll
                for (int b = 2 * pair; b < 2 * pair + 2; ++b) {
                    rev[b] = __builtin_bitreverse32(view);
                    uint32_t n = table_byte<LDS_TAB>(g_len, t_len | (view & 0xffu), b * 256);
                    n += rev[b] > L[4 * b] ? 1u : 0u;
                    n += rev[b] > L[4 * b + 1] ? 1u : 0u;
                    n += rev[b] > L[4 * b + 2] ? 1u : 0u;
                    len[b] = n;
                    view >>= n;
                }
                const uint32_t was = pos >> 5;
                pos += len[2 * pair] + len[2 * pair + 1];
                const bool on = (pos >> 5) != was;
                w0 = on ? w1 : w0;
                w1 = on ? w2 : w1;
                w2 = on ? w3 : w2;
            }
        };
        auto offsets = [&](uint32_t t_off, const uint32_t (&len)[4], uint32_t (&off)[4]) {
#pragma unroll
            for (int b = 0; b < 4; ++b) off[b] = table_byte<LDS_TAB>(g_off, t_off + len[b], b * kDecOff);
        };
        auto symbols = [&](uint32_t t_sym, const uint32_t (&rev)[4], const uint32_t (&len)[4], const uint32_t (&off)[4], uint32_t (&byte)[4]) {
#pragma unroll
            for (int b = 0; b < 4; ++b) {
                const uint32_t rank = (rev[b] >> ((32u - len[b]) & 31u)) - off[b];
                byte[b] = table_byte<LDS_TAB>(g_sym, t_sym | (rank & 0xffu), b * 256);
            }
        };
        auto joined = [](const uint32_t (&byte)[4]) { return byte[0] | (byte[1] << 8) | (byte[2] << 16) | (byte[3] << 24); };
        if (live) first_window();
        for (uint32_t p0 = 0; p0 < per_row; p0 += kDecSegment / 4) {
            const uint32_t p1 = min(per_row, p0 + (uint32_t)kDecSegment / 4u);
            if (LDS_TAB && (c == 0 || per_row > (uint32_t)kDecSegment / 4u)) {
                __syncthreads();
                const uint32_t n = 4u * (p1 - p0);             // rows
                // (a piece of all three tables requested together: one table after the other, 64 tensors of 6000 tokens of 16 bytes took 14.2 us, 12.3 so)
                static_assert(kDecSegment <= 256, "a piece of offsets per thread");
                const uint4* from_len = reinterpret_cast<const uint4*>(g_len + 4u * p0 * 256u);
                const uint4* from_sym = reinterpret_cast<const uint4*>(g_sym + 4u * p0 * 256u);
                const uint4* from_off = reinterpret_cast<const uint4*>(g_off + 4u * p0 * kDecOff);
                uint4* to = reinterpret_cast<uint4*>(tab32);
                uint4 o{};
                if (threadIdx.x < n) o = from_off[threadIdx.x];
#pragma unroll 4
                for (uint32_t i = threadIdx.x; i < n * 16u; i += blockDim.x) {
                    const uint4 l = from_len[i], s = from_sym[i];
                    to[i] = l;
                    to[seg * 16u + i] = s;
                }
                if (threadIdx.x < n) to[seg * 32u + threadIdx.x] = o;
                __syncthreads();
            }
            if (!live) continue;
            // kDecBatch dwords of every row at a time: collected in LDS, stored as whole 64-byte pieces
            const uint32_t row0 = LDS_TAB ? 0u : 4u * p0;
            for (uint32_t d0 = p0; d0 < p1; d0 += kDecBatch) {
                const uint32_t nd = min(p1 - d0, (uint32_t)kDecBatch);
                uint32_t* to = out + lane * kDecPitch;
                uint32_t rev[2][4], len[2][4], off[2][4], byte[2][4];           // of the dwords whose lengths were found last
                uint32_t row = row0 + 4u * (d0 - p0), d = 0;
                // the symbols of two dwords are looked up while the lengths of the next two are found: only those wait for each other
                auto pair_of = [&](auto first_tag, auto both_tag) {
                    constexpr bool kFirst = decltype(first_tag)::value, kBoth = decltype(both_tag)::value;
                    const u32x16 La = lim[d0 + d], Lb = lim[min(d0 + d + 1u, per_row - 1u)];
                    uint32_t rev_n[2][4], len_n[2][4];
                    if constexpr (!kFirst) {
                        offsets(tab_off + (row - 8u) * kDecOff, len[0], off[0]);
                        offsets(tab_off + (row - 4u) * kDecOff, len[1], off[1]);
                    }
                    lengths(tab + row * 256u, La, rev_n[0], len_n[0]);
                    const bool more = d0 + d + (kBoth ? 2u : 1u) < per_row;
                    if (more) request();
                    if constexpr (!kFirst) {
                        symbols(tab_sym + (row - 8u) * 256u, rev[0], len[0], off[0], byte[0]);
                        symbols(tab_sym + (row - 4u) * 256u, rev[1], len[1], off[1], byte[1]);
                    }
                    if constexpr (kBoth) lengths(tab + row * 256u + 1024u, Lb, rev_n[1], len_n[1]);
                    if constexpr (!kFirst) {
                        to[d - 2u] = joined(byte[0]);
                        to[d - 1u] = joined(byte[1]);
                    }
                    if (more) choose();
#pragma unroll
                    for (int b = 0; b < 4; ++b) {
                        rev[0][b] = rev_n[0][b];
                        len[0][b] = len_n[0][b];
                        if constexpr (kBoth) {
                            rev[1][b] = rev_n[1][b];
                            len[1][b] = len_n[1][b];
                        }
                    }
                    d += kBoth ? 2u : 1u;
                    row += kBoth ? 8u : 4u;
                };
                auto rest = [&](uint32_t at_d, uint32_t at_row, int k) {
                    offsets(tab_off + at_row * kDecOff, len[k], off[k]);
                    symbols(tab_sym + at_row * 256u, rev[k], len[k], off[k], byte[k]);
                    to[at_d] = joined(byte[k]);
                };
                if (nd >= 2u) {
                    pair_of(std::true_type(), std::true_type());
                    while (d + 2u <= nd) pair_of(std::false_type(), std::true_type());
                    rest(d - 2u, row - 8u, 0);
                    rest(d - 1u, row - 4u, 1);
                }
                if (d < nd) {
                    pair_of(std::true_type(), std::false_type());
                    rest(d - 1u, row - 4u, 0);
                }
                wave_fence();
                {
                    const uint32_t n_rows = (uint32_t)min(v.T - chunk * kChunk, (int64_t)kChunk);
                    uint32_t* to = v.rec + chunk * kChunk * per_row + d0;
                    if (nd == kDecBatch) {
#pragma unroll
                        for (uint32_t i = 0; i < 4; ++i) {
                            const uint32_t r = 16u * i + (lane >> 2), k = 4u * (lane & 3u);
                            const uint4 q = *reinterpret_cast<const uint4*>(out + r * kDecPitch + k);
                            if (r < n_rows) *reinterpret_cast<Dwords4*>(to + r * per_row + k) = Dwords4{{q.x, q.y, q.z, q.w}};
                        }
                    } else {
                        const uint32_t k = lane & 15u;
                        for (uint32_t r = lane >> 4; r < n_rows; r += 4u)
                            if (k < nd) to[r * per_row + k] = out[r * kDecPitch + k];
                    }
                }
                wave_fence();
            }
        }
    }
}

// decode of records of up to kLogMost bytes under complete codes: a lane per token as above, but the string comes through LDS, where a code's window is one read
// whatever the lane's place in it, and a length is one lookup (kLogRow): 9 vector instructions to a symbol where the form above has 21.  A lane fetches 68
// bytes for every 32 positions, eight positions ahead of their use, or under the chunk before; the records leave as the flat runs of bytes that they are,
// whole lines, past the caches (they pushed the strings out of the L2s that are read up to four times).  A wave takes four codes from a window of 64 bits, and looks
// up four symbols meanwhile.  Bound by the LDS, 3.9 reads to a symbol and in use for half of the time, with four waves to a SIMD, as many as the strings leave room
// for, that wait for each other's lookups.
// 256 MiB of records of 128 bytes: 264 us by the form above, 162 to 175 so, by the card (192 with 64-byte pieces of rows and windows of two codes); 64 tensors of 30000 tokens of 100
// bytes 292 and 117; one of 64 tokens 16 and 13, with waves that help to copy the tables 11.  With stores that the caches keep: 256 MiB 196 for 185, 64 MiB 51.2 49.6, 32 MiB 29.5
// 27.5, 1 MiB 12.1 11.9; and with kvtc_decode_batch behind it, which reads the records again: 1442 1442, 379 348, 167 169, 22.2 22.3 (16 and 128 MiB 88 91, 716 734).
template <int N> using row_of = std::integral_constant<int, N>;
__global__ void __launch_bounds__(1024) entropy_decode_staged_kernel(const EntropyArgs a) {
    extern __shared__ uint32_t lds[];
    typedef const uint8_t __attribute__((address_space(3))) * lds_u8;
    typedef uint32_t __attribute__((address_space(3))) * lds_u32;
    typedef const char __attribute__((address_space(1))) * global_ptr;
    const uint32_t lane = threadIdx.x & 63u, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), n_waves = a.waves;
    const uint32_t R = (uint32_t)a.R, per_row = R / 4u;
    const JobView v = job_view(a, blockIdx.y);
    const int64_t first = (int64_t)blockIdx.x * n_waves * a.chunks_per_wave;
    if (!v.ok || first >= v.n_chunks) return;
    const uint32_t slot = (uint32_t)log_bytes((int)R) + wave * kLogSlot, slot_bit = slot / 8u, lane4 = lane * 4u;

    // the chunk being decoded: its string less a dword, the last dword of the payload from its first on; the slot's first dword
    uint64_t src = 0;
    int last = 0;
    uint32_t base = 0, at = 0;                                     // at: slot_bit + the lane's next bit from the slot's first on, less 32 for every code since
    uint32_t q[kLogString];                                        // the slot's next content
    auto request = [&](uint32_t d) {
        if (__all((int)d <= last - (kLogString - 1))) {
            const global_ptr from = (global_ptr)src + (d * 4u + 4u);
#pragma unroll
            for (int i = 0; i < kLogString / 4; ++i) {
                const u32x4_any w = reinterpret_cast<const u32x4_any __attribute__((address_space(1)))*>(from)[i];
#pragma unroll
                for (int k = 0; k < 4; ++k) q[4 * i + k] = w[k];
            }
            q[kLogString - 1] = reinterpret_cast<const uint32_t __attribute__((address_space(1)))*>(from)[kLogString - 1];
        } else {                                                    // near the payload's end: dword by dword, none behind it
#pragma unroll
            for (int i = 0; i < kLogString; ++i)
                q[i] = *reinterpret_cast<const uint32_t __attribute__((address_space(1)))*>((global_ptr)src + (uint32_t)(min((int)d + i, last) + 1) * 4u);
        }
    };
    uint32_t next_off = 0, next_own = 0;                            // of the next chunk, on their way
    auto directory = [&](int64_t chunk) {
        next_off = v.chunk_off[chunk];
        next_own = v.len_bits[chunk * kChunk + lane];
    };
    // the next chunk's first string; returns the lane's first bit in it
    auto enter = [&](int64_t chunk) {
        uint64_t begin = (uint32_t)__builtin_amdgcn_readfirstlane((int)next_off);
        begin = (begin < v.payload_cap ? begin : v.payload_cap) & ~3ull;
        const uint64_t left = (v.payload_cap - begin) / 4u;
        last = (int)(left < 0x7fffffffull ? left : 0x7fffffffull) - 1;
        src = (uint64_t)uniform_ptr(v.payload + begin) - 4u;        // (of an empty payload: the directory's last dword)
        uint32_t bit = wave_inclusive_scan(next_own) - next_own;
        if (chunk * kChunk + lane >= v.T) bit = 0u;                 // (lanes behind the last token run along on the first one's string)
        base = bit >> 5;
        request(base);
        return bit & 31u;
    };

    int64_t chunk = first + wave;
    const bool live = wave < n_waves && chunk < v.n_chunks;
    if (live) directory(chunk);
    {
        const uint4* from = reinterpret_cast<const uint4*>(a.log + v.table * kLogRow);
        uint4* to = reinterpret_cast<uint4*>(lds);
        const uint32_t n_sym = R * 16u, n_off = n_sym + R * (kDecOff / 16), n = R * (kLogRow / 16);
#pragma unroll 6
        for (uint32_t i = threadIdx.x; i < n; i += blockDim.x)
            to[i < n_sym ? i : (i < n_off ? i - n_sym + kLogOff / 16 : i - n_off + kLogLen / 16)] = from[i];
    }
    if (live) at = slot_bit + enter(chunk);
    __syncthreads();
    if (wave >= n_waves) return;
    for (int c = 0; c < a.chunks_per_wave; ++c, chunk += n_waves) {
        if (chunk >= v.n_chunks) break;
        const bool follows = c + 1 < a.chunks_per_wave && chunk + n_waves < v.n_chunks;
        uint32_t o[kLogMost / 4];                                   // the row
        uint32_t rev[4], m[4];                                      // of the four codes found last: the string from there, first bit on top; 32 - length
        auto length = [&](uint32_t bits, auto row_tag) {
            // 1 + half the string's first 22 bits as a fraction, taken from 1.5 - 2^-23: half of their complement; times 2^-119, all of it exact
            const float x = __uint_as_float(__builtin_amdgcn_alignbit(0x3f800000u >> 22, bits, 10));
            const float f = __builtin_fmaf(x, -0x1p-119f, (float)(1.5 - 0x1p-23) * 0x1p-119f);
            return (uint32_t)((lds_u8)__builtin_amdgcn_alignbit(1u, __float_as_uint(f), 17))[kLogLen - 32768 + decltype(row_tag)::value * kLogEntries];
        };
        // the ranks of two symbols: the code less its length's offset, modulo 256.  (The wait state is for a vector instruction that reads the second.)
        auto ranks = [&](int b, const uint32_t (&off)[4], uint32_t (&rank)[4]) {
            asm("v_sub_u16_sdwa %0, %2, %3 dst_sel:BYTE_0 dst_unused:UNUSED_PAD src0_sel:WORD_0 src1_sel:WORD_0\n\t"
                "v_sub_u16_sdwa %1, %4, %5 dst_sel:BYTE_0 dst_unused:UNUSED_PAD src0_sel:WORD_0 src1_sel:WORD_0\n\t"
                "s_nop 0"
                : "=&v"(rank[b]), "=v"(rank[b + 1])
                : "v"(rev[b] >> (m[b] & 31u)), "v"(off[b]), "v"(rev[b + 1] >> (m[b + 1] & 31u)), "v"(off[b + 1]));
        };
        // the codes of positions row .. row + 3, and meanwhile the symbols of the four before, two at a time
        auto four = [&](auto row_tag) {
            constexpr int row = decltype(row_tag)::value, k = row % kLogUnit;
            constexpr bool before = row > 0;
            const lds_u32 w = (lds_u32)(((at << 3) & ~255u) | lane4);
            const uint32_t w0 = w[k * 64], w1 = w[k * 64 + 64], w2 = w[k * 64 + 128];
            uint32_t off[4], rank[4], byte[4];
            if constexpr (before) {
#pragma unroll
                for (int b = 0; b < 4; ++b) off[b] = ((lds_u8)m[b])[kLogOff - 16 + (row - 4 + b) * kDecOff];
            }
            __builtin_amdgcn_sched_barrier(0);
            uint32_t r[4], n[4];
            r[0] = __builtin_bitreverse32(__builtin_amdgcn_alignbit(w1, w0, at));
            n[0] = length(r[0], row_of<row>());
            uint32_t low = __builtin_bitreverse32(__builtin_amdgcn_alignbit(w2, w1, at));
            __builtin_amdgcn_sched_barrier(0);
            if constexpr (before) {
                ranks(0, off, rank);
#pragma unroll
                for (int b = 0; b < 2; ++b) byte[b] = ((lds_u8)rank[b])[kLogSym + (row - 4 + b) * 256];
            }
            __builtin_amdgcn_sched_barrier(0);
            r[1] = __builtin_amdgcn_alignbit(r[0], low, n[0]);
            n[1] = length(r[1], row_of<row + 1>());
            low = __builtin_amdgcn_alignbit(low, 0u, n[0]);
            __builtin_amdgcn_sched_barrier(0);
            if constexpr (before) {
                ranks(2, off, rank);
#pragma unroll
                for (int b = 2; b < 4; ++b) byte[b] = ((lds_u8)rank[b])[kLogSym + (row - 4 + b) * 256];
            }
            __builtin_amdgcn_sched_barrier(0);
            r[2] = __builtin_amdgcn_alignbit(r[1], low, n[1]);
            n[2] = length(r[2], row_of<row + 2>());
            __builtin_amdgcn_sched_barrier(0);
            if constexpr (before) o[row / 4 - 1] = byte[0] | (byte[1] << 8) | (byte[2] << 16) | (byte[3] << 24);
            __builtin_amdgcn_sched_barrier(0);
            r[3] = __builtin_amdgcn_alignbit(r[2], 0u, n[2]);
            n[3] = length(r[3], row_of<row + 3>());
            __builtin_amdgcn_sched_barrier(0);
            at -= n[0] + n[1] + n[2] + n[3];
#pragma unroll
            for (int b = 0; b < 4; ++b) {
                rev[b] = r[b];
                m[b] = n[b];
            }
            __builtin_amdgcn_sched_barrier(0);
        };
        auto has = [&](uint32_t row) {                              // (compared where it is asked: 32 answers kept through the loop are too many)
            uint32_t r = R;
            asm volatile("" : "+s"(r));
            return row < r;
        };
        uint32_t then = 0;                                          // where the next chunk begins
        auto unit = [&](auto row_tag) {
            constexpr int row = decltype(row_tag)::value;
#pragma unroll
            for (int i = 0; i < kLogString; ++i) ((lds_u32)(slot + lane4))[i * 64] = q[i];
            if (row == 0 && follows) directory(chunk + n_waves);
            const bool final = !has(row + kLogUnit);
            if (final && follows) then = slot_bit + enter(chunk + n_waves);
            four(row_of<row>());
            if (has(row + 4u)) four(row_of<row + 4>());
            if (has(row + 8u)) four(row_of<row + 8>());
            if (has(row + 12u)) four(row_of<row + 12>());
            if (has(row + 16u)) four(row_of<row + 16>());
            if (has(row + 20u)) four(row_of<row + 20>());
            uint32_t moved = 0;
            if (!final) {
                moved = (uint32_t)((int)(at - slot_bit) >> 5) + (kLogUnit - kLogAhead);
                base += moved;
                request(base);
            }
            if (has(row + 24u)) four(row_of<row + 24>());
            if (has(row + 28u)) four(row_of<row + 28>());
            at += 32u * (kLogUnit - moved);
        };
        unit(row_of<0>());
        if (has(32u)) unit(row_of<32>());
        if (has(64u)) unit(row_of<64>());
        if (has(96u)) unit(row_of<96>());
        uint32_t tail = 0;                                          // the row's last dword, whose symbols are still to be looked up
#pragma unroll
        for (uint32_t b = 0; b < 4; ++b) {
            const uint32_t row = R - 4u + b, off = ((lds_u8)(m[b] + row * kDecOff))[kLogOff - 16];
            tail |= (uint32_t)((lds_u8)((((rev[b] >> (m[b] & 31u)) - off) & 0xffu) + row * 256u))[kLogSym] << (8 * b);
        }
        at = then;
        // (the next string has landed by now: waited for in front of the stores, so that nothing waits for those)
#pragma unroll
        for (int i = 0; i < kLogString; ++i) asm volatile("" : "+v"(q[i]));
        // the rows, 32 at a time, through the slot, and from there as the flat run of bytes that they are.  (16-byte pieces of rows of a power of two are
        // permuted, so that 16 rows' pieces lie on different banks.)
        const uint32_t n_rows = (uint32_t)min(v.T - chunk * kChunk, (int64_t)kChunk);
        uint32_t* const img = lds + slot / 4u;
        const uint32_t swizzle = per_row == 32u ? 7u : (per_row == 16u ? 3u : 0u);
        uint32_t l = lane;
        asm volatile("" : "+v"(l));                                 // (addresses are worked out here, not kept through the loop)
        for (uint32_t r0 = 0; r0 < n_rows; r0 += 32u) {
            if ((l & 32u) == r0) {
                const uint32_t r = l & 31u, x = (per_row == 32u ? r >> 1 : r >> 2) & swizzle;
                if (per_row % 4u == 0u) {
#pragma unroll
                    for (uint32_t k = 0; k < kLogMost / 16; ++k)
                        if (has(16u * k)) *reinterpret_cast<uint4*>(img + r * per_row + 4u * (k ^ x)) = make_uint4(o[4 * k], o[4 * k + 1], o[4 * k + 2], o[4 * k + 3]);
                } else {
#pragma unroll
                    for (uint32_t d = 0; d < kLogMost / 4; ++d)
                        if (has(4u * d)) img[r * per_row + d] = o[d];
                }
                img[r * per_row + (per_row - 1u ^ 4u * x)] = tail;
            }
            wave_fence();
            const uint32_t n = min(n_rows - r0, 32u) * per_row;
            uint32_t* to = v.rec + (chunk * kChunk + r0) * per_row;
#pragma unroll
            for (uint32_t i = 0; i < kLogMost / 32; ++i) {
                const uint32_t f = 64u * i + l, d = 4u * f;
                if (d >= n) break;
                const uint4 w = *reinterpret_cast<const uint4*>(img + 4u * (f ^ ((f >> 4) & swizzle)));
                if (d + 4u <= n) {
                    __builtin_nontemporal_store(u32x4{w.x, w.y, w.z, w.w}, reinterpret_cast<u32x4_any*>(to + d));
                } else {
                    to[d] = w.x;
                    if (d + 1u < n) to[d + 1] = w.y;
                    if (d + 2u < n) to[d + 2] = w.z;
                }
            }
            wave_fence();
        }
    }
}

uint32_t reverse_bits(uint32_t v, int n) { return __builtin_bitreverse32(v) >> (32 - n); }      // n from 1 up

// 32 - length by the float index of u, for a complete code with count[L] codes of L bits.  (Length by length, not entry by entry: 64 tensors' tables of 128
// positions would take 4 ms more to create.)
void log_lengths(const uint32_t (&count)[kMaxLen + 1], uint8_t* entries) {
    auto first_at = [](uint32_t u) {                                // the first index whose u is no smaller
        if (u < 128) return (int)u;
        const int octave = 25 - __builtin_clz(u);
        return 64 * octave + (int)((u + (1u << octave) - 1) >> octave);
    };
    int done = 0;
    for (uint32_t below = 0, len = kMaxLen; len >= 1; --len) {      // u is below `below` for codes of `len` bits and more
        below += count[len] << (kMaxLen - len);
        const int end = len > 1 ? std::min(first_at(below), kLogEntries) : kLogEntries;
        memset(entries + done, (int)(32 - len), (size_t)(end - done));
        done = end;
    }
}

size_t bound_of(int R, int64_t n_tokens) {
    const int64_t n_chunks = (n_tokens + kChunk - 1) / kChunk;
    return (size_t)header_bytes(n_chunks) + (size_t)n_chunks * chunk_image_dwords(R) * 4;
}

// The shape of a launch over `n_chunks` chunks of each of n_jobs jobs.  A launch all of whose chunks can run at once does that, with
// the fewest waves per workgroup, from four up, that allow it: the compute units share the chunks, and each of their waves has
// more of its vector unit.  A larger one runs workgroups of 16 waves, or 8 where that lets more waves share a compute unit's LDS
// (4 where the jobs have no more chunks).  Each wave takes as many chunks in turn (at most in_turn) as end soonest: every compute unit works through its
// workgroups, each of which first copies its table (64 KiB for 128-byte records, against 8 KiB of records per chunk; counted as a fifth of a round of chunks),
// as long as every place on the chip is taken.  (Rounded down from the chunks to a place, 64 tensors of 469 chunks of 100 bytes were 320 workgroups on 256 compute units:
// encode 178 us and 168 now, 37 of 360 of 120 bytes 130 and 102.  The general decoder's tables of short records are small: at most eight chunks, 1000 tensors of 8000 tokens
// of 4 bytes 79 us, 91 with sixteen.)  Without a
// table in LDS workgroups are as small as they can be, or, with more jobs than compute units, a job (of up to 16 chunks) each: then a
// compute unit's caches hold few tables.
// (2188 chunks of 128-byte records, encode and decode: 75 + 102 us with four waves that took two chunks in turn on one workgroup per
// compute unit, 45 + 31 so, 35 + 18 with the kernels as they are; 64 tensors of 63 chunks 83 + 145, 41 + 39, 39 + 26 (of 64).  Ten waves in a workgroup, two of which a
// compute unit has room for at 128 bytes, 20 waves instead of 16, but twice the copies of the table: encode of 64 tensors of 512 chunks 211 us and 215 so.)
struct Shape { int waves, chunks_per_wave; unsigned blocks; size_t lds; };
Shape launch_shape(size_t table_b, size_t wave_b, int64_t n_chunks, int n_jobs, int in_turn = 16) {
    const int64_t total = n_chunks * n_jobs, cus = compute_units();
    auto shape = [&](int waves, int64_t per) { return Shape{waves, (int)per, (unsigned)((n_chunks + waves * per - 1) / (waves * per)), table_b + (size_t)waves * wave_b}; };
    if (table_b == 0) return shape(n_jobs > cus ? (int)std::clamp<int64_t>(n_chunks, 4, 16) : total > cus ? 2 : 1, 1);
    auto places = [&](int w) -> int64_t {                        // workgroups a compute unit takes
        const size_t b = table_b + (size_t)w * wave_b;
        return b > (size_t)kLdsMost ? 0 : std::min<int64_t>(kLdsBudget / b, 32 / w);
    };
    for (const int w : {4, 6, 8, 12, 16})
        if ((n_chunks + w - 1) / w * n_jobs <= cus * places(w)) return shape(w, 1);
    int waves = 4;
    for (const int w : {8, 16})
        if (n_chunks > w / 2 && places(w) > 0 && (waves == 4 || places(w) * w >= places(waves) * waves)) waves = w;
    int64_t best = 1, least = INT64_MAX;
    for (int64_t per = 1; per <= in_turn; ++per) {
        const int64_t to_each = ((n_chunks + waves * per - 1) / (waves * per) * n_jobs + cus - 1) / cus, cost = to_each * (5 * per + 1);
        if (per > 1 && to_each < places(waves)) break;
        if (cost < least) least = cost, best = per;
    }
    return shape(waves, best);
}

// Whether jobs of a few chunks each, a workgroup per job, would wait for others to leave the LDS.  Then they read their tables from global
// memory instead: 1000 tensors of one chunk, 128-byte records: encode 36 us with the tables in LDS, 28 without, decode 76 and 34
// (25 and 26 without, with the kernels as they are); with places for all, 250 tensors: 22 and 23, 21 and 31.  (At three chunks in encode, five in decode, the copy pays again.)
bool jobs_wait(size_t table_b, size_t wave_b, int n_jobs) { return n_jobs > compute_units() * (int)(kLdsBudget / (table_b + 4 * wave_b)); }

// Whether decode reads its strings in pieces of 16 bytes, each once, and not a whole window for every eight bytes: where the records that the
// chip works on at a time, and their strings, do not fit the L2s (4 MiB on each of 8 XCDs), so that a line read again comes from behind them.  Waves of
// a launch of one round go through their records in step; a second round is shorter, or the first one's last waves run beside it; in more the
// waves are spread over their records.  Records shorter than a line share it with their neighbours' strings.
// Both sides, us, whole windows and pieces: 4096 chunks at once of records of 120 bytes 34.4 and 36.6, 128 bytes 43.3 and 35.1, 200 bytes 107 and 74;
// 3008 chunks of 160 bytes 41.6 and 42.6, 176 bytes 49.4 and 46.9; two rounds of 3008 chunks of 140 bytes 75.5 and 77.2, 148 bytes 91.2 and 87.3; 12032 chunks
// of 148 bytes 161 and 165, 160 bytes 184 and 171, 256 bytes 418 and 276 (326 with a 64-bit buffer per lane).
bool decode_in_pieces(const Shape& sh, int R, int64_t n_chunks, int n_jobs) {
    const int64_t places = compute_units() * std::min<int64_t>(kLdsBudget / sh.lds, 32 / sh.waves);        // workgroups at once
    const int64_t rounds = ((int64_t)sh.blocks * n_jobs + places - 1) / places * sh.chunks_per_wave;
    const int64_t at_once = (rounds <= 2 ? n_chunks * n_jobs / rounds : places * sh.waves) * kChunk * R;
    return R >= 128 && (rounds == 1 ? at_once > 30 << 20 : rounds == 2 ? at_once > 26 << 20 : at_once >= 40 << 20);
}

// Whether the staged decoder, with more LDS to a workgroup, would run jobs of a few chunks in more rounds of workgroups than the other, each of which copies its
// tables for little work.  (LDS is given out in pieces of 1280 bytes.)  us, the other and the staged, one round against two: 1000 jobs of one chunk of 36 bytes 9.2 and 13.3, 400 of
// four of 100 bytes 18.6 and 24.3, of five of 64 bytes 13.4 and 15.4, 257 of seven of 36 bytes 9.7 and 12.8, of twelve 11.5 and 15.0, 400 of twelve 15.1 and 15.5, of eight
// of 48 bytes 13.9 and 13.7; two against three, 600 of seven of 36 bytes, 17.9 and 19.7, of sixteen, three and three, 36.7 and 27.4.
bool small_jobs_wait(const Shape& staged, const Shape& other, int64_t n_chunks, int n_jobs) {
    auto rounds = [&](const Shape& s) {
        const int64_t places = compute_units() * std::min<int64_t>(kLdsBudget / ((s.lds + 1279) / 1280 * 1280), 32 / s.waves);
        return ((int64_t)s.blocks * n_jobs + places - 1) / places;
    };
    return n_chunks <= 12 && rounds(staged) > rounds(other);
}

// The staged decoder's tables begin at the LDS's address 0: a build that gave the kernel LDS of its own in front of what a launch asks for must not run it.
bool staged_lds_at_zero() {
    static std::atomic<bool> seen{false};
    hipFuncAttributes attr;
    if (!seen && hipFuncGetAttributes(&attr, reinterpret_cast<const void*>(&entropy_decode_staged_kernel)) == hipSuccess && attr.sharedSizeBytes == 0) seen = true;
    return seen;
}

// Records of less than a piece of 16 bytes gain little by the staged decoder, or lose by its larger tables where there are more jobs than compute units.
// (us, the other and the staged: 4 bytes, a tensor of one token 3.2 and 3.6, 64 of 1000 4.7 and 5.1, of 30000 25.4 and 25.3, 1000 of 1000 14.4 and 19.3; 8 bytes 3.7 and 3.9, 5.1
// and 5.0, 31.1 and 27.2, 16.9 and 20.8; 12 bytes 4.1 and 4.0, 5.7 and 5.5, 37.5 and 29.2, 19.8 and 22.7; 16 bytes 4.3 and 3.9, 5.9 and 4.8, 40.8 and 27.0, 21.9 and 21.1.)
constexpr int kLogLeast = 12;
bool log_pays(int R, int n_jobs) { return R >= 16 || (R >= kLogLeast && n_jobs <= compute_units()); }

// helpers: the kernel copies tables once and lets waves that take no chunk go, so that the launch may have more of them.
kvtc_status launch(const char* who, void (*fn)(EntropyArgs), const Shape& sh, int n_jobs, EntropyArgs a, hipStream_t st, bool helpers = false) {
    if (allow_full_lds(reinterpret_cast<const void*>(fn)) != hipSuccess) return set_error(KVTC_E_HIP, "%s: cannot size the LDS", who);
    a.waves = sh.waves;
    a.chunks_per_wave = sh.chunks_per_wave;
    const int waves = helpers && (int64_t)sh.blocks * n_jobs <= compute_units() ? 16 : sh.waves;
    hipLaunchKernelGGL(fn, dim3(sh.blocks, (unsigned)n_jobs), dim3(64 * waves), sh.lds, st, a);
    return KVTC_OK;
}

kvtc_status run_encode(const char* who, const kvtc_entropy* e, const EntropyArgs& a_in, int n_jobs, int64_t max_tokens, hipStream_t st) {
    const int R = e->record_bytes;
    const int64_t max_chunks = (max_tokens + kChunk - 1) / kChunk;
    EntropyArgs a = a_in;
    a.max_tokens = max_tokens;
    kvtc_status rc = KVTC_OK;
    if (max_chunks > 0) {
        // (of long records with a chunk to a wave, where a workgroup's copy of the table and the kernel's first pass through the code are most of it, the plain form: 1000 jobs
        // of 128 records of 200 bytes 18.9 us, 21.9 in the other, 700 of 192 of 400 bytes 44 and 50; of 32768 of 128 bytes 80 and 75, one of 64 of 256 bytes, all three launches, 26.5 and 25.5)
        const Shape sh = launch_shape((size_t)R * kLenRow, kChunk * 4, max_chunks, n_jobs);
        rc = launch(who, sh.chunks_per_wave > 1 || R <= 128 || max_chunks * n_jobs <= 2 * compute_units() ? &entropy_size_kernel<true> : &entropy_size_kernel<false>, sh, n_jobs, a, st, true);
    }
    if (rc != KVTC_OK) return rc;
    hipLaunchKernelGGL(entropy_scan_kernel, dim3((unsigned)n_jobs), dim3(max_chunks <= 64 ? 64 : max_chunks <= 256 ? 256 : 1024), 0, st, a);
    if (max_chunks > 0) {
        const bool tab_lds = R <= kMaxLdsRecord &&
                             !(max_chunks <= 2 && jobs_wait((size_t)R * kEncRow, kImageDw * 4, n_jobs));
        rc = launch(who, tab_lds ? &entropy_write_kernel<true> : n_jobs > compute_units() ? &entropy_write_global_kernel : &entropy_write_kernel<false>,
                    launch_shape(tab_lds ? (size_t)R * kEncRow : 0, kImageDw * 4, max_chunks, n_jobs), n_jobs, a, st, tab_lds);
        if (rc != KVTC_OK) return rc;
    }
    const hipError_t err = hipGetLastError();
    if (err != hipSuccess) return set_error(KVTC_E_HIP, "%s: launch failed: %s", who, hipGetErrorString(err));
    return KVTC_OK;
}

kvtc_status run_decode(const char* who, const kvtc_entropy* e, const EntropyArgs& a_in, int n_jobs, int64_t max_tokens, hipStream_t st) {
    const int R = e->record_bytes;
    EntropyArgs a = a_in;
    a.max_tokens = max_tokens;
    const int64_t max_chunks = (max_tokens + kChunk - 1) / kChunk;
    if (max_chunks == 0) return KVTC_OK;
    const size_t table_b = (size_t)(R < kDecSegment ? R : kDecSegment) * kDecRow, wave_b = kChunk * kDecPitch * 4;
    const bool tab_lds = !(max_chunks <= 4 && jobs_wait(table_b, wave_b, n_jobs));
    const Shape sh = launch_shape(tab_lds ? table_b : 0, wave_b, max_chunks, n_jobs, 8);
    void (*const fn)(EntropyArgs) = !tab_lds                                        ? &entropy_decode_kernel<false, false>
                                    : decode_in_pieces(sh, R, max_chunks, n_jobs) ? &entropy_decode_kernel<true, true>
                                                                                    : &entropy_decode_kernel<true, false>;
    const Shape staged = a.log && tab_lds && log_pays(R, n_jobs) && staged_lds_at_zero() ? launch_shape(log_bytes(R), kLogSlot, max_chunks, n_jobs) : Shape{};
    const kvtc_status rc = staged.waves && !small_jobs_wait(staged, sh, max_chunks, n_jobs) ? launch(who, &entropy_decode_staged_kernel, staged, n_jobs, a, st, true)
                                                                                           : launch(who, fn, sh, n_jobs, a, st);
    if (rc != KVTC_OK) return rc;
    const hipError_t err = hipGetLastError();
    if (err != hipSuccess) return set_error(KVTC_E_HIP, "%s: launch failed: %s", who, hipGetErrorString(err));
    return KVTC_OK;
}

EntropyArgs base_args(const kvtc_entropy* e) {
    EntropyArgs a;
    memset(&a, 0, sizeof(a));
    a.enc = e->enc_dev;
    a.len = e->len_dev;
    a.dec = e->dec_dev;
    a.lim = e->lim_dev;
    a.log = e->log_dev;
    a.R = e->record_bytes;
    a.n_tables = e->n_tables;
    return a;
}

}  // namespace

extern "C" {

kvtc_status kvtc_entropy_create(kvtc_entropy** out, int record_bytes, int n_tables, const uint8_t* code_len_host, kvtc_stream stream) {
    if (out) *out = nullptr;
    if (!out || !code_len_host) return set_error(KVTC_E_ARG, "kvtc_entropy_create: null argument");
    const int R = record_bytes;
    if (R < 4 || R % 4 != 0) return set_error(KVTC_E_ARG, "kvtc_entropy_create: record_bytes=%d must be a positive multiple of 4", R);
    if (R > kMaxRecord) return set_error(KVTC_E_UNSUPPORTED, "kvtc_entropy_create: record_bytes=%d above %d", R, kMaxRecord);
    if (n_tables < 1 || n_tables > 4096) return set_error(KVTC_E_ARG, "kvtc_entropy_create: n_tables=%d outside 1..4096", n_tables);
    const size_t rows = (size_t)n_tables * R;
    // (not cleared first, which for 64 tables of 128 positions is a millisecond: all of it is written below)
    const size_t enc_b = rows * 512, dec_b = rows * kDecRow, lim_b = rows * 16, len_b = rows * 256;
    size_t log_b = R >= kLogLeast && R <= kLogMost ? rows * kLogRow : 0;
    const std::unique_ptr<uint16_t[]> enc(new (std::nothrow) uint16_t[rows * 256]);
    const std::unique_ptr<uint8_t[]> dec(new (std::nothrow) uint8_t[dec_b]), log(log_b ? new (std::nothrow) uint8_t[log_b] : nullptr);
    const std::unique_ptr<uint32_t[]> lim(new (std::nothrow) uint32_t[rows * 4]);
    if (!enc || !dec || !lim) return set_error(KVTC_E_NOMEM, "kvtc_entropy_create: host allocation failed");
    if (!log) log_b = 0;                                            // (the other decoder needs none of it)
    for (size_t k = 0; k < rows; ++k) {
        const uint8_t* L = code_len_host + k * 256;
        // canonical codes: by length, then by symbol (RFC 1951, section 3.2.2); Kraft's inequality must hold
        uint32_t count[kMaxLen + 1] = {0};
        for (int s = 0; s < 256; ++s) {
            if (L[s] < 1 || L[s] > kMaxLen)
                return set_error(KVTC_E_ARG, "kvtc_entropy_create: table %d, position %d, symbol %d: length %d outside 1..%d", (int)(k / R), (int)(k % R), s, (int)L[s], kMaxLen);
            ++count[L[s]];
        }
        uint32_t kraft = 0, next[kMaxLen + 1], rank[kMaxLen + 1], code = 0, shorter = 0;
        uint8_t *D = &dec[k * 256], *S = &dec[(rows + k) * 256], *O = &dec[rows * 512 + k * kDecOff];      // lengths, symbols, offsets
        int least = 9;                                              // what the table says for codes of 9 bits or more
        memset(O, 0, kDecOff);
        for (int i = 0; i < 4; ++i) lim[k * 4 + i] = 0xffffffffu;
        for (int len = 1; len <= kMaxLen; ++len) {
            kraft += count[len] << (kMaxLen - len);
            next[len] = code;                                       // first code of this length, and its rank
            rank[len] = shorter;
            O[len] = (uint8_t)(code - shorter);
            code += count[len];
            shorter += count[len];
            if (len >= 9 && len < kMaxLen) {
                if (code != 0) lim[k * 4 + len - 9] = (uint32_t)(((uint64_t)code << (32 - len)) - 1u);
                else ++least;                                       // no code is as short: the table says so, the limit stays out of reach
            }
            code <<= 1;
        }
        if (kraft != (1u << kMaxLen)) log_b = 0;
        if (kraft > (1u << kMaxLen))
            return set_error(KVTC_E_ARG, "kvtc_entropy_create: table %d, position %d: the lengths are not those of a prefix code", (int)(k / R), (int)(k % R));
        memset(D, least, 256);
        for (int s = 0; s < 256; ++s) {
            const int len = L[s];
            const uint32_t rev = reverse_bits(next[len]++, len);
            enc[k * 256 + s] = (uint16_t)(rev | ((uint32_t)len << 12));
            S[rank[len]++] = (uint8_t)s;
            if (len <= 8)
                for (uint32_t i = rev; i < 256u; i += 1u << len) D[i] = (uint8_t)len;
        }
        if (log_b != 0) {
            uint8_t* const set = &log[k / R * R * kLogRow];
            const size_t pos = k % R;
            memcpy(set + pos * 256, S, 256);
            for (int len = 1; len <= kDecOff; ++len) set[(size_t)R * 256 + pos * kDecOff + 16 - len] = len <= kMaxLen ? O[len] : 0;
            log_lengths(count, set + (size_t)R * (256 + kDecOff) + pos * kLogEntries);
        }
    }
    // one allocation: codes, the decoders' tables and limits, lengths
    const size_t least_b = enc_b + dec_b + lim_b + len_b;
    char* blob = nullptr;
    if (log_b != 0 && hipMalloc(reinterpret_cast<void**>(&blob), least_b + log_b) != hipSuccess) {
        (void)hipGetLastError();
        log_b = 0;                                                  // no room for the staged decoder's: the other decoder serves these records
    }
    if (log_b == 0 && hipMalloc(reinterpret_cast<void**>(&blob), least_b) != hipSuccess) {
        (void)hipGetLastError();
        return set_error(KVTC_E_NOMEM, "kvtc_entropy_create: hipMalloc of %zu bytes failed", least_b);
    }
    hipStream_t st = static_cast<hipStream_t>(stream);
    hipError_t e = hipSuccess;
    size_t at = 0;
    auto put = [&](const void* src, size_t n) {
        char* dst = blob + at;
        if (e == hipSuccess) e = hipMemcpyAsync(dst, src, n, hipMemcpyHostToDevice, st);
        at += n;
        return dst;
    };
    const char* enc_d = put(enc.get(), enc_b);
    const char* lim_d = put(lim.get(), lim_b);
    const char* dec_d = put(dec.get(), dec_b);
    const char* len_d = put(code_len_host, len_b);
    const char* log_d = log_b ? put(log.get(), log_b) : nullptr;
    if (e == hipSuccess) e = hipStreamSynchronize(st);           // the host images die with this call
    kvtc_entropy* h = e == hipSuccess ? new (std::nothrow) kvtc_entropy : nullptr;
    if (!h) {
        (void)hipFree(blob);
        return e != hipSuccess ? set_error(KVTC_E_HIP, "kvtc_entropy_create: upload failed: %s", hipGetErrorString(e))
                               : set_error(KVTC_E_NOMEM, "kvtc_entropy_create: host allocation failed");
    }
    h->record_bytes = R;
    h->n_tables = n_tables;
    h->blob = blob;
    h->enc_dev = reinterpret_cast<const uint16_t*>(enc_d);
    h->lim_dev = reinterpret_cast<const uint32_t*>(lim_d);
    h->dec_dev = reinterpret_cast<const uint8_t*>(dec_d);
    h->len_dev = reinterpret_cast<const uint8_t*>(len_d);
    h->log_dev = reinterpret_cast<const uint8_t*>(log_d);
    *out = h;
    return KVTC_OK;
}

void kvtc_entropy_destroy(kvtc_entropy* e) {
    if (!e) return;
    (void)hipFree(e->blob);
    delete e;
}

size_t kvtc_entropy_bound(const kvtc_entropy* e, int64_t n_tokens) {
    if (!e || n_tokens <= 0) return e ? (size_t)header_bytes(0) : 0;
    return bound_of(e->record_bytes, n_tokens);
}

kvtc_status kvtc_entropy_encode(const kvtc_entropy* e, int table, const void* records_dev, int64_t n_tokens, void* out_dev, size_t out_cap,
                                uint64_t* out_bytes_dev, kvtc_stream stream) {
    if (!e) return set_error(KVTC_E_ARG, "kvtc_entropy_encode: null tables");
    if (table < 0 || table >= e->n_tables) return set_error(KVTC_E_ARG, "kvtc_entropy_encode: table=%d outside 0..%d", table, e->n_tables - 1);
    if (n_tokens < 0 || n_tokens > 0x7fffffffLL) return set_error(KVTC_E_ARG, "kvtc_entropy_encode: n_tokens=%lld", (long long)n_tokens);
    if (!out_bytes_dev) return set_error(KVTC_E_ARG, "kvtc_entropy_encode: null out_bytes_dev");
    const int R = e->record_bytes;
    const int64_t n_chunks = (n_tokens + kChunk - 1) / kChunk;
    const uint64_t hdr = header_bytes(n_chunks);
    if (!out_dev || (n_tokens > 0 && !records_dev)) return set_error(KVTC_E_ARG, "kvtc_entropy_encode: null buffer");
    if ((reinterpret_cast<uintptr_t>(records_dev) & 3u) || (reinterpret_cast<uintptr_t>(out_dev) & 3u) || (reinterpret_cast<uintptr_t>(out_bytes_dev) & 7u))
        return set_error(KVTC_E_ARG, "kvtc_entropy_encode: records and output must be 4-byte aligned, out_bytes_dev 8-byte aligned");
    if ((uint64_t)bound_of(R, n_tokens) - hdr >= (1ull << 32))
        return set_error(KVTC_E_UNSUPPORTED, "kvtc_entropy_encode: %lld tokens of %d bytes may exceed the 4 GiB a container addresses", (long long)n_tokens, R);
    if (out_cap < hdr) return set_error(KVTC_E_SMALL, "kvtc_entropy_encode: out_cap=%zu cannot hold the directory of %llu bytes", out_cap, (unsigned long long)hdr);
    EntropyArgs a = base_args(e);
    a.n_jobs = 1;
    a.single = kvtc_entropy_job{table, (int32_t)n_tokens, 0, 0, out_cap};
    a.records = static_cast<const uint8_t*>(records_dev);
    a.records_cap = (uint64_t)n_tokens * R;
    a.coded = static_cast<uint8_t*>(out_dev);
    a.coded_total = out_cap;
    a.coded_bytes = out_bytes_dev;
    return run_encode("kvtc_entropy_encode", e, a, 1, n_tokens, static_cast<hipStream_t>(stream));
}

kvtc_status kvtc_entropy_decode(const kvtc_entropy* e, int table, const void* in_dev, size_t in_bytes, int64_t n_tokens, void* records_out_dev,
                                size_t out_cap, kvtc_stream stream) {
    if (!e) return set_error(KVTC_E_ARG, "kvtc_entropy_decode: null tables");
    if (table < 0 || table >= e->n_tables) return set_error(KVTC_E_ARG, "kvtc_entropy_decode: table=%d outside 0..%d", table, e->n_tables - 1);
    if (n_tokens < 0 || n_tokens > 0x7fffffffLL) return set_error(KVTC_E_ARG, "kvtc_entropy_decode: n_tokens=%lld", (long long)n_tokens);
    if (n_tokens == 0) return KVTC_OK;
    if (!in_dev || !records_out_dev) return set_error(KVTC_E_ARG, "kvtc_entropy_decode: null buffer");
    if ((reinterpret_cast<uintptr_t>(in_dev) & 3u) || (reinterpret_cast<uintptr_t>(records_out_dev) & 3u))
        return set_error(KVTC_E_ARG, "kvtc_entropy_decode: buffers must be 4-byte aligned");
    const int R = e->record_bytes;
    const uint64_t hdr = header_bytes((n_tokens + kChunk - 1) / kChunk);
    if (in_bytes < hdr) return set_error(KVTC_E_SMALL, "kvtc_entropy_decode: in_bytes=%zu below the directory's %llu", in_bytes, (unsigned long long)hdr);
    if (out_cap < (size_t)n_tokens * R) return set_error(KVTC_E_SMALL, "kvtc_entropy_decode: out_cap=%zu < %zu", out_cap, (size_t)n_tokens * R);
    EntropyArgs a = base_args(e);
    a.n_jobs = 1;
    a.single = kvtc_entropy_job{table, (int32_t)n_tokens, 0, 0, in_bytes};
    a.records = static_cast<const uint8_t*>(records_out_dev);
    a.records_cap = (uint64_t)n_tokens * R;
    a.coded = static_cast<uint8_t*>(const_cast<void*>(in_dev));
    a.coded_total = in_bytes;
    return run_decode("kvtc_entropy_decode", e, a, 1, n_tokens, static_cast<hipStream_t>(stream));
}

static kvtc_status batch_checks(const char* who, const kvtc_entropy* e, const kvtc_entropy_job* jobs_dev, int n_jobs, int64_t max_tokens,
                                const void* records, const void* coded, bool* nothing) {
    *nothing = false;
    if (!e) return set_error(KVTC_E_ARG, "%s: null tables", who);
    if (n_jobs < 0 || max_tokens < 0 || max_tokens > 0x7fffffffLL) return set_error(KVTC_E_ARG, "%s: n_jobs=%d, max_tokens=%lld", who, n_jobs, (long long)max_tokens);
    if (n_jobs == 0) { *nothing = true; return KVTC_OK; }
    if (n_jobs > kMaxEntropyJobs) return set_error(KVTC_E_UNSUPPORTED, "%s: %d jobs, at most %d per call", who, n_jobs, kMaxEntropyJobs);
    if (!jobs_dev || !records || !coded) return set_error(KVTC_E_ARG, "%s: null buffer", who);
    if ((reinterpret_cast<uintptr_t>(records) & 3u) || (reinterpret_cast<uintptr_t>(coded) & 3u) || (reinterpret_cast<uintptr_t>(jobs_dev) & 7u))
        return set_error(KVTC_E_ARG, "%s: buffers must be 4-byte aligned, the job table 8-byte aligned", who);
    if ((uint64_t)bound_of(e->record_bytes, max_tokens) >= (1ull << 32))
        return set_error(KVTC_E_UNSUPPORTED, "%s: %lld tokens of %d bytes may exceed the 4 GiB a container addresses", who, (long long)max_tokens, e->record_bytes);
    return KVTC_OK;
}

kvtc_status kvtc_entropy_encode_batch(const kvtc_entropy* e, const kvtc_entropy_job* jobs_dev, int n_jobs, int64_t max_tokens,
                                      const void* records_base_dev, size_t records_bytes, void* coded_base_dev, size_t coded_cap,
                                      uint64_t* coded_bytes_dev, kvtc_stream stream) {
    bool nothing;
    kvtc_status st = batch_checks("kvtc_entropy_encode_batch", e, jobs_dev, n_jobs, max_tokens, records_base_dev, coded_base_dev, &nothing);
    if (st != KVTC_OK || nothing) return st;
    if (!coded_bytes_dev || (reinterpret_cast<uintptr_t>(coded_bytes_dev) & 7u))
        return set_error(KVTC_E_ARG, "kvtc_entropy_encode_batch: coded_bytes_dev must be an 8-byte aligned device array");
    EntropyArgs a = base_args(e);
    a.jobs = jobs_dev;
    a.n_jobs = n_jobs;
    a.records = static_cast<const uint8_t*>(records_base_dev);
    a.records_cap = records_bytes;
    a.coded = static_cast<uint8_t*>(coded_base_dev);
    a.coded_total = coded_cap;
    a.coded_bytes = coded_bytes_dev;
    return run_encode("kvtc_entropy_encode_batch", e, a, n_jobs, max_tokens, static_cast<hipStream_t>(stream));
}

kvtc_status kvtc_entropy_decode_batch(const kvtc_entropy* e, const kvtc_entropy_job* jobs_dev, int n_jobs, int64_t max_tokens,
                                      const void* coded_base_dev, size_t coded_bytes, void* records_base_dev, size_t records_cap,
                                      kvtc_stream stream) {
    bool nothing;
    kvtc_status st = batch_checks("kvtc_entropy_decode_batch", e, jobs_dev, n_jobs, max_tokens, records_base_dev, coded_base_dev, &nothing);
    if (st != KVTC_OK || nothing) return st;
    EntropyArgs a = base_args(e);
    a.jobs = jobs_dev;
    a.n_jobs = n_jobs;
    a.records = static_cast<const uint8_t*>(records_base_dev);
    a.records_cap = records_cap;
    a.coded = static_cast<uint8_t*>(const_cast<void*>(coded_base_dev));
    a.coded_total = coded_bytes;
    return run_decode("kvtc_entropy_decode_batch", e, a, n_jobs, max_tokens, static_cast<hipStream_t>(stream));
}

}  // extern "C"
