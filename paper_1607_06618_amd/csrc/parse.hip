// FASTA / FASTQ text to CSR reads, on the device (the input formats of
// App. B; the paper's parser stage feeds the counting pipeline, Sec. 2.3.1).
//
// The text is cut into lines by a newline compaction; every later step works
// on lines, never on the text again, except for the copy of the sequence
// bytes:
//   1. newlines per byte tile (64 or 16 KB in rounds of 4 KB, 16 B per lane);
//   2. one workgroup scans the tile counts (line count, final line);
//   3. each newline writes a line word: its position (40 bits), whether the
//      byte before it is '\r' (bit 40), and the first byte of the next line
//      (bits 48-55);
//   4. per line tile: sequence bytes kept and reads started, from the format
//      (FASTQ: line index mod 4; FASTA: a '>' first byte), plus the format
//      checks;
//   5. one workgroup scans the tile sums;
//   6. per line: the offset of its kept bytes, and the read offsets;
//   7. per line tile, the kept bytes are gathered into aligned 16-byte
//      chunks of the output.
#include "../../include/gerbil.h"
#include "common.h"
#include "internal.h"

namespace gerbil {
namespace {

constexpr uint32_t kPB = 256;                        // threads of the tile kernels
constexpr uint32_t kChunk = 16;                      // text bytes per lane and round
// Rounds of a byte tile, a multiple of 4 (four share one scan): tiles of 64 KB,
// or of 16 KB for texts of fewer than eight of those per CU (23 MB: newlines
// written in 31 us from large tiles, 23 from small ones).
constexpr uint32_t kRoundsBig = 16, kRoundsSmall = 4;
constexpr uint64_t tile_bytes(uint32_t rounds) { return (uint64_t)kPB * kChunk * rounds; }
constexpr uint64_t kByteBigFrom = 2048 * tile_bytes(kRoundsBig);
__host__ __device__ inline uint32_t rounds_of(uint64_t n) { return n >= kByteBigFrom ? kRoundsBig : kRoundsSmall; }
constexpr uint32_t kLinesPer = 8;                    // lines per lane
constexpr uint64_t kLineTile = (uint64_t)kPB * kLinesPer;          // 2048 lines
constexpr uint32_t kScanBlock = 1024;                // threads of the one-workgroup scans
constexpr uint64_t kPosMask = (1ull << 40) - 1;

constexpr uint32_t kMaxTileGridParse = 8192;

struct Ws {
    uint64_t* tile_nl;     // [n_btiles + 1]
    uint64_t* line;        // [lines_cap] line words
    uint64_t* line_off;    // [lines_cap]
    uint64_t* lt_kept;     // [n_ltiles + 1]
    uint64_t* lt_reads;    // [n_ltiles + 1]
};

__host__ __device__ inline uint64_t n_btiles_of(uint64_t n) { return (n + tile_bytes(rounds_of(n)) - 1) / tile_bytes(rounds_of(n)); }
__host__ __device__ inline uint64_t n_ltiles_of(uint64_t lines) { return (lines + kLineTile - 1) / kLineTile; }

// Byte tiles a workspace for n bytes has room for: never fewer for a longer text.
inline uint64_t btiles_room(uint64_t n) {
    const uint64_t t = n_btiles_of(n), most_small = n_btiles_of(kByteBigFrom - 1);
    return n < kByteBigFrom || t > most_small ? t : most_small;
}

inline uint64_t ws_layout(uint64_t n, uint64_t lines_cap, uint8_t* base, Ws* w) {
    uint64_t off = 0;
    auto take = [&](uint64_t bytes) {
        uint8_t* p = base ? base + off : nullptr;
        off += align256(bytes);
        return (uint64_t*)p;
    };
    Ws x;
    x.tile_nl = take(8 * (btiles_room(n) + 1));
    x.line = take(8 * (lines_cap + 1));
    x.line_off = take(8 * (lines_cap + 1));
    x.lt_kept = take(8 * (n_ltiles_of(lines_cap) + 1));
    x.lt_reads = take(8 * (n_ltiles_of(lines_cap) + 1));
    if (w) *w = x;
    return off;
}

// 0x80 in every byte of x that equals 0x0A, else 0 (exact, no carries).
__device__ __forceinline__ uint32_t nl_bytes(uint32_t x) {
    const uint32_t y = x ^ 0x0A0A0A0Au;
    return ~(((y & 0x7F7F7F7Fu) + 0x7F7F7F7Fu) | y | 0x7F7F7F7Fu);
}

// The 16 bytes of chunk c (c * 16 .. c * 16 + 15 of the text) as four words;
// bytes outside [0, n) read as 0. Whole chunks use one 16-byte load when the
// text is 16-byte aligned, else byte loads.
__device__ __forceinline__ void load_chunk(const uint8_t* __restrict__ text, uint64_t n, uint64_t c, bool aligned,
                                           uint32_t (&w)[4]) {
    const uint64_t b = c * kChunk;
    if (aligned && b + kChunk <= n) {
        const uint4 v = *(const uint4*)(text + b);
        w[0] = v.x; w[1] = v.y; w[2] = v.z; w[3] = v.w;
        return;
    }
#pragma unroll
    for (int i = 0; i < 4; i++) {
        uint32_t x = 0;
#pragma unroll
        for (int j = 0; j < 4; j++) {
            const uint64_t p = b + 4 * i + j;
            x |= (uint32_t)(p < n ? text[p] : 0u) << (8 * j);
        }
        w[i] = x;
    }
}

// Newlines of a chunk, one bit a byte.
__device__ __forceinline__ uint32_t chunk_mask(const uint32_t (&w)[4]) {
    const uint32_t lo = __builtin_amdgcn_udot4(nl_bytes(w[1]) >> 7, 0x80402010u, __builtin_amdgcn_udot4(nl_bytes(w[0]) >> 7, 0x08040201u, 0u, false), false);
    const uint32_t hi = __builtin_amdgcn_udot4(nl_bytes(w[3]) >> 7, 0x80402010u, __builtin_amdgcn_udot4(nl_bytes(w[2]) >> 7, 0x08040201u, 0u, false), false);
    return lo | hi << 8;
}

__device__ __forceinline__ uint32_t chunk_newlines(const uint32_t (&w)[4]) {
    uint32_t c = 0;
#pragma unroll
    for (int i = 0; i < 4; i++) c += __builtin_popcount(nl_bytes(w[i]));
    return c;
}

template <typename T>
__device__ __forceinline__ T wave_incl_scan(T v) {
    const uint32_t lane = __lane_id();
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const T y = __shfl_up(v, off);
        if (lane >= (uint32_t)off) v += y;
    }
    return v;
}

// Exclusive scan of one uint64 per thread over the block; wsum holds
// blockDim/64 + 1 entries.
__device__ __forceinline__ uint64_t block_scan64(uint64_t v, uint64_t* wsum, uint64_t& total) {
    const uint32_t lane = __lane_id(), wave = threadIdx.x >> 6, nw = blockDim.x >> 6;
    const uint64_t incl = wave_incl_scan<uint64_t>(v);
    if (lane == 63) wsum[wave] = incl;
    __syncthreads();
    if (wave == 0) {
        const uint64_t s = lane < nw ? wsum[lane] : 0ull;
        const uint64_t si = wave_incl_scan<uint64_t>(s);
        if (lane < nw) wsum[lane] = si - s;
        if (lane == 63) wsum[nw] = si;
    }
    __syncthreads();
    const uint64_t r = wsum[wave] + incl - v;
    total = wsum[nw];
    __syncthreads();   // wsum is reused by the next call
    return r;
}

// In-place exclusive scan of v[0..n) by one workgroup of kScanBlock threads;
// returns the total to every thread. Eight consecutive values a thread at a
// time, all in flight (29 000 tile counts: 28 us; a run of 29 per thread, one
// load after the other, took 66).
__device__ uint64_t wg_scan_inplace(uint64_t* v, uint64_t n, uint64_t* wsum) {
    constexpr uint32_t kPer = 8;
    uint64_t before = 0;
    for (uint64_t i0 = 0; i0 < n; i0 += kPer * kScanBlock) {
        const uint64_t i = i0 + kPer * threadIdx.x;
        uint64_t x[kPer], s = 0;
#pragma unroll
        for (uint32_t j = 0; j < kPer; j++) x[j] = i + j < n ? v[i + j] : 0ull;
#pragma unroll
        for (uint32_t j = 0; j < kPer; j++) s += x[j];
        uint64_t total;
        uint64_t run = before + block_scan64(s, wsum, total);
#pragma unroll
        for (uint32_t j = 0; j < kPer; j++) {
            if (i + j < n) v[i + j] = run;
            run += x[j];
        }
        before += total;
    }
    return before;
}

// --------------------------------------------------------------- kernels

__global__ void k_parse_init(const uint8_t* __restrict__ text, uint64_t n, uint32_t format,
                             uint64_t* __restrict__ offsets, gerbil_parsed* out) {
    if (threadIdx.x != 0 || blockIdx.x != 0) return;
    uint32_t fmt = format, status = 0;
    if (fmt == GERBIL_FORMAT_DETECT && n) {
        const uint8_t c = text[0];
        fmt = c == '@' ? GERBIL_FORMAT_FASTQ : c == '>' ? GERBIL_FORMAT_FASTA : 0u;
        if (!fmt) status = GERBIL_PARSE_EFORMAT;
    }
    offsets[0] = 0;   // (an empty text of no format has no later step)
    out->n_reads = 0;
    out->n_bytes = 0;
    out->n_lines = 0;
    out->status = status;
    out->format = fmt;
}

// 1. newlines per byte tile
template <uint32_t kRounds>
__global__ void __launch_bounds__(kPB) k_nl_count(const uint8_t* __restrict__ text, uint64_t n, bool aligned,
                                                  uint64_t* __restrict__ tile_nl) {
    __shared__ uint64_t wsum[kPB / 64 + 1];
    const uint64_t nt = n_btiles_of(n);
    for (uint64_t t = blockIdx.x; t < nt; t += gridDim.x) {
        uint32_t c = 0;
#pragma unroll
        for (uint32_t r = 0; r < kRounds; r++) {
            uint32_t w[4];
            load_chunk(text, n, (t * kRounds + r) * kPB + threadIdx.x, aligned, w);
            c += chunk_newlines(w);
        }
        uint64_t total;
        (void)block_scan64(c, wsum, total);
        if (threadIdx.x == 0) tile_nl[t] = total;
    }
}

// 2. scan of the tile counts; the final line without a newline
__global__ void __launch_bounds__(kScanBlock) k_nl_scan(const uint8_t* __restrict__ text, uint64_t n,
                                                        uint64_t* __restrict__ tile_nl, uint64_t* __restrict__ line,
                                                        uint64_t lines_cap, gerbil_parsed* out) {
    __shared__ uint64_t wsum[kScanBlock / 64 + 1];
    const uint64_t nt = n_btiles_of(n);
    const uint64_t nl = wg_scan_inplace(tile_nl, nt, wsum);
    if (threadIdx.x != 0) return;
    const bool open_end = n > 0 && text[n - 1] != '\n';
    const uint64_t lines = nl + (open_end ? 1 : 0);
    out->n_lines = lines;
    if (lines > lines_cap) {
        out->status |= GERBIL_PARSE_ELINECAP;
        return;
    }
    if (open_end) line[nl] = n | ((uint64_t)(text[n - 1] == '\r') << 40);   // no next line: first byte 0
}

// 3. the line words. Four rounds share one block scan: their newline counts
// (at most 16 per lane and round, at most 4096 per round) ride in 16-bit
// fields of two words. The bytes around a newline come from the lane's chunk
// or its neighbours'; those of the wave's first and last lane are loaded with
// the chunks, so that nothing is loaded while newlines are written. 1.9 GB of
// text in 0.49 ms (a load per newline at a chunk's edge and a loop per word
// of four bytes: 1.04 ms).
__device__ __forceinline__ uint32_t chunk_byte(const uint32_t (&w)[4], uint32_t idx) {
    const uint32_t a = idx & 4 ? w[1] : w[0], b = idx & 4 ? w[3] : w[2];
    return ((idx & 8 ? b : a) >> (8 * (idx & 3))) & 0xFFu;
}

template <uint32_t kRounds>
__global__ void __launch_bounds__(kPB) k_nl_write(const uint8_t* __restrict__ text, uint64_t n, bool aligned,
                                                  const uint64_t* __restrict__ tile_nl, uint64_t* __restrict__ line,
                                                  uint64_t lines_cap) {
    __shared__ uint2 wsum[2][kPB / 64];
    const uint64_t nt = n_btiles_of(n);
    const uint32_t lane = __lane_id(), wave = threadIdx.x >> 6;
    // byte before the first lane's chunk, after the last lane's
    auto edge_of = [&](uint64_t c) -> uint32_t {
        const uint64_t p = lane == 0 ? c * kChunk - 1 : c * kChunk + kChunk;   // (wraps before the text: not loaded)
        return (lane == 0 || lane == 63) && p < n ? (uint32_t)text[p] : 0u;
    };
    for (uint64_t t = blockIdx.x; t < nt; t += gridDim.x) {
        uint64_t base = tile_nl[t];
        uint32_t w[4][4], nx[4][4];   // this group's chunks, the next group's (loaded ahead)
        uint32_t edge[4], edge_nx[4];
#pragma unroll
        for (uint32_t rr = 0; rr < 4; rr++) {
            const uint64_t c = (t * kRounds + rr) * kPB + threadIdx.x;
            load_chunk(text, n, c, aligned, nx[rr]);
            edge_nx[rr] = edge_of(c);
        }
#pragma unroll 1
        for (uint32_t g = 0; g < kRounds; g += 4) {
            uint32_t m[4];
#pragma unroll
            for (uint32_t rr = 0; rr < 4; rr++) {
#pragma unroll
                for (int i = 0; i < 4; i++) w[rr][i] = nx[rr][i];
                edge[rr] = edge_nx[rr];
                m[rr] = chunk_mask(w[rr]);
            }
            if (g + 4 < kRounds) {
#pragma unroll
                for (uint32_t rr = 0; rr < 4; rr++) {
                    const uint64_t c = (t * kRounds + g + 4 + rr) * kPB + threadIdx.x;
                    load_chunk(text, n, c, aligned, nx[rr]);
                    edge_nx[rr] = edge_of(c);
                }
            }
            const uint2 own = make_uint2((uint32_t)__popc(m[0]) | (uint32_t)__popc(m[1]) << 16,
                                         (uint32_t)__popc(m[2]) | (uint32_t)__popc(m[3]) << 16);
            const uint2 incl = make_uint2(wave_incl_sum(own.x), wave_incl_sum(own.y));
            uint2* ws = wsum[(g >> 2) & 1];   // (two in turn: one barrier a group)
            if (lane == 63) ws[wave] = incl;
            __syncthreads();
            uint2 excl = make_uint2(incl.x - own.x, incl.y - own.y), total = make_uint2(0, 0);
#pragma unroll
            for (uint32_t i = 0; i < kPB / 64; i++) {
                const uint2 s = ws[i];
                excl.x += i < wave ? s.x : 0u;
                excl.y += i < wave ? s.y : 0u;
                total.x += s.x;
                total.y += s.y;
            }
#pragma unroll
            for (uint32_t rr = 0; rr < 4; rr++) {
                const uint64_t c = (t * kRounds + g + rr) * kPB + threadIdx.x;
                uint64_t idx = base + (((rr & 2 ? excl.y : excl.x) >> (16 * (rr & 1))) & 0xFFFFu);
                // (by every lane: a lane that is not running gives nothing)
                const uint32_t below = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)w[rr][3], 0x138, 0xf, 0xf, false);   // wave shifts by one lane
                const uint32_t above = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)w[rr][0], 0x130, 0xf, 0xf, false);
                const uint32_t prev = lane == 0 ? edge[rr] : below >> 24, next = lane == 63 ? edge[rr] : above & 0xFFu;
                for (uint32_t left = m[rr]; left; left &= left - 1) {
                    const uint32_t j = (uint32_t)__builtin_ctz(left);   // byte of the chunk
                    const uint64_t p = c * kChunk + j;                  // < n: bytes past n read as 0
                    const uint32_t before = j ? chunk_byte(w[rr], j - 1) : prev;
                    const uint32_t after = j < kChunk - 1 ? chunk_byte(w[rr], j + 1) : next;
                    if (idx < lines_cap) line[idx] = p | ((uint64_t)(before == '\r') << 40) | ((uint64_t)after << 48);
                    idx++;
                }
                base += ((rr & 2 ? total.y : total.x) >> (16 * (rr & 1))) & 0xFFFFu;
            }
        }
        __syncthreads();   // the sums of the last group are read
    }
}

struct LineInfo {
    uint64_t kept;    // sequence bytes of the line
    uint32_t starts;  // 1 if the line starts a read
    uint32_t err;     // GERBIL_PARSE_* bits found at this line
};

__device__ __forceinline__ uint64_t line_start(const uint64_t* line, uint64_t i) {
    return i ? (line[i - 1] & kPosMask) + 1 : 0ull;
}
__device__ __forceinline__ uint64_t line_body(const uint64_t* line, uint64_t i) {
    const uint64_t w = line[i];
    const uint64_t e = w & kPosMask, s = line_start(line, i);
    return e - s - ((w >> 40) & 1ull);
}
__device__ __forceinline__ uint32_t line_first(const uint64_t* line, uint64_t i, uint32_t first0) {
    return i ? (uint32_t)(line[i - 1] >> 48) & 0xFFu : first0;
}

__device__ __forceinline__ LineInfo classify(const uint64_t* line, uint64_t i, uint64_t lines, uint32_t fmt,
                                             uint32_t first0) {
    LineInfo x{0, 0, 0};
    if (fmt == GERBIL_FORMAT_FASTQ) {
        if ((i & 3) != 1) return x;
        x.starts = 1;
        x.kept = line_body(line, i);
        // an empty header line has the newline itself as "first byte"
        if (line_first(line, i - 1, first0) != '@') x.err |= GERBIL_PARSE_EHEADER;
        if (i + 1 < lines && line_first(line, i + 1, first0) != '+') x.err |= GERBIL_PARSE_EPLUS;
        if (i + 2 < lines && line_body(line, i + 2) != x.kept) x.err |= GERBIL_PARSE_EQUAL;
    } else {
        const bool empty = (line[i] & kPosMask) == line_start(line, i);
        if (!empty && line_first(line, i, first0) == '>') {
            x.starts = 1;
        } else {
            x.kept = line_body(line, i);
        }
    }
    return x;
}

__device__ __forceinline__ bool lines_usable(const gerbil_parsed* out, uint64_t& lines, uint32_t& fmt) {
    const uint32_t st = out->status;
    fmt = out->format;
    lines = out->n_lines;
    return fmt != 0 && !(st & (GERBIL_PARSE_ELINECAP | GERBIL_PARSE_EFORMAT));
}

// 4. kept bytes and reads per line tile; format checks
__global__ void __launch_bounds__(kPB) k_line_sums(const uint8_t* __restrict__ text, const uint64_t* __restrict__ line,
                                                   uint64_t* __restrict__ lt_kept, uint64_t* __restrict__ lt_reads,
                                                   gerbil_parsed* out) {
    __shared__ uint64_t wsum[kPB / 64 + 1];
    __shared__ uint32_t err_s;
    uint64_t lines;
    uint32_t fmt;
    if (!lines_usable(out, lines, fmt)) return;
    const uint32_t first0 = lines ? text[0] : 0u;
    const uint64_t nt = n_ltiles_of(lines);
    for (uint64_t t = blockIdx.x; t < nt; t += gridDim.x) {
        if (threadIdx.x == 0) err_s = 0;
        uint64_t kept = 0, reads = 0;
        uint32_t err = 0;
        const uint64_t i0 = t * kLineTile + (uint64_t)threadIdx.x * kLinesPer;
        for (uint32_t j = 0; j < kLinesPer; j++) {
            const uint64_t i = i0 + j;
            if (i >= lines) break;
            const LineInfo x = classify(line, i, lines, fmt, first0);
            kept += x.kept;
            reads += x.starts;
            err |= x.err;
        }
        uint64_t tk, tr;
        (void)block_scan64(kept, wsum, tk);
        (void)block_scan64(reads, wsum, tr);
        if (err) atomicOr(&err_s, err);
        __syncthreads();
        if (threadIdx.x == 0) {
            lt_kept[t] = tk;
            lt_reads[t] = tr;
            if (err_s) set_status(&out->status, err_s);
        }
    }
}

// 5. scan of the line tile sums; totals and capacity checks
__global__ void __launch_bounds__(kScanBlock) k_line_scan(uint64_t* __restrict__ lt_kept, uint64_t* __restrict__ lt_reads,
                                                          uint64_t* __restrict__ offsets, uint64_t seq_cap,
                                                          uint64_t reads_cap, gerbil_parsed* out) {
    __shared__ uint64_t wsum[kScanBlock / 64 + 1];
    uint64_t lines;
    uint32_t fmt;
    if (!lines_usable(out, lines, fmt)) return;
    const uint64_t nt = n_ltiles_of(lines);
    const uint64_t bytes = wg_scan_inplace(lt_kept, nt, wsum);
    const uint64_t reads = wg_scan_inplace(lt_reads, nt, wsum);
    if (threadIdx.x != 0) return;
    uint32_t st = 0;
    if (fmt == GERBIL_FORMAT_FASTQ && (lines & 3)) st |= GERBIL_PARSE_ELINES;
    if (fmt == GERBIL_FORMAT_FASTA && reads == 0 && bytes > 0) st |= GERBIL_PARSE_EORPHAN;
    if (bytes > seq_cap) st |= GERBIL_PARSE_EBYTES;
    if (reads > reads_cap) st |= GERBIL_PARSE_EREADS;
    else offsets[reads] = bytes;
    out->n_bytes = bytes;
    out->n_reads = reads;
    if (st) set_status(&out->status, st);
}

// 6. line offsets and read offsets
__global__ void __launch_bounds__(kPB) k_line_apply(const uint8_t* __restrict__ text, const uint64_t* __restrict__ line,
                                                    const uint64_t* __restrict__ lt_kept,
                                                    const uint64_t* __restrict__ lt_reads,
                                                    uint64_t* __restrict__ line_off, uint64_t* __restrict__ offsets,
                                                    uint64_t reads_cap, gerbil_parsed* out) {
    __shared__ uint64_t wsum[kPB / 64 + 1];
    uint64_t lines;
    uint32_t fmt;
    if (!lines_usable(out, lines, fmt)) return;
    const uint32_t first0 = lines ? text[0] : 0u;
    const uint64_t nt = n_ltiles_of(lines);
    for (uint64_t t = blockIdx.x; t < nt; t += gridDim.x) {
        const uint64_t i0 = t * kLineTile + (uint64_t)threadIdx.x * kLinesPer;
        LineInfo x[kLinesPer];
        uint64_t kept = 0, reads = 0;
#pragma unroll
        for (uint32_t j = 0; j < kLinesPer; j++) {
            x[j] = i0 + j < lines ? classify(line, i0 + j, lines, fmt, first0) : LineInfo{0, 0, 0};
            kept += x[j].kept;
            reads += x[j].starts;
        }
        uint64_t tk, tr;
        uint64_t ko = lt_kept[t] + block_scan64(kept, wsum, tk);
        uint64_t ro = lt_reads[t] + block_scan64(reads, wsum, tr);
        bool orphan = false;
#pragma unroll
        for (uint32_t j = 0; j < kLinesPer; j++) {
            if (i0 + j >= lines) break;
            line_off[i0 + j] = ko;
            if (x[j].starts) {
                if (ro < reads_cap) offsets[ro] = ko;
                orphan |= fmt == GERBIL_FORMAT_FASTA && ro == 0 && ko != 0;
                ro++;
            }
            ko += x[j].kept;
        }
        if (orphan) set_status(&out->status, GERBIL_PARSE_EORPHAN);
    }
}

// 7. per line tile: the tile's lines own the output range [O0, O1); each
// lane fills aligned 16-byte chunks of it (two at a time, so that their loads
// overlap). The line holding a chunk's first byte is found by binary search
// in the tile's offsets, which sit in LDS with the line starts. A chunk's part
// of a line is two aligned 16-byte loads and a byte funnel shift; one that
// spans two lines that have bytes is put together from both (a chunk in nine at 150
// bytes a line, so that nearly every wave has some). One of more lines, or at
// the ends of the text, of the range or of seq_cap is gathered and written
// byte by byte (its bytes outside the range belong to neighbouring tiles).
// 0.9 GB of 150-byte reads in 0.75 ms, where gathering every chunk of two
// lines byte by byte took 1.36 ms.
constexpr uint32_t kCopyBatch = 2;
// Lines per copy tile: 1024 (20 KB of LDS, seven workgroups per CU), or 256
// where those would be fewer than some ten per CU (14 000 lines of a 0.5 MB text:
// 128 us a call with the large tiles, 90 us with the small ones).
constexpr uint32_t kCopyTileBig = 4 * kPB, kCopyTileSmall = kPB;
constexpr uint64_t kCopyBigFrom = 8192ull * kCopyTileBig;   // of the capacity for lines, some three times their number
// Output bytes of a tile that one workgroup copies at a time, about: lines
// longer than 128 bytes on average are shared out over several, or few long
// lines would leave the chip idle (500 MB in lines of 10 KB: 1.2 ms with a
// workgroup per 512 lines, 0.51 ms with slices).
constexpr uint64_t kCopySlice = 128 * 1024;

// bytes [o, o + 16) of the 32 bytes a, b (o < 16)
__device__ __forceinline__ uint4 funnel16(const uint4 a, const uint4 b, uint32_t o) {
    const uint32_t r = o & 3;
    uint32_t e0, e1, e2, e3, e4;
    switch (o >> 2) {
        case 0: e0 = a.x; e1 = a.y; e2 = a.z; e3 = a.w; e4 = b.x; break;
        case 1: e0 = a.y; e1 = a.z; e2 = a.w; e3 = b.x; e4 = b.y; break;
        case 2: e0 = a.z; e1 = a.w; e2 = b.x; e3 = b.y; e4 = b.z; break;
        default: e0 = a.w; e1 = b.x; e2 = b.y; e3 = b.z; e4 = b.w; break;
    }
    return make_uint4(__builtin_amdgcn_alignbyte(e1, e0, r), __builtin_amdgcn_alignbyte(e2, e1, r),
                      __builtin_amdgcn_alignbyte(e3, e2, r), __builtin_amdgcn_alignbyte(e4, e3, r));
}

// First line whose offset in s exceeds q, less one (s[0] <= q).
template <typename T>
__device__ __forceinline__ uint32_t line_of(const T* s, uint32_t cnt, T q) {
    uint32_t lo = 0, hi = cnt;
    while (hi - lo > 1) {
        const uint32_t mid = (lo + hi) >> 1;
        if (s[mid] <= q) lo = mid; else hi = mid;
    }
    return lo;
}

template <uint32_t kCopyTile>
__global__ void __launch_bounds__(kPB, 7) k_line_copy(const uint8_t* __restrict__ text, uint64_t n,
                                                   const uint64_t* __restrict__ line,
                                                   const uint64_t* __restrict__ line_off, uint8_t* __restrict__ seq,
                                                   uint64_t seq_cap, gerbil_parsed* out) {
    __shared__ uint64_t s_off[kCopyTile + 1];
    __shared__ uint64_t s_start[kCopyTile];
    __shared__ uint32_t s_rel[kCopyTile + 1];   // offsets from the tile's first
    uint64_t lines;
    uint32_t fmt;
    if (!lines_usable(out, lines, fmt)) return;
    const uint64_t total = out->n_bytes;
    const uint64_t ms = ((uintptr_t)seq) & 15;   // chunks are aligned in the address space
    const uintptr_t t_lo = (uintptr_t)text, t_hi = (uintptr_t)text + n;
    const uint64_t nt = (lines + kCopyTile - 1) / kCopyTile;
    const uint32_t S = nt ? (uint32_t)(total / nt / kCopySlice) + 1u : 1u;   // slices of a tile
    for (uint64_t unit = blockIdx.x; unit < nt * S; unit += gridDim.x) {
        const uint64_t t = S == 1 ? unit : unit / S;
        const uint32_t slice = (uint32_t)(unit - t * S), step = S * kPB * kCopyBatch;
        const uint64_t i0 = t * kCopyTile;
        const uint32_t cnt = (uint32_t)(lines - i0 < kCopyTile ? lines - i0 : kCopyTile);
        // the tables: every load issued before any is used
        uint64_t o_v[kCopyTile / kPB + 1], s_v[kCopyTile / kPB];
#pragma unroll
        for (uint32_t r = 0; r <= kCopyTile / kPB; r++) {
            const uint32_t j = threadIdx.x + r * kPB;
            const uint64_t i = i0 + j;
            o_v[r] = j <= cnt ? (i < lines ? line_off[i] : total) : 0ull;
            if (r < kCopyTile / kPB) s_v[r] = j < cnt && i ? line[i - 1] : 0ull;
        }
#pragma unroll
        for (uint32_t r = 0; r <= kCopyTile / kPB; r++) {
            const uint32_t j = threadIdx.x + r * kPB;
            if (j <= cnt) s_off[j] = o_v[r];
            if (r < kCopyTile / kPB && j < cnt) s_start[j] = i0 + j ? (s_v[r] & kPosMask) + 1 : 0ull;
        }
        __syncthreads();
        const uint64_t O0 = s_off[0], O1 = s_off[cnt];
        const bool narrow = O1 - O0 < 1ull << 32;
#pragma unroll
        for (uint32_t r = 0; r <= kCopyTile / kPB; r++) {
            const uint32_t j = threadIdx.x + r * kPB;
            if (j <= cnt) s_rel[j] = (uint32_t)(o_v[r] - O0);
        }
        __syncthreads();
        if (O1 > O0) {
            const uint64_t c0 = (O0 + ms) / kChunk, c1 = (O1 + ms + kChunk - 1) / kChunk;
            for (uint64_t cb = c0 + (slice * kPB * kCopyBatch + threadIdx.x); cb < c1; cb += step) {
                uint4 v[kCopyBatch];
                bool fast[kCopyBatch];
#pragma unroll
                for (uint32_t b = 0; b < kCopyBatch; b++) {
                    const uint64_t c = cb + (uint64_t)b * kPB;
                    fast[b] = false;
                    v[b] = make_uint4(0u, 0u, 0u, 0u);
                    if (c >= c1) continue;
                    // byte k of the chunk is output byte a0 + k - ms; it belongs to this
                    // tile iff O0 + ms <= a0 + k < O1 + ms (never negative: no wrap)
                    const uint64_t a0 = c * kChunk;
                    const uint64_t qs = (a0 > O0 + ms ? a0 : O0 + ms) - ms;
                    // last line whose offset is <= qs: the line holding byte qs
                    uint32_t j = narrow ? line_of<uint32_t>(s_rel, cnt, (uint32_t)(qs - O0)) : line_of<uint64_t>(s_off, cnt, qs);
                    uint64_t lend = s_off[j + 1];
                    const bool whole = a0 >= O0 + ms && a0 + kChunk <= O1 + ms && a0 + kChunk <= seq_cap + ms;
                    if (whole) {
                        const uint64_t q0 = a0 - ms;
                        // the 16 bytes from the one that output byte q0 would be in line j
                        const uintptr_t src = (uintptr_t)text + s_start[j] + (q0 - s_off[j]), A = src & ~(uintptr_t)15;
                        bool ok = A >= t_lo && A + 32 <= t_hi;
                        uintptr_t src2 = src, A2 = A;
                        const bool two = q0 + kChunk > lend;
                        if (two) {   // the next line that has bytes
                            uint32_t j2 = j + 1;
                            while (s_off[j2 + 1] == lend) j2++;   // (byte lend is in the range: one has it)
                            ok = ok && q0 + kChunk <= s_off[j2 + 1];
                            src2 = (uintptr_t)text + s_start[j2] - (uintptr_t)(lend - q0);
                            A2 = src2 & ~(uintptr_t)15;
                            ok = ok && A2 >= t_lo && A2 + 32 <= t_hi;
                        }
                        if (ok) {
                            const uint4 x = *(const uint4*)A, y = *(const uint4*)(A + 16);
                            v[b] = funnel16(x, y, (uint32_t)(src & 15));
                            if (two) {
                                const uint4 x2 = *(const uint4*)A2, y2 = *(const uint4*)(A2 + 16);
                                const uint4 z = funnel16(x2, y2, (uint32_t)(src2 & 15));
                                const uint32_t cut = (uint32_t)(lend - q0);   // bytes of the first line, 1 .. 15
                                auto join = [&](uint32_t e, uint32_t f, uint32_t at) {
                                    const uint32_t keep = cut >= at + 4 ? 0xFFFFFFFFu : cut <= at ? 0u : 0xFFFFFFFFu >> (32 - 8 * (cut - at));
                                    return (e & keep) | (f & ~keep);
                                };
                                v[b] = make_uint4(join(v[b].x, z.x, 0), join(v[b].y, z.y, 4), join(v[b].z, z.z, 8), join(v[b].w, z.w, 12));
                            }
                            fast[b] = true;
                            continue;
                        }
                    }
                    uint32_t w[4] = {0u, 0u, 0u, 0u};
#pragma unroll
                    for (uint32_t k = 0; k < kChunk; k++) {
                        if (a0 + k >= O0 + ms && a0 + k < O1 + ms) {
                            const uint64_t q = a0 + k - ms;
                            while (q >= lend) lend = s_off[++j + 1];
                            w[k >> 2] |= (uint32_t)text[s_start[j] + (q - s_off[j])] << (8 * (k & 3));
                        }
                    }
                    v[b] = make_uint4(w[0], w[1], w[2], w[3]);
                }
#pragma unroll
                for (uint32_t b = 0; b < kCopyBatch; b++) {
                    const uint64_t c = cb + (uint64_t)b * kPB;
                    if (c >= c1) continue;
                    const uint64_t a0 = c * kChunk;
                    if (fast[b] || (a0 >= O0 + ms && a0 + kChunk <= O1 + ms && a0 + kChunk <= seq_cap + ms)) {
                        *(uint4*)(seq + (a0 - ms)) = v[b];
                    } else {
                        const uint32_t w[4] = {v[b].x, v[b].y, v[b].z, v[b].w};
#pragma unroll
                        for (uint32_t k = 0; k < kChunk; k++) {
                            if (a0 + k >= O0 + ms && a0 + k < O1 + ms && a0 + k < seq_cap + ms)
                                seq[a0 + k - ms] = (uint8_t)(w[k >> 2] >> (8 * (k & 3)));
                        }
                    }
                }
            }
        }
        __syncthreads();   // the LDS tables are refilled for the next tile
    }
}

uint32_t grid_of(uint64_t tiles) {
    return (uint32_t)(tiles == 0 ? 1 : tiles < kMaxTileGridParse ? tiles : kMaxTileGridParse);
}

}  // namespace
}  // namespace gerbil

using namespace gerbil;

extern "C" {

int32_t gerbil_parse_workspace(uint64_t n, uint64_t lines_cap, uint64_t* bytes) {
    if (!bytes || n >= (1ull << 40) || lines_cap > n + 1) return GERBIL_EINVAL;
    *bytes = ws_layout(n, lines_cap, nullptr, nullptr);
    return GERBIL_OK;
}

int32_t gerbil_parse(const uint8_t* text, uint64_t n, uint32_t format, void* ws, uint64_t ws_bytes,
                     uint64_t lines_cap, uint8_t* seq, uint64_t seq_cap, uint64_t* offsets, uint64_t reads_cap,
                     gerbil_parsed* out, hipStream_t stream) {
    if (!out || !offsets || !ws || (n && !text) || (seq_cap && !seq)) return GERBIL_EINVAL;
    if (format > GERBIL_FORMAT_FASTA || n >= (1ull << 40) || lines_cap > n + 1) return GERBIL_EINVAL;
    if (((uintptr_t)ws) & 255) return GERBIL_EINVAL;
    Ws w;
    if (ws_bytes < ws_layout(n, lines_cap, (uint8_t*)ws, &w)) return GERBIL_EINVAL;
    const bool aligned = (((uintptr_t)text) & 15) == 0;
    const uint64_t bt = n_btiles_of(n), lt = n_ltiles_of(lines_cap);
    hipLaunchKernelGGL(k_parse_init, dim3(1), dim3(64), 0, stream, text, n, format, offsets, out);
    const bool big = rounds_of(n) == kRoundsBig;
    hipLaunchKernelGGL(big ? k_nl_count<kRoundsBig> : k_nl_count<kRoundsSmall>, dim3(grid_of(bt)), dim3(kPB), 0, stream, text,
                       n, aligned, w.tile_nl);
    hipLaunchKernelGGL(k_nl_scan, dim3(1), dim3(kScanBlock), 0, stream, text, n, w.tile_nl, w.line, lines_cap, out);
    hipLaunchKernelGGL(big ? k_nl_write<kRoundsBig> : k_nl_write<kRoundsSmall>, dim3(grid_of(bt)), dim3(kPB), 0, stream, text,
                       n, aligned, w.tile_nl, w.line, lines_cap);
    hipLaunchKernelGGL(k_line_sums, dim3(grid_of(lt)), dim3(kPB), 0, stream, text, w.line, w.lt_kept, w.lt_reads, out);
    hipLaunchKernelGGL(k_line_scan, dim3(1), dim3(kScanBlock), 0, stream, w.lt_kept, w.lt_reads, offsets, seq_cap,
                       reads_cap, out);
    hipLaunchKernelGGL(k_line_apply, dim3(grid_of(lt)), dim3(kPB), 0, stream, text, w.line, w.lt_kept, w.lt_reads,
                       w.line_off, offsets, reads_cap, out);
    if (lines_cap >= kCopyBigFrom)
        hipLaunchKernelGGL(k_line_copy<kCopyTileBig>, dim3(grid_of((lines_cap + kCopyTileBig - 1) / kCopyTileBig + n / kCopySlice)),
                           dim3(kPB), 0, stream, text, n, w.line, w.line_off, seq, seq_cap, out);
    else
        hipLaunchKernelGGL(k_line_copy<kCopyTileSmall>, dim3(grid_of((lines_cap + kCopyTileSmall - 1) / kCopyTileSmall + n / kCopySlice)),
                           dim3(kPB), 0, stream, text, n, w.line, w.line_off, seq, seq_cap, out);
    return hipGetLastError() == hipSuccess ? GERBIL_OK : GERBIL_EDEVICE;
}

}  // extern "C"
