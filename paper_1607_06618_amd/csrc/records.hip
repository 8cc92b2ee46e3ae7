// Binary output records of the emitted pairs (App. C): the counter -- one
// byte when it is below 255, else the byte 0xFF and the count as a
// big-endian 32-bit word -- then the k-mer, four bases per byte with the first
// base in the top bits and the last byte padded with zero bits.
//
// Record sizes take two values (1 + kb or 5 + kb bytes, kb = ceil(k/4)), so
// the offset of record i is i (1 + kb) + 4 x (large counters before i): an
// exclusive scan of one flag per pair. Three launches: flags per tile, a
// scan of the tile totals, then per tile and round the records are built in
// LDS, a word of the key at a time, and the round's byte range is copied out
// in aligned 16-byte words.
#include <mutex>

#include "../../include/gerbil.h"
#include "table.h"

namespace gerbil {
namespace {

constexpr uint32_t kRecBlock = 1024;
// Rounds of kRecBlock pairs per tile: eight, so that the next one's pairs are on
// their way, or one where tiles of eight would be fewer than one per CU
// (50 000 pairs of k = 28: 59 us a call with eight, 39 with one).
constexpr uint32_t kRecRoundsBig = 8, kRecRoundsSmall = 1;
constexpr uint64_t kRecBigFrom = 256ull * kRecBlock * kRecRoundsBig;
constexpr uint64_t tiles_of(uint64_t n, uint32_t rounds) { return (n + (uint64_t)kRecBlock * rounds - 1) / ((uint64_t)kRecBlock * rounds); }
// Tiles a workspace for n pairs has room for: never fewer for more pairs.
constexpr uint64_t tiles_for(uint64_t n) {
    return n < kRecBigFrom ? tiles_of(n, kRecRoundsSmall)
                           : tiles_of(n, kRecRoundsBig) > tiles_of(kRecBigFrom, kRecRoundsSmall)
                                 ? tiles_of(n, kRecRoundsBig)
                                 : tiles_of(kRecBigFrom, kRecRoundsSmall);
}

__device__ __forceinline__ uint32_t block_sum(uint32_t v, uint32_t* wsum) {
    uint32_t total;
    (void)block_excl_scan(v, wsum, total);
    return total;
}

// Large counters (>= 255) per tile.
template <uint32_t kRecRounds>
__global__ void __launch_bounds__(kRecBlock) k_rec_flags(const uint32_t* __restrict__ counts, uint64_t n,
                                                         uint32_t* __restrict__ tile_big) {
    __shared__ uint32_t wsum[32];
    constexpr uint64_t kRecTile = (uint64_t)kRecBlock * kRecRounds;
    const uint64_t n_tiles = tiles_of(n, kRecRounds);
    for (uint64_t t = blockIdx.x; t < n_tiles; t += gridDim.x) {
        uint32_t big = 0;
#pragma unroll
        for (uint32_t r = 0; r < kRecRounds; r++) {
            const uint64_t i = t * kRecTile + (uint64_t)r * kRecBlock + threadIdx.x;
            big += (i < n && counts[i] >= 255u) ? 1u : 0u;
        }
        const uint32_t tot = block_sum(big, wsum);
        if (threadIdx.x == 0) tile_big[t] = tot;
        __syncthreads();
    }
}

// Exclusive prefix of the tile totals (one workgroup); writes the stream size.
__global__ void __launch_bounds__(kRecBlock) k_rec_scan(const uint32_t* __restrict__ tile_big, uint64_t n_tiles,
                                                        uint64_t* __restrict__ tile_base, uint64_t n, uint32_t kb,
                                                        uint64_t* out_bytes) {
    __shared__ uint64_t part[kRecBlock];
    const uint32_t tid = threadIdx.x;
    const uint64_t per = (n_tiles + kRecBlock - 1) / kRecBlock;
    uint64_t sum = 0;
    for (uint64_t e = 0; e < per; e++) {
        const uint64_t j = tid * per + e;
        if (j < n_tiles) sum += tile_big[j];
    }
    part[tid] = sum;
    __syncthreads();
    for (uint32_t off = 1; off < kRecBlock; off <<= 1) {
        const uint64_t y = tid >= off ? part[tid - off] : 0ull;
        __syncthreads();
        part[tid] += y;
        __syncthreads();
    }
    uint64_t run = tid ? part[tid - 1] : 0ull;
    for (uint64_t e = 0; e < per; e++) {
        const uint64_t j = tid * per + e;
        if (j < n_tiles) {
            tile_base[j] = run;
            run += tile_big[j];
        }
    }
    if (tid == kRecBlock - 1) *out_bytes = n * (1ull + kb) + 4ull * part[kRecBlock - 1];
}

// A word's bytes to p, the most significant first.
__device__ __forceinline__ void put64(uint8_t* p, uint64_t x) {
    x = __builtin_bswap64(x);
    __builtin_memcpy(p, &x, 8);
}

// The stage holds a round's records at their place modulo 16 in the output, so
// that it is copied out in aligned 16-byte words. The next round's pairs are
// requested before this one's are staged. Bound by memory: 20 M pairs of k =
// 65 (560 MB in, 360 MB out) in 0.19 ms; byte by byte it was bound by the LDS
// and store instructions, 0.39 ms.
template <int W, uint32_t kRecRounds>
__global__ void __launch_bounds__(kRecBlock) k_rec_write(const uint64_t* __restrict__ keys,
                                                         const uint32_t* __restrict__ counts, uint64_t n, uint32_t k,
                                                         const uint64_t* __restrict__ tile_base,
                                                         uint8_t* __restrict__ out, uint64_t out_cap) {
    constexpr uint32_t P = W <= 2 && kRecRounds > 1 ? 2 : 1;   // pairs a thread, kRecBlock apart: short ones leave room for two
    constexpr uint64_t kRecTile = (uint64_t)kRecBlock * kRecRounds;
    constexpr uint32_t kRound = P * kRecBlock;
    extern __shared__ __align__(16) uint8_t stage[];   // one round of records
    __shared__ uint32_t wsum[32];
    const uint32_t tid = threadIdx.x;
    const uint32_t kb = (k + 3) / 4;
    const uint32_t left = 2 * (32 * W - k);            // the last word is right-aligned
    const uint32_t end = kb - 8 * (W - 1);             // bytes of the last word, 1 .. 8
    const uint64_t n_tiles = tiles_of(n, kRecRounds);
    for (uint64_t t = blockIdx.x; t < n_tiles; t += gridDim.x) {
        uint64_t big_before = tile_base[t];   // large counters before this round
        uint32_t c_nxt[P];
        uint64_t key_nxt[P][W];
        auto request = [&](uint64_t i) {
#pragma unroll
            for (uint32_t q = 0; q < P; q++, i += kRecBlock) {
                c_nxt[q] = i < n ? counts[i] : 0u;
#pragma unroll
                for (int w = 0; w < W; w++) key_nxt[q][w] = i < n ? keys[i * W + w] : 0ull;
            }
        };
        request(t * kRecTile + tid);
        for (uint32_t r = 0; r < kRecRounds / P; r++) {
            const uint64_t i0 = t * kRecTile + (uint64_t)r * kRound;
            if (i0 >= n) break;
            uint32_t c[P], bigs = 0;   // (a half word for each of the pairs)
            uint64_t key[P][W];
#pragma unroll
            for (uint32_t q = 0; q < P; q++) {
                c[q] = c_nxt[q];
                bigs |= (c[q] >= 255u ? 1u : 0u) << (16 * q);
#pragma unroll
                for (int w = 0; w < W; w++) key[q][w] = key_nxt[q][w];
            }
            if (r + 1 < kRecRounds / P) request(i0 + kRound + tid);
            uint32_t big_round;
            uint32_t big_pre = block_excl_scan(bigs, wsum, big_round);
            if (P == 2) {   // the second pairs come after all the first
                big_pre += big_round << 16;
                big_round = (big_round & 0xFFFFu) + (big_round >> 16);
            }
            // the round's bytes start at the record offset of pair i0
            const uint64_t base = i0 * (1ull + kb) + 4ull * big_before;
            const uint32_t sh = (uint32_t)((uintptr_t)out + base) & 15u;
            const uint32_t n_here = (uint32_t)((n - i0) < kRound ? (n - i0) : kRound);
            const uint32_t round_bytes = n_here * (1u + kb) + 4u * big_round;
#pragma unroll
            for (uint32_t q = 0; q < P; q++) {
                if (tid + q * kRecBlock >= n_here) continue;
                const bool big = c[q] >= 255u;
                uint8_t* p = stage + sh + (tid + q * kRecBlock) * (1u + kb) + 4u * ((big_pre >> (16 * q)) & 0xFFFFu);
                *p++ = big ? 0xFF : (uint8_t)c[q];
                if (big) {
                    const uint32_t x = __builtin_bswap32(c[q]);
                    __builtin_memcpy(p, &x, 4);
                    p += 4;
                }
#pragma unroll
                for (int w = 0; w + 1 < W; w++, p += 8) put64(p, key[q][w]);
                uint64_t x = key[q][W - 1] << left;   // (zero bits after the last base)
                if (end == 8) {
                    put64(p, x);
                } else {
                    if (end & 4) {
                        const uint32_t y = __builtin_bswap32((uint32_t)(x >> 32));
                        __builtin_memcpy(p, &y, 4);
                        p += 4;
                        x <<= 32;
                    }
                    if (end & 2) {
                        const uint16_t y = __builtin_bswap16((uint16_t)(x >> 48));
                        __builtin_memcpy(p, &y, 2);
                        p += 2;
                        x <<= 16;
                    }
                    if (end & 1) *p = (uint8_t)(x >> 56);
                }
            }
            __syncthreads();
            for (uint32_t b = 16 * tid; b < sh + round_bytes; b += 16 * kRecBlock) {
                const uint64_t g = base + b - sh;   // (wraps for bytes before the round's first: not written)
                if (b >= sh && b + 16 <= sh + round_bytes && g + 16 <= out_cap) {
                    *(uint4*)(out + g) = *(const uint4*)(stage + b);
                } else {
                    for (uint32_t e = 0; e < 16; e++)
                        if (b + e >= sh && b + e < sh + round_bytes && g + e < out_cap) out[g + e] = stage[b + e];
                }
            }
            big_before += big_round;
            __syncthreads();   // the stage is reused by the next round
        }
    }
}

template <int W, uint32_t kRecRounds>
hipError_t rec_write(const uint64_t* keys, const uint32_t* counts, uint64_t n, uint32_t k, const uint64_t* tile_base,
                     uint8_t* out, uint64_t out_cap, uint32_t grid, hipStream_t s) {
    const uint32_t lds = (W <= 2 && kRecRounds > 1 ? 2 : 1) * kRecBlock * (5 + (k + 3) / 4) + 16;   // up to 128 KB: above the default dynamic LDS limit
    // set on every call: the attribute belongs to the current device's module
    const hipError_t e = hipFuncSetAttribute((const void*)k_rec_write<W, kRecRounds>,
                                             hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((k_rec_write<W, kRecRounds>), dim3(grid), dim3(kRecBlock), lds, s, keys, counts, n, k, tile_base, out,
                       out_cap);
    return hipGetLastError();
}

// Workspace bytes for n_tiles tiles: the large-counter count per tile, then
// the large counters before each tile.
constexpr uint64_t rec_ws_bytes(uint64_t n_tiles) { return 256 + ((4 * n_tiles + 255) & ~255ull) + 8 * n_tiles; }

template <uint32_t kRecRounds>
hipError_t enqueue_rounds(const uint64_t* keys, const uint32_t* counts, uint64_t n, uint32_t k, uint8_t* ws,
                          uint8_t* out, uint64_t out_cap, uint64_t* out_bytes, hipStream_t stream) {
    const uint32_t kb = (k + 3) / 4;
    const uint64_t n_tiles = tiles_of(n, kRecRounds);
    uint32_t* tile_big = (uint32_t*)(ws + 256);
    uint64_t* tile_base = (uint64_t*)(ws + 256 + ((4 * n_tiles + 255) & ~255ull));
    const uint32_t grid = (uint32_t)(n_tiles < 4096 ? n_tiles : 4096);
    hipLaunchKernelGGL((k_rec_flags<kRecRounds>), dim3(grid), dim3(kRecBlock), 0, stream, counts, n, tile_big);
    hipLaunchKernelGGL(k_rec_scan, dim3(1), dim3(kRecBlock), 0, stream, tile_big, n_tiles, tile_base, n, kb, out_bytes);
    switch ((k + 31) / 32) {
        case 1: return rec_write<1, kRecRounds>(keys, counts, n, k, tile_base, out, out_cap, grid, stream);
        case 2: return rec_write<2, kRecRounds>(keys, counts, n, k, tile_base, out, out_cap, grid, stream);
        case 3: return rec_write<3, kRecRounds>(keys, counts, n, k, tile_base, out, out_cap, grid, stream);
        case 4: return rec_write<4, kRecRounds>(keys, counts, n, k, tile_base, out, out_cap, grid, stream);
        case 5: return rec_write<5, kRecRounds>(keys, counts, n, k, tile_base, out, out_cap, grid, stream);
        case 6: return rec_write<6, kRecRounds>(keys, counts, n, k, tile_base, out, out_cap, grid, stream);
        case 7: return rec_write<7, kRecRounds>(keys, counts, n, k, tile_base, out, out_cap, grid, stream);
        case 8: return rec_write<8, kRecRounds>(keys, counts, n, k, tile_base, out, out_cap, grid, stream);
        case 9: return rec_write<9, kRecRounds>(keys, counts, n, k, tile_base, out, out_cap, grid, stream);
        case 10: return rec_write<10, kRecRounds>(keys, counts, n, k, tile_base, out, out_cap, grid, stream);
        case 11: return rec_write<11, kRecRounds>(keys, counts, n, k, tile_base, out, out_cap, grid, stream);
        case 12: return rec_write<12, kRecRounds>(keys, counts, n, k, tile_base, out, out_cap, grid, stream);
        case 13: return rec_write<13, kRecRounds>(keys, counts, n, k, tile_base, out, out_cap, grid, stream);
        case 14: return rec_write<14, kRecRounds>(keys, counts, n, k, tile_base, out, out_cap, grid, stream);
        case 15: return rec_write<15, kRecRounds>(keys, counts, n, k, tile_base, out, out_cap, grid, stream);
    }
    return hipErrorInvalidValue;
}

hipError_t enqueue_records(const uint64_t* keys, const uint32_t* counts, uint64_t n, uint32_t k, uint8_t* ws,
                           uint8_t* out, uint64_t out_cap, uint64_t* out_bytes, hipStream_t stream) {
    if (n == 0) return launch_fill_u64(out_bytes, 1, 0ull, stream);
    return n >= kRecBigFrom ? enqueue_rounds<kRecRoundsBig>(keys, counts, n, k, ws, out, out_cap, out_bytes, stream)
                            : enqueue_rounds<kRecRoundsSmall>(keys, counts, n, k, ws, out, out_cap, out_bytes, stream);
}

// The allocation-free variant keeps the workspace in a static device array
// of the library: one copy per GPU, at that GPU's own address, which the host
// learns once per device with hipGetSymbolAddress. The array's name in host
// code is only a host-side stand-in and is never passed to a kernel.
constexpr uint64_t kScratchBytes = rec_ws_bytes(tiles_for(GERBIL_RECORDS_NOALLOC_MAX));
constexpr int kMaxDevices = 64;

}  // namespace

static __device__ __align__(256) uint8_t scratch[kScratchBytes];

namespace {

std::mutex g_scratch_mu;
void* g_scratch[kMaxDevices] = {};

// Device address of `scratch` on the current device (looked up once per device).
hipError_t scratch_address(void** out) {
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    if (!g_scratch[dev]) {
        void* p = nullptr;
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return e;
        if (!p) return hipErrorInvalidSymbol;
        g_scratch[dev] = p;
    }
    *out = g_scratch[dev];
    return hipSuccess;
}

}  // namespace
}  // namespace gerbil

using namespace gerbil;

extern "C" {

int32_t gerbil_records_workspace(uint64_t n, uint64_t* bytes) {
    if (!bytes) return GERBIL_EINVAL;
    *bytes = rec_ws_bytes(tiles_for(n));
    return GERBIL_OK;
}

int32_t gerbil_records(const uint64_t* keys, const uint32_t* counts, uint64_t n, uint32_t k, void* ws,
                       uint64_t ws_bytes, uint8_t* out, uint64_t out_cap, uint64_t* out_bytes, hipStream_t stream) {
    if (!out_bytes || k < 1 || k > 32 * GERBIL_MAX_W) return GERBIL_EINVAL;
    if (n && (!keys || !counts || !ws || (out_cap && !out))) return GERBIL_EINVAL;
    if (n && (ws_bytes < rec_ws_bytes(tiles_for(n)) || (((uintptr_t)ws) & 255))) return GERBIL_EINVAL;
    return enqueue_records(keys, counts, n, k, (uint8_t*)ws, out, out_cap, out_bytes, stream) == hipSuccess
               ? GERBIL_OK
               : GERBIL_EDEVICE;
}

int32_t gerbil_records_noalloc(const uint64_t* keys, const uint32_t* counts, uint64_t n, uint32_t k, uint8_t* out,
                               uint64_t out_cap, uint64_t* out_bytes, hipStream_t stream) {
    if (!out_bytes || k < 1 || k > 32 * GERBIL_MAX_W || n > GERBIL_RECORDS_NOALLOC_MAX) return GERBIL_EINVAL;
    if (n && (!keys || !counts || (out_cap && !out))) return GERBIL_EINVAL;
    void* ws = nullptr;
    if (scratch_address(&ws) != hipSuccess) return GERBIL_EDEVICE;
    return enqueue_records(keys, counts, n, k, (uint8_t*)ws, out, out_cap, out_bytes, stream) == hipSuccess
               ? GERBIL_OK
               : GERBIL_EDEVICE;
}

}  // extern "C"
