// Distribution into bins (phase one, Sec. 2.1 and Sec. 2.3.1 splitter step).
//
// The minimizer of a k-mer is its smallest m-mer under a total order on
// m-mers (Sec. 2.1); here the m-mers are canonical (smaller of the m-mer and
// its reverse complement) so that a k-mer and its reverse complement share a
// minimizer and therefore a bin. Orders (Sec. 3.1): KMC2-style -- canonical
// code c, moved behind all others (c + 4^m) when it starts with AAA or ACA --
// or plain lexicographic. A super-mer is a maximal run of consecutive valid
// k-mers with equal minimizers (Fig. 1); all of its k-mers go to the bin of
// that minimizer, so every occurrence of a canonical k-mer lands in one bin
// (the partition property of Sec. 2.1).
//
// The read stream is cut into tiles of kTile k-mer start positions; super-mers
// are also cut at tile boundaries (both pieces keep the same bin). A workgroup
// takes runs of consecutive tiles. A thread owns 8 positions of each: it
// computes the ranks of their m-mers for the next tile while it takes the
// minima of this one's windows of w = k-m+1 ranks, each as the suffix minimum
// of its own ranks (registers), the shared middle (minima of the threads'
// blocks) and the prefix minimum of the ranks where the windows end. Then
// one descriptor per super-mer piece is written into the workgroup's chunk of
// the list. Per-bin super-mer counts are privatised
// in LDS. A scan and an LDS-privatised scatter then group the descriptors by
// bin.
//
// The tile kernel is bound by vector issue (28 instructions a position, 75 %
// of the cycles): 3.0 G bases at k = 65 take 3.0 ms, against 6.8 ms when ranks
// were rolled one by one, windows read their ends rank by rank and one lane in
// two wrote descriptors. The descriptors are 1.0 GB of that, 0.2 ms.
#include "../../include/gerbil.h"
#include "common.h"
#include "internal.h"

namespace gerbil {

constexpr uint32_t kBinBlock = 256;
constexpr uint32_t kPer = 8;                                       // positions per thread
static_assert(kTile == kBinBlock * kPer, "one run of positions per thread");
// Ranks past the tile that its last windows reach (w <= 32 GERBIL_MAX_W, and
// the whole run of a thread).
constexpr uint32_t kHalo = 64;                                     // threads' runs
constexpr uint32_t kRow = kBinBlock + kHalo;
static_assert(kPer * kHalo >= 32 * GERBIL_MAX_W + 2 * kPer, "the longest window ends in the halo");
constexpr uint32_t kTileRun = 16;                                  // consecutive tiles of a workgroup at most

__device__ __forceinline__ uint32_t rank_of(uint64_t fw, uint64_t rc, uint32_t m, uint32_t order,
                                            const uint32_t* __restrict__ table) {
    uint64_t c = fw < rc ? fw : rc;
    if (order == GERBIL_ORDER_TABLE) return table[c];
    if (order == 0 && m >= 3) {
        uint64_t head = c >> (2 * m - 6);
        if (head == 0 /* AAA */ || head == 4 /* ACA */) c += 1ull << (2 * m);
    }
    return (uint32_t)c;
}

// Global data a thread needs for its 8 positions of a tile, loaded ahead.
struct TileFetch {
    uint32_t a, b;     // the 32 bases from the 16-base half that holds the first position
    uint32_t ok, ok0;  // valid-window bits of the positions (8), and of the 8 before them
};

__device__ __forceinline__ TileFetch tile_fetch(const BinArgs& a, uint64_t tile, bool wanted) {
    TileFetch f{0, 0, 0, 0};
    const uint64_t p = tile * kTile + threadIdx.x * kPer;
    if (!wanted || p >= a.n_bytes) return f;
    const uint32_t* P = (const uint32_t*)a.packed;   // a word's first 16 bases are its high half
    const uint8_t* ok = (const uint8_t*)a.kmer_ok;
    const uint64_t h = p >> 4;                       // (h + 1) / 2 is at most one word past the last
    f.a = P[h ^ 1];
    f.b = P[(h + 1) ^ 1];
    f.ok = ok[p >> 3];
    if (p) f.ok0 = ok[(p >> 3) - 1];
    return f;
}

// Ranks of the m-mers at a thread's 8 positions. Forward and reverse-complement
// codes are cut out of 32 bases of either strand by constant shifts, left-
// aligned with whatever follows them below: the smaller one is the same, and
// the last shift drops the rest. Six instructions a position.
__device__ __forceinline__ void ranks8(const BinArgs& a, const TileFetch& f, uint32_t (&r)[kPer]) {
    const bool mid = threadIdx.x & 1u;   // the first position is the 9th base of its half word
    const uint32_t hi = mid ? funnel(f.a, f.b, 16) : f.a;
    const uint32_t lo = mid ? f.b << 16 : f.b;
    // reverse complement; the m-mer at position 7 in the top bits
    const uint64_t y = (((uint64_t)revcomp16(lo) << 32) | revcomp16(hi)) << (2 * (32 - a.m) - 14);
    const uint32_t yhi = (uint32_t)(y >> 32), ylo = (uint32_t)y;
    const uint32_t down = 32 - 2 * a.m;
    // KMC2 order: AAA and ACA (first bits 000000 and 000100) come behind all
    // others; nothing is left of the saturated difference for the rest
    const uint32_t head = a.order == 0 && a.m >= 3 ? 0xEC000000u : 0u, one = head ? 1u : 0u;
#pragma unroll
    for (uint32_t e = 0; e < kPer; e++) {
        const uint32_t fw = e ? funnel(hi, lo, 32 - 2 * e) : hi;
        const uint32_t rc = e < 7 ? funnel(yhi, ylo, 18 + 2 * e) : yhi;
        const uint32_t c = fw < rc ? fw : rc;
        const uint32_t moved = __builtin_elementwise_sub_sat(one, c & head);
        r[e] = funnel(moved, c, down);   // moved 4^m + code
    }
    if (a.order == GERBIL_ORDER_TABLE) {
#pragma unroll
        for (uint32_t e = 0; e < kPer; e++) r[e] = a.rank_table[r[e]];
    }
}

// Minima of a thread's 8 windows, to M, and which of them differ from the one
// before (the first window's bit on top). kR: (w - 1) mod 8, so that every
// address is a constant away from the thread's column.
template <uint32_t kR>
__device__ __forceinline__ uint32_t window_minima(const uint32_t* R, const uint32_t* BM, uint32_t* M,
                                                  const uint32_t (&cur)[kPer], uint32_t before, uint32_t q) {
    const uint32_t tid = threadIdx.x;
    const uint32_t* Rq = R + tid + q;
    // [8 tid + 8, 8 tid + w - 1): in every one of these windows
    uint32_t mid = 0xFFFFFFFFu;
#pragma unroll
    for (uint32_t e = 0; e < kR; e++) mid = min(mid, Rq[e * kRow]);
    const uint32_t* B = BM + tid + 1;
    uint32_t j = q - 1;
    for (; j >= 6; j -= 6, B += 6)
        mid = min(min(min(mid, min(B[0], B[1])), min(B[2], B[3])), min(B[4], B[5]));
    if (j & 4) {
        mid = min(min(mid, min(B[0], B[1])), min(B[2], B[3]));
        B += 4;
    }
    if (j & 2) {
        mid = min(mid, min(B[0], B[1]));
        B += 2;
    }
    if (j & 1) mid = min(mid, B[0]);
    uint32_t suf[kPer];
    suf[7] = cur[7];
#pragma unroll
    for (int e = 6; e >= 0; e--) suf[e] = min(cur[e], suf[e + 1]);
    uint32_t mn = min(min(before, suf[0]), mid), diff = 0;
#pragma unroll
    for (uint32_t e = 0; e < kPer; e++) {
        constexpr uint32_t P = kPer;
        mid = min(mid, Rq[((kR + e) % P) * kRow + (kR + e) / P]);   // the rank that this window ends with
        const uint32_t v = min(suf[e], mid);
        diff = diff + diff + (v != mn ? 1u : 0u);
        M[e * kBinBlock + tid] = v;
        mn = v;
    }
    return diff;
}

__global__ void __launch_bounds__(kBinBlock, 6) k_bin_tiles(BinArgs a, uint32_t run) {
    // Rank of position 8 j + e of the tile at row e, column j (the halo
    // included): every access is to consecutive words across the lanes.
    __shared__ uint32_t R[kPer * kRow];
    __shared__ uint32_t BM[kRow];                     // minima of the columns
    __shared__ uint32_t M[kPer * kBinBlock];          // minimizer of the window at position 8 j + e: row e, column j
    __shared__ uint16_t Q[kBinBlock / 64][kPer * 64]; // starts of every wave
    __shared__ uint64_t brk[kTile / 64];              // starts and positions without a window
    __shared__ uint32_t cnt[kTileWaves];              // starts of every wave
    __shared__ uint64_t s_chunk;
    extern __shared__ uint32_t bin_cnt[];             // [n_bins]

    const uint32_t tid = threadIdx.x, lane = __lane_id(), wave = uniform(tid >> 6);
    const uint32_t w = a.k - a.m + 1;
    const uint64_t n_tiles = (a.n_bytes + kTile - 1) / kTile;
    const uint32_t code_mask = (uint32_t)((1ull << (2 * a.m)) - 1ull);
    const bool in_halo = tid * kPer < w + kPer;       // columns of the next tile that this one reads
    // list slots of this workgroup's current chunk [ch_cur, ch_end): every wave
    // keeps the same account. The first chunk is its own; more are reserved.
    uint64_t ch_cur = (uint64_t)blockIdx.x * a.list_chunk, ch_end = ch_cur + a.list_chunk;

    for (uint32_t b = tid; b < a.n_bins; b += kBinBlock) bin_cnt[b] = 0;

    for (uint64_t t0 = (uint64_t)blockIdx.x * run; t0 < n_tiles; t0 += (uint64_t)gridDim.x * run) {
        const uint64_t t1 = t0 + run < n_tiles ? t0 + run : n_tiles;
        TileFetch f = tile_fetch(a, t0, true);
        uint32_t cur[kPer];
        ranks8(a, f, cur);
        uint32_t ok = f.ok, ok0 = f.ok0;
        f = tile_fetch(a, t0 + 1, t0 + 1 < t1 || in_halo);
        for (uint64_t tile = t0; tile < t1; tile++) {
            // 1. this tile's ranks to LDS (nothing reads the last tile's any
            //    more), and the next one's: of the last tile of a run only
            //    what the windows of this one reach
            uint32_t nxt[kPer];
            {
                uint32_t bm = cur[0];
#pragma unroll
                for (uint32_t e = 0; e < kPer; e++) {
                    R[e * kRow + tid] = cur[e];
                    bm = min(bm, cur[e]);
                }
                BM[tid] = bm;
            }
            if (tile + 1 < t1 || wave * 64 * kPer < w + kPer) {
                ranks8(a, f, nxt);
                if (wave == 0) {
                    uint32_t bm = nxt[0];
#pragma unroll
                    for (uint32_t e = 0; e < kPer; e++) {
                        R[e * kRow + kBinBlock + lane] = nxt[e];
                        bm = min(bm, nxt[e]);
                    }
                    BM[kBinBlock + lane] = bm;
                }
            }
            const uint32_t ok_nxt = f.ok, ok0_nxt = f.ok0;
            f = tile_fetch(a, tile + 2, tile + 2 < t1 || (tile + 2 == t1 && in_halo));
            __syncthreads();
            // 2. minimizers: window e of the thread is ranks [8 tid + e, 8 tid + e + w).
            const uint32_t before = R[7 * kRow + (tid ? tid - 1 : 0)];   // (any value for the tile's first)
            uint32_t diff = 0;
            if (w > kPer) {
                const uint32_t q = (w - 1) / kPer;
                switch ((w - 1) % kPer) {
                    case 0: diff = window_minima<0>(R, BM, M, cur, before, q); break;
                    case 1: diff = window_minima<1>(R, BM, M, cur, before, q); break;
                    case 2: diff = window_minima<2>(R, BM, M, cur, before, q); break;
                    case 3: diff = window_minima<3>(R, BM, M, cur, before, q); break;
                    case 4: diff = window_minima<4>(R, BM, M, cur, before, q); break;
                    case 5: diff = window_minima<5>(R, BM, M, cur, before, q); break;
                    case 6: diff = window_minima<6>(R, BM, M, cur, before, q); break;
                    default: diff = window_minima<7>(R, BM, M, cur, before, q); break;
                }
            } else {
                uint32_t mn = before;
                for (uint32_t i = 0; i + 1 < w; i++) mn = min(mn, R[i * kRow + tid]);
#pragma unroll
                for (uint32_t e = 0; e < kPer; e++) {
                    uint32_t v = 0xFFFFFFFFu;
                    for (uint32_t i = e; i < e + w; i++) v = min(v, R[(i % kPer) * kRow + i / kPer + tid]);
                    diff = diff + diff + (v != mn ? 1u : 0u);
                    M[e * kBinBlock + tid] = v;
                    mn = v;
                }
            }
            diff = __builtin_bitreverse32(diff) >> 24;
            // 3. super-mer starts; the first position of a tile always starts a piece (the tile cut)
            uint32_t st = ok & (diff | ~((ok << 1) | (ok0 >> 7)) | (tid == 0 ? 1u : 0u));
            ((uint8_t*)brk)[tid] = (uint8_t)(st | ~ok);
            const uint32_t mine = (uint32_t)__popc(st), incl = wave_incl_sum(mine);
            const uint32_t n_st = __builtin_amdgcn_readlane(incl, 63);
            for (uint32_t at = incl - mine; st; at++, st &= st - 1) Q[wave][at] = (uint16_t)(tid * kPer + __builtin_ctz(st));
            if (lane == 0) cnt[wave] = n_st;
            __syncthreads();
            // 4. one descriptor per start. List slots: the rest of the chunk first,
            //    then a new chunk (reserved only when the current one runs
            //    out), so only the unused end of a workgroup's last chunk is
            //    left as a hole. One address takes an atomic every 10 ns or
            //    so: a chunk per wave and tile, of 512 slots, would bound the
            //    kernel.
            const uint32_t n0 = uniform(cnt[0]), n1 = n0 + uniform(cnt[1]), n2 = n1 + uniform(cnt[2]);
            const uint32_t all = n2 + uniform(cnt[3]);
            const uint64_t b1 = ch_cur;
            uint64_t b2 = 0;
            const uint32_t rest = (uint32_t)(ch_end - ch_cur), split = rest < all ? rest : all;
            if (all > split) {
                const uint32_t need = all - split, take = need > a.list_chunk ? need : a.list_chunk;
                if (tid == 0) s_chunk = (uint64_t)gridDim.x * a.list_chunk + add_dev(a.list_used, (uint64_t)take);
                __syncthreads();
                b2 = uniform(s_chunk);
                ch_cur = b2 + need;
                ch_end = b2 + take;
            } else {
                ch_cur += all;
            }
            // (some 110 starts at k = 65: the waves take turns at them 64 at a
            // time, rather than each its own in a third of its lanes)
            for (uint32_t i = ((tid + (uint32_t)tile * 64) % kBinBlock); i < all; i += kBinBlock) {
                const uint32_t v = (i >= n0 ? 1u : 0u) + (i >= n1 ? 1u : 0u) + (i >= n2 ? 1u : 0u);
                const uint32_t t = Q[v][i - (v == 0 ? 0u : v == 1 ? n0 : v == 2 ? n1 : n2)], c = t >> 6, bit = t & 63;
                uint64_t above = (brk[c] >> bit) >> 1;
                uint32_t end = t + 1;
                if (above) {
                    end += (uint32_t)__builtin_ctzll(above);
                } else {
                    end = kTile;
                    for (uint32_t d = c + 1; d < kTile / 64; d++) {
                        if (brk[d]) { end = d * 64 + (uint32_t)__builtin_ctzll(brk[d]); break; }
                    }
                }
                const uint32_t mr = M[(t % kPer) * kBinBlock + t / kPer];
                uint32_t bin = a.bin_map ? a.bin_map[mr & code_mask] : (mr % a.n_bins);
                if (bin >= a.n_bins) bin = a.n_bins - 1;   // defensive: a bad map must not index out of range
                atomicAdd(&bin_cnt[bin], 1u);
                const uint64_t idx = i < split ? b1 + i : b2 + (i - split);
                if (idx < a.list_cap) {
                    a.list_desc[idx] = ((tile * kTile + t) << 24) | (end - t);
                    a.list_bin[idx] = bin;
                } else {
                    set_status(a.status, ST_SUPERM_CAP);
                }
            }
#pragma unroll
            for (uint32_t e = 0; e < kPer; e++) cur[e] = nxt[e];
            ok = ok_nxt;
            ok0 = ok0_nxt;
        }
    }
    // the unused end of the last chunk is a hole
    for (uint64_t i = ch_cur + tid; i < ch_end; i += kBinBlock)
        if (i < a.list_cap) a.list_bin[i] = kHole;
    __syncthreads();
    uint32_t* total = a.bin_count + (blockIdx.x % kBinCopies) * a.n_bins;
    for (uint32_t b = tid; b < a.n_bins; b += kBinBlock)
        if (bin_cnt[b]) atomicAdd(&total[b], bin_cnt[b]);
}

// Exclusive prefix of the per-bin super-mer counts (single workgroup).
__global__ void __launch_bounds__(1024) k_bin_scan(BinArgs a) {
    __shared__ uint64_t part[1024];
    const uint32_t tid = threadIdx.x;
    const uint32_t per = (a.n_bins + 1023) / 1024;
    uint64_t local[4];
    uint64_t s = 0;
    for (uint32_t e = 0; e < per; e++) {
        uint32_t b = tid * per + e;
        uint64_t v = 0;
        if (b < a.n_bins)
            for (uint32_t c = 0; c < kBinCopies; c++) v += a.bin_count[c * a.n_bins + b];
        local[e] = s;
        s += v;
    }
    part[tid] = s;
    __syncthreads();
    for (uint32_t off = 1; off < 1024; off <<= 1) {
        uint64_t y = tid >= off ? part[tid - off] : 0ull;
        __syncthreads();
        part[tid] += y;
        __syncthreads();
    }
    uint64_t base = tid ? part[tid - 1] : 0ull;
    for (uint32_t e = 0; e < per; e++) {
        uint32_t b = tid * per + e;
        if (b < a.n_bins) {
            a.bin_off[b] = base + local[e];
            a.bin_fill[b] = 0;
            a.bin_kmers[b] = 0;
        }
    }
    if (tid == 1023) {
        a.bin_off[a.n_bins] = part[1023];
        *a.n_superm = part[1023];
    }
}

constexpr uint32_t kScatterPer = 16;   // descriptors per thread per chunk
// Chunks of 16384 descriptors, so that a bin's share of one (32 of 512 bins)
// is a few whole lines in the one L2 its workgroup writes through; shares of 8
// from chunks of 4096 took 1.28 ms for 80 M descriptors, these 0.57 ms.
// Lists that would not fill the chip with those take the small chunks.
constexpr uint32_t kScatterBig = 1024;
constexpr uint64_t kScatterBigFrom = 1ull << 23;   // list slots: two chunks per CU

template <uint32_t B>
__global__ void __launch_bounds__(B) k_bin_scatter(BinArgs a) {
    extern __shared__ uint64_t sh[];
    uint64_t* lh = sh;                              // [n_bins] count << 32 | k-mers in this chunk
    uint64_t* tk = sh + a.n_bins;                   // [n_bins] k-mers of this workgroup's chunks, added to the bins' totals once at the end
    uint32_t* gb = (uint32_t*)(sh + 2 * a.n_bins);  // [n_bins] place of this chunk's share in the list of bins
    const uint32_t tid = threadIdx.x;
    uint64_t n = a.list_first + ld_dev(a.list_used);   // list slots handed out, holes included
    if (n > a.list_cap) n = a.list_cap;
    const uint64_t chunk = (uint64_t)B * kScatterPer;
    for (uint32_t b = tid; b < a.n_bins; b += B) tk[b] = 0;   // read back only by thread b % B
    for (uint64_t c0 = blockIdx.x * chunk; c0 < n; c0 += (uint64_t)gridDim.x * chunk) {
        for (uint32_t b = tid; b < a.n_bins; b += B) lh[b] = 0;
        uint64_t d[kScatterPer];
        uint32_t bn[kScatterPer], lr[kScatterPer];
#pragma unroll
        for (uint32_t e = 0; e < kScatterPer; e++) {
            uint64_t i = c0 + tid + (uint64_t)e * B;
            bn[e] = 0xFFFFFFFFu;
            d[e] = 0;
            if (i < n) {
                bn[e] = a.list_bin[i];
                d[e] = a.list_desc[i];
            }
        }
        __syncthreads();
#pragma unroll
        for (uint32_t e = 0; e < kScatterPer; e++) {
            if (bn[e] < a.n_bins)
                lr[e] = (uint32_t)(atomicAdd((unsigned long long*)&lh[bn[e]], (1ull << 32) | (d[e] & 0xFFFFFFull)) >> 32);
            else
                bn[e] = 0xFFFFFFFFu;   // a hole
        }
        __syncthreads();
        for (uint32_t b = tid; b < a.n_bins; b += B) {
            const uint64_t c = lh[b];
            if (c) {
                gb[b] = atomicAdd(&a.bin_fill[b], (uint32_t)(c >> 32));
                tk[b] += (uint32_t)c;
            }
        }
        __syncthreads();
#pragma unroll
        for (uint32_t e = 0; e < kScatterPer; e++) {
            if (bn[e] == 0xFFFFFFFFu) continue;
            uint64_t pos = a.bin_off[bn[e]] + gb[bn[e]] + lr[e];
            if (pos < a.bin_off[bn[e] + 1] && pos < a.cap) a.desc[pos] = d[e];
        }
        __syncthreads();
    }
    for (uint32_t b = tid; b < a.n_bins; b += B)
        if (tk[b]) add_dev(&a.bin_kmers[b], tk[b]);
}

template <uint32_t B>
hipError_t run_bin_scatter(const BinArgs& a, hipStream_t s) {
    const size_t sh = 20 * (size_t)a.n_bins;
    if (sh > 65536) {   // above the default limit of dynamic LDS per workgroup (n_bins > 3276)
        const hipError_t e = hipFuncSetAttribute((const void*)k_bin_scatter<B>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)sh);
        if (e != hipSuccess) return e;
    }
    const uint64_t chunks = (a.list_cap + (uint64_t)B * kScatterPer - 1) / ((uint64_t)B * kScatterPer);
    const uint32_t most = 2048 * 256 / B, g = (uint32_t)(chunks < most ? (chunks ? chunks : 1) : most);
    hipLaunchKernelGGL(k_bin_scatter<B>, dim3(g), dim3(B), sh, s, a);
    return hipGetLastError();
}

// Bin of each key, as the tile kernel assigns it: the smallest rank over the
// k-m+1 canonical m-mers of the k-mer the key encodes, then bin_map or
// rank mod n_bins. (A key's m-mers are those of every window that holds it,
// on either strand, so the bin is the one its occurrences went to.)
__global__ void __launch_bounds__(256) k_key_bins(const uint64_t* __restrict__ keys, uint64_t n, uint32_t k,
                                                  uint32_t W, uint32_t m, uint32_t order,
                                                  const uint32_t* __restrict__ rank_table,
                                                  const uint32_t* __restrict__ bin_map, uint32_t n_bins,
                                                  uint32_t* __restrict__ bins) {
    const uint64_t mmask = (1ull << (2 * m)) - 1ull;
    for (uint64_t i = (uint64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (uint64_t)gridDim.x * 256) {
        const uint64_t* key = keys + i * W;
        uint64_t fw = 0, rc = 0;
        uint32_t best = 0xFFFFFFFFu, p = 0;
        for (uint32_t w = 0; w < W; w++) {
            const uint64_t x = key[w];
            const uint32_t r = w + 1 < W ? 32u : k - 32u * (W - 1);   // bases in this word, right-aligned
            for (uint32_t o = 0; o < r; o++, p++) {
                const uint64_t b = (x >> (2 * (r - 1 - o))) & 3ull;
                fw = ((fw << 2) | b) & mmask;
                rc = (rc >> 2) | ((3ull - b) << (2 * m - 2));
                if (p + 1 >= m) best = min(best, rank_of(fw, rc, m, order, rank_table));
            }
        }
        uint32_t bin = bin_map ? bin_map[best & (uint32_t)mmask] : best % n_bins;
        if (bin >= n_bins) bin = n_bins - 1;   // defensive, as in the tile kernel
        bins[i] = bin;
    }
}

hipError_t launch_key_bins(const uint64_t* keys, uint64_t n, const BinArgs& a, uint32_t* bins, hipStream_t s) {
    if (n == 0) return hipSuccess;
    const uint64_t g = (n + 255) / 256;
    hipLaunchKernelGGL(k_key_bins, dim3((uint32_t)(g < 65536 ? g : 65536)), dim3(256), 0, s, keys, n, a.k,
                       (a.k + 31) / 32, a.m, a.order, a.rank_table, a.bin_map, a.n_bins, bins);
    return hipGetLastError();
}

hipError_t launch_bin(BinArgs a, uint32_t max_grid, uint32_t cus, hipStream_t s) {
    size_t sh_tiles = (size_t)a.n_bins * sizeof(uint32_t);
    // as many workgroups as are resident at once (a second, partial wave of
    // workgroups would double the time of a grid-stride kernel)
    if (a.k - a.m + 1 > 32 * GERBIL_MAX_W) return hipErrorInvalidValue;
    int per_cu = 0;
    const hipError_t oe = hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, k_bin_tiles, kBinBlock, sh_tiles);
    if (oe != hipSuccess || per_cu < 1) per_cu = 1;
    uint64_t grid = (uint64_t)cus * (uint32_t)per_cu;
    if (grid > max_grid) grid = max_grid;
    if (grid < 1) grid = 1;
    // Consecutive tiles share the ranks at their boundary; at least four runs
    // per workgroup even out parts of the stream with more or fewer starts.
    const uint64_t n_tiles = (a.n_bytes + kTile - 1) / kTile;
    uint64_t run = n_tiles / (4 * grid);
    if (run < 1) run = (n_tiles + grid - 1) / grid;
    if (run < 1) run = 1;
    if (run > kTileRun) run = kTileRun;
    // a chunk holds about what a workgroup finds, so that a small input leaves few holes
    const uint64_t tiles = (n_tiles + grid - 1) / grid;
    const uint64_t est = tiles * kTile * 5 / (2 * (a.k - a.m + 2)) / 64 * 64 + 64;
    a.list_chunk = (uint32_t)(est < kListChunk ? est : kListChunk);
    a.list_first = grid * a.list_chunk;
    hipLaunchKernelGGL(k_bin_tiles, dim3((uint32_t)grid), dim3(kBinBlock), sh_tiles, s, a, (uint32_t)run);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_bin_scan, dim3(1), dim3(1024), 0, s, a);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
    return a.list_cap >= kScatterBigFrom + kListSlack ? run_bin_scatter<kScatterBig>(a, s) : run_bin_scatter<kBinBlock>(a, s);
}

}  // namespace gerbil
