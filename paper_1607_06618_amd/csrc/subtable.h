// The table kernel of the batched counter: every sub-table of the piece
// partition (pieces.h) counted by one workgroup in an LDS hash table
// (Sec. 2.2, Alg. 1; Sec. 2.3.2: the hasher with its own table).
//
// A workgroup copies the packed bases of its sub-table's pieces into LDS,
// rolls every k-mer of them and inserts it. A slot does not hold the key: it
// is one 64-bit word [tag 29 | reference 19 | count 16], where the tag is part
// of the key's hash and the reference says where in the staged bases the key
// was first seen and which strand is its canonical form. A key of any length
// so takes 8 bytes (a 65-mer 24, a 200-mer 56 when it is stored), one CAS
// claims and publishes a slot at once, and a lookup whose tag agrees is
// verified base by base against the staged bases, so counts are exact
// whatever the hash does. A key that fails theta probes goes to the emergency
// area (Sec. 3.4.3).
//
// Keys are held left-aligned in D 32-bit words, D = ceil(k / 16): the forward
// strand and the reverse complement both roll by one funnel shift per word.
#pragma once
#include "pieces.h"
#include "table.h"

namespace gerbil {
namespace sub {

constexpr uint32_t kSeg = 8;             // k-mers a lane rolls from one start
constexpr uint32_t kRefBits = 19;        // base in the staged ones, strand
constexpr uint32_t kSegBaseBits = 18;

// (hi:lo) >> s, low word, 0 <= s < 32.
__device__ __forceinline__ uint32_t funnel(uint32_t hi, uint32_t lo, uint32_t s) {
    return __builtin_amdgcn_alignbit(hi, lo, s);
}
// The 16 bases of x in reverse order, complemented.
__device__ __forceinline__ uint32_t revcomp16(uint32_t x) {
    x = __builtin_bitreverse32(~x);
    return ((x >> 1) & 0x55555555u) | ((x & 0x55555555u) << 1);
}

// Bases o.. of the staged ones as D left-aligned words (the bits past k
// bases cleared). b32 holds 16 bases a word, in order; word -1 exists.
template <int D>
__device__ __forceinline__ void window(const uint32_t* b32, uint32_t o, uint32_t tail_mask, uint32_t (&x)[D]) {
    // shifts of 2..32 from the half that holds base o - 1, so that a funnel
    // shift by 32 - 2..32 never needs the case of no shift
    const int32_t h = ((int32_t)o - 1) >> 4;
    const uint32_t s = 30u - 2u * ((o - 1u) & 15u);
    uint32_t w[D + 1];
#pragma unroll
    for (int i = 0; i <= D; i++) w[i] = b32[h + i];
#pragma unroll
    for (int i = 0; i < D; i++) x[i] = funnel(w[i], w[i + 1], s);
    x[D - 1] &= tail_mask;
}

// Reverse complement of D left-aligned words of k bases (pad = 32 D - 2 k bits).
template <int D>
__device__ __forceinline__ void revcomp(const uint32_t (&x)[D], uint32_t pad, uint32_t tail_mask, uint32_t (&y)[D]) {
    uint32_t r[D + 1];
#pragma unroll
    for (int i = 0; i < D; i++) r[i] = revcomp16(x[D - 1 - i]);
    r[D] = 0;
    if (pad) {
#pragma unroll
        for (int i = 0; i < D; i++) y[i] = funnel(r[i], r[i + 1], 32u - pad);
    } else {
#pragma unroll
        for (int i = 0; i < D; i++) y[i] = r[i];
    }
    y[D - 1] &= tail_mask;
}

// Words of the key layout of the ABI (the last one right-aligned).
template <int D>
__device__ __forceinline__ void to_words(const uint32_t (&x)[D], uint32_t k, uint64_t (&w)[(D + 1) / 2]) {
    constexpr int W = (D + 1) / 2;
#pragma unroll
    for (int i = 0; i < W; i++) w[i] = ((uint64_t)x[2 * i] << 32) | (2 * i + 1 < D ? x[2 * i + 1] : 0u);
    w[W - 1] >>= 2 * (32u * W - k);
}

// Hash of a key: a multilinear sum of its words modulo 2^64 (any difference of
// two words changes it). lo, whose top bits choose the slot, is mixed once
// more; hi is the tag.
template <int D>
__device__ __forceinline__ void hash_key(const uint32_t (&x)[D], uint32_t& hi, uint32_t& lo) {
    uint64_t s = 0x243F6A8885A308D3ull;
#pragma unroll
    for (int i = 0; i < D; i++) {
        // odd constants from SplitMix64's increment, one per word
        const uint32_t m = (uint32_t)((0x9E3779B97F4A7C15ull * (2 * i + 3)) >> 29) | 1u;
        s += (uint64_t)x[i] * m;
    }
    hi = (uint32_t)(s >> 32);
    lo = (uint32_t)s ^ hi;
    lo = (lo ^ (lo >> 15)) * 0x2C1B3C6Du;
}

template <int D, uint32_t B>
struct Wg {
    using Sh = SubShape<B>;
    uint8_t* lds;
    __device__ __forceinline__ uint32_t* hist() const { return (uint32_t*)(lds + Sh::hist_at); }
    __device__ __forceinline__ uint32_t* probes() const { return (uint32_t*)(lds + Sh::probe_at); }
    __device__ __forceinline__ uint32_t* wsum() const { return (uint32_t*)(lds + Sh::scan_at); }
    __device__ __forceinline__ uint64_t* base() const { return (uint64_t*)(lds + Sh::base_at); }
    __device__ __forceinline__ uint32_t* cls() const { return (uint32_t*)(lds + Sh::cls_at); }
    __device__ __forceinline__ uint32_t* segs() const { return (uint32_t*)(lds + Sh::seg_at); }
    __device__ __forceinline__ uint64_t* piece() const { return (uint64_t*)(lds + Sh::piece_at); }
    __device__ __forceinline__ uint32_t* pbase() const { return (uint32_t*)(lds + Sh::pbase_at); }
    __device__ __forceinline__ uint32_t* bases() const { return (uint32_t*)(lds + Sh::bases_at); }
    // emission queue of a wave, over the segments and the piece table: 128 slots each
    __device__ __forceinline__ uint64_t* queue() const {
        return (uint64_t*)(lds + Sh::seg_at) + 128u * (threadIdx.x >> 6);
    }
};

// Insert the key of a rolled k-mer (fw, its reverse complement rc, base o of
// the staged words). One loop with one exit: a lane stays in it until its key
// has a slot or theta probes have failed.
template <int D, uint32_t B>
__device__ __forceinline__ void insert(const CountArgs& a, const SubArgs& t, const Wg<D, B>& g, uint64_t* slots,
                                       const uint32_t* b32, const uint32_t (&fw)[D], const uint32_t (&rc)[D],
                                       uint32_t o, uint32_t tail_mask, uint64_t kx, uint32_t V, uint32_t v) {
    constexpr int W = (D + 1) / 2;
    // canonical strand: the first 32 bases nearly always decide
    const uint64_t f0 = ((uint64_t)fw[0] << 32) | fw[1], r0 = ((uint64_t)rc[0] << 32) | rc[1];
    bool take = r0 < f0;
    if (D > 2 && __ballot(r0 == f0) != 0ull) {
        bool same = r0 == f0;
#pragma unroll
        for (int i = 2; i < D; i++) {
            take = same ? rc[i] < fw[i] : take;
            same = same && rc[i] == fw[i];
        }
    }
    take = take && a.canonical;
    uint32_t key[D];
#pragma unroll
    for (int i = 0; i < D; i++) key[i] = take ? rc[i] : fw[i];
    uint32_t hi, lo;
    hash_key<D>(key, hi, lo);
    if (V > 1 && fastrange32(hi << 9, V) != v) return;   // another slice's key
    // (its other half: the one first word that is never stored in a table)
    bool pend = ((key[0] ^ (uint32_t)(kx >> 32)) & (key[1] ^ (uint32_t)kx)) == 0xFFFFFFFFu;
    uint32_t tries = 0;
    if (!pend) {
        const uint32_t C = t.slots, f = take ? 1u : 0u;
        uint32_t s = fastrange32(lo, C);
        const uint32_t st = 1u + (hi & 1023u);
        const uint32_t ref = (o << 1) | f;
        const uint32_t mine_hi = ((hi >> 6) << 6) | ((lo & 7u) << 3) | (ref >> 16), mine_lo = (ref << 16) | 1u;
        const uint64_t mine = ((uint64_t)mine_hi << 32) | mine_lo;
        do {
            uint64_t* p = slots + s;
            uint64_t cur = __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
            if (cur == 0)   // claim it, with a count of one; cur stays 0 if that works
                __hip_atomic_compare_exchange_strong(p, &cur, mine, __ATOMIC_RELAXED, __ATOMIC_RELAXED,
                                                     __HIP_MEMORY_SCOPE_WORKGROUP);
            pend = cur != 0;
            if (pend && (((uint32_t)(cur >> 32)) ^ mine_hi) < 8u) {
                // the tag agrees: compare with the first occurrence, base by base
                const uint32_t r = (uint32_t)(cur >> 16) & ((1u << kRefBits) - 1u);
                uint32_t x[D];
                window<D>(b32, r >> 1, tail_mask, x);
                const bool other = (r ^ f) & 1u;
                uint32_t diff = 0;
#pragma unroll
                for (int i = 0; i < D; i++) diff |= x[i] ^ (other ? rc[i] : fw[i]);
                if (diff == 0) {
                    __hip_atomic_fetch_add((uint32_t*)p, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                    pend = false;
                }
            }
            s += st;
            s = min(s, s - C);   // s - C wraps to a large value below C
            tries++;
        } while (pend && tries < t.theta);
    }
    if (pend) {
        uint64_t w[W];
        to_words<D>(key, a.k, w);
        w[0] ^= kx;
        overflow_push<W>(a, w);
        tries = kProbeHist;
    }
    if (t.probe_hist) atomicAdd(&g.probes()[tries < kProbeHist - 1 ? tries : kProbeHist - 1], 1u);
}

// The pairs of up to 64 queued slots, one per lane, to output positions from pos0.
template <int D, uint32_t B>
__device__ __forceinline__ void emit(const CountArgs& a, const uint32_t* b32, const uint64_t* queue, uint32_t m,
                                     uint64_t pos0, uint32_t pad, uint32_t tail_mask) {
    constexpr int W = (D + 1) / 2;
    const uint32_t lane = __lane_id();
    if (lane >= m) return;
    const uint64_t e = queue[lane], pos = pos0 + lane;
    if (pos >= a.cap) {
        set_status(a.status, ST_OUT_CAP);
        return;
    }
    const uint32_t r = (uint32_t)(e >> 16) & ((1u << kRefBits) - 1u);
    uint32_t x[D];
    window<D>(b32, r >> 1, tail_mask, x);
    if (r & 1u) {
        uint32_t y[D];
        revcomp<D>(x, pad, tail_mask, y);
#pragma unroll
        for (int i = 0; i < D; i++) x[i] = y[i];
    }
    uint64_t w[W];
    to_words<D>(x, a.k, w);
#pragma unroll
    for (int i = 0; i < W; i++) a.out_keys[pos * W + i] = w[i];
    a.out_counts[pos] = (uint32_t)e & 0xFFFFu;
}

template <int D, uint32_t B>
__global__ void __launch_bounds__(B, (D <= 16 ? 4 : 2)) k_sub_tables(CountArgs a, SubArgs t) {
    using Sh = SubShape<B>;
    extern __shared__ __align__(16) uint8_t lds_raw[];
    const Wg<D, B> g{lds_raw};
    const uint32_t tid = threadIdx.x, lane = __lane_id(), wave = tid >> 6;
    const uint32_t k = a.k, C = t.slots;
    const uint32_t pad = 32u * D - 2u * k;   // 0 .. 30 bits
    const uint32_t tail_mask = 0xFFFFFFFFu << pad;
    const uint64_t kx = stored_xor(a.canonical, k);
    uint32_t* hist = g.hist();
    uint32_t* bases = g.bases();
    const uint32_t* b32 = bases;
    uint64_t* slots = (uint64_t*)(bases + t.halves);   // (an even number)
    const uint32_t* packed = (const uint32_t*)a.packed;
    uint32_t* segs = g.segs();
    for (uint32_t i = tid; i < kLdsHist; i += B) hist[i] = 0;
    if (tid < kProbeHist) g.probes()[tid] = 0;
    if (tid == 0) bases[-1] = 0;
    for (uint32_t i = tid; i < C; i += B) slots[i] = 0;
    if (tid < 8) g.cls()[tid] = 0;
    __syncthreads();
    uint32_t wmax = 0;
    const uint32_t n_sub = (uint32_t)*t.n_sub;
    const uint32_t G = 1u << t.group_log2;
    // a sub-table's size and place are read two of them ahead, its first pieces one ahead
    uint32_t j = blockIdx.x;
    uint64_t meta = j < n_sub ? t.sub_cnt[j] : 0ull, off = j < n_sub ? t.sub_off[j] : 0ull;
    uint64_t first = tid < (uint32_t)(meta >> 32) ? t.pieces[off + tid] : 0ull;
    for (; j < n_sub; ) {
        const uint32_t N = (uint32_t)meta, np = (uint32_t)(meta >> 32), jn = j + gridDim.x;
        const uint64_t* in = t.pieces + off;
        const uint64_t meta_n = jn < n_sub ? t.sub_cnt[jn] : 0ull, off_n = jn < n_sub ? t.sub_off[jn] : 0ull;
        uint64_t first_n = 0;
        const uint64_t t0 = t.stage_clocks ? wall_clock64() : 0;
        // more k-mers than the table takes for sure: one pass per slice of the keys' hashes
        const uint32_t V = N == 0 ? 0u : N <= t.max_kmers ? 1u : (N + t.slice_kmers - 1) / t.slice_kmers;
        if (V == 0 && tid < (uint32_t)(meta_n >> 32)) first_n = t.pieces[off_n + tid];
        for (uint32_t v = 0; v < V; v++) {
            uint32_t wbase = 0;   // half words staged so far
            for (uint32_t p0 = 0; p0 < np; p0 += B) {
                const uint32_t nb = np - p0 < B ? np - p0 : B;
                uint64_t start = 0;
                uint32_t n = 0, nw = 0, rank = 0;
                if (tid < nb) {
                    const uint64_t d = p0 ? in[p0 + tid] : first;
                    start = piece_start(d);
                    n = piece_kmers(d);
                    nw = ((uint32_t)(start & 15) + n + k + 14) >> 4;
                    // segments of kSeg k-mers, and one of the rest: ordered by length, so
                    // that the lanes of a wave roll equally far
                    if (n % kSeg) rank = atomicAdd(&g.cls()[n % kSeg], 1u);
                }
                uint32_t total;
                const uint32_t pre = block_excl_scan(nw | ((n / kSeg) << 16), g.wsum(), total);
                const uint32_t wpre = wbase + (pre & 0xFFFFu), spre = pre >> 16, F = total >> 16;
                uint32_t S = F, at = 0;
                for (uint32_t c = kSeg - 1; c > 0; c--) {
                    const uint32_t x = g.cls()[c];
                    if (c == n % kSeg) at = S + rank;
                    S += x;
                }
                if (tid < nb) {
                    g.piece()[tid] = ((start >> 4) << 16) | nw;
                    g.pbase()[tid] = wpre;
                }
                for (uint32_t s0 = 0; s0 < S; s0 += Sh::segs) {
                    if (s0) __syncthreads();
                    const uint32_t o = 16u * wpre + (uint32_t)(start & 15);
                    for (uint32_t i = 0; i < n / kSeg; i++) {
                        const uint32_t x = spre + i - s0;
                        if (x < Sh::segs) segs[x] = (o + i * kSeg) | ((kSeg - 1u) << kSegBaseBits);
                    }
                    if (n % kSeg && at - s0 < Sh::segs)
                        segs[at - s0] = (o + (n & ~(kSeg - 1u))) | ((n % kSeg - 1u) << kSegBaseBits);
                    if (s0 == 0) {
                        __syncthreads();
                        if (tid < 8) g.cls()[tid] = 0;   // (read by every thread before the barrier)
                        // G lanes copy a piece's half words, four pieces of a group in flight
                        const uint32_t sub = tid & (G - 1), stride = B >> t.group_log2;
                        for (uint32_t p = tid >> t.group_log2; p < nb; p += 4 * stride) {
                            uint64_t info[4];
                            uint32_t to[4], x[4];
#pragma unroll
                            for (uint32_t e = 0; e < 4; e++) {
                                const uint32_t pp = p + e * stride;
                                info[e] = pp < nb ? g.piece()[pp] : 0ull;
                                to[e] = pp < nb ? g.pbase()[pp] : 0u;
                            }
#pragma unroll
                            for (uint32_t e = 0; e < 4; e++)   // a word's first 16 bases are its high half
                                x[e] = sub < (uint32_t)(info[e] & 0xFFFFu) ? packed[((info[e] >> 16) + sub) ^ 1] : 0u;
#pragma unroll
                            for (uint32_t e = 0; e < 4; e++) {
                                const uint32_t m = (uint32_t)(info[e] & 0xFFFFu);
                                if (sub < m) bases[to[e] + sub] = x[e];
                                for (uint32_t i = sub + G; i < m; i += G)
                                    bases[to[e] + i] = packed[((info[e] >> 16) + i) ^ 1];
                            }
                        }
                        // the next sub-table's pieces arrive while this one is counted
                        if (v + 1 == V && p0 + B >= np && tid < (uint32_t)(meta_n >> 32)) first_n = t.pieces[off_n + tid];
                    }
                    __syncthreads();
                    const uint32_t sn = S - s0 < Sh::segs ? S - s0 : Sh::segs;
                    for (uint32_t x = tid; x < sn; x += B) {
                        const uint32_t sg = segs[x];
                        const uint32_t o0 = sg & ((1u << kSegBaseBits) - 1u), len = (sg >> kSegBaseBits) + 1u;
                        uint32_t fw[D], rc[D];
                        window<D>(b32, o0, tail_mask, fw);
                        revcomp<D>(fw, pad, tail_mask, rc);
                        // the bases that follow the first k-mer (at most kSeg - 1)
                        uint32_t nx[1];
                        window<1>(b32, o0 + k, 0xFFFFFFFFu, nx);
                        for (uint32_t i = 0;;) {
                            insert<D, B>(a, t, g, slots, b32, fw, rc, o0 + i, tail_mask, kx, V, v);
                            if (++i >= len) break;
                            const uint32_t bb = nx[0] >> 30;
                            nx[0] <<= 2;
#pragma unroll
                            for (int q = 0; q + 1 < D; q++) fw[q] = funnel(fw[q], fw[q + 1], 30);
                            fw[D - 1] = (fw[D - 1] << 2) | (bb << pad);
#pragma unroll
                            for (int q = D - 1; q > 0; q--) rc[q] = funnel(rc[q - 1], rc[q], 2);
                            rc[0] = (rc[0] >> 2) | ((3u - bb) << 30);
                            rc[D - 1] &= tail_mask;
                        }
                    }
                }
                wbase += total & 0xFFFFu;
                if (p0 + B < np) __syncthreads();   // the batch's segments and piece table are done with
            }
            __syncthreads();
            // dump: count the pairs and the histogram, reserve, then write and clear
            uint32_t mine = 0;   // the wave's pairs (uniform)
            for (uint32_t s0 = 0; s0 < C; s0 += B) {
                const uint32_t s = s0 + tid;
                const uint32_t c = s < C ? ((const uint32_t*)(slots + s))[0] & 0xFFFFu : 0u;
                const uint64_t ones = __ballot(c == 1u);
                if (ones && lane == (uint32_t)__builtin_ctzll(ones)) atomicAdd(&hist[1], (uint32_t)__popcll(ones));
                if (c > 1u) {
                    if (c < kLdsHist) atomicAdd(&hist[c], 1u);
                    else add_dev(&a.hist[c], 1ull);   // at most 65535, the last bucket
                }
                wmax = c > wmax ? c : wmax;
                mine += (uint32_t)__popcll(__ballot(c != 0u && c >= a.threshold));
            }
            if (lane == 0) g.wsum()[wave] = mine;
            __syncthreads();
            if (tid == 0) {
                uint32_t all = 0;
                for (uint32_t i = 0; i < B / 64; i++) all += g.wsum()[i];
                *g.base() = all ? add_dev(a.n_out, (uint64_t)all) : 0ull;
            }
            __syncthreads();
            uint64_t pos = *g.base();
            for (uint32_t i = 0; i < wave; i++) pos += g.wsum()[i];
            uint64_t* queue = g.queue();
            uint32_t qn = 0;
            for (uint32_t s0 = 0; s0 < C; s0 += B) {
                const uint32_t s = s0 + tid;
                const uint64_t e = s < C ? slots[s] : 0ull;
                if (e) slots[s] = 0;
                const uint32_t c = (uint32_t)e & 0xFFFFu;
                const bool want = c != 0u && c >= a.threshold;
                const uint64_t m = __ballot(want);
                if (want) queue[qn + __popcll(m & ((1ull << lane) - 1ull))] = e;
                qn += (uint32_t)__popcll(m);
                if (qn >= 64) {
                    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
                    emit<D, B>(a, b32, queue, 64, pos, pad, tail_mask);
                    pos += 64;
                    qn -= 64;
                    const uint64_t rest = queue[64 + lane];
                    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
                    queue[lane] = rest;
                }
            }
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            if (qn) emit<D, B>(a, b32, queue, qn, pos, pad, tail_mask);
            __syncthreads();
        }
        if (t.stage_clocks && tid == 0 && V) {
            add_dev(&t.stage_clocks[3], wall_clock64() - t0);
            add_dev(&t.stage_clocks[7], 1ull);
        }
        j = jn;
        meta = meta_n;
        off = off_n;
        first = first_n;
    }
    flush_max(a.max_count, wmax);
    __syncthreads();
    for (uint32_t i = tid; i < kLdsHist; i += B)
        if (hist[i]) add_dev(&a.hist[i], (uint64_t)hist[i]);
    if (t.probe_hist && tid < kProbeHist && g.probes()[tid]) add_dev(&t.probe_hist[tid], (uint64_t)g.probes()[tid]);
}

template <int D, uint32_t B>
hipError_t run(const CountArgs& a, const SubArgs& t, uint32_t cus, hipStream_t s) {
    // set on every launch: the attribute belongs to the current device's module
    hipError_t e = hipFuncSetAttribute((const void*)k_sub_tables<D, B>, hipFuncAttributeMaxDynamicSharedMemorySize,
                                       (int)SubShape<B>::bytes);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((k_sub_tables<D, B>), dim3(cus * (1024u / B)), dim3(B), SubShape<B>::bytes, s, a, t);
    return hipGetLastError();
}

}  // namespace sub

// One translation unit per range of key lengths (D = ceil(k / 16)).
hipError_t sub_tables_2(const CountArgs& a, const SubArgs& t, uint32_t D, uint32_t B, uint32_t cus, hipStream_t s);
hipError_t sub_tables_9(const CountArgs& a, const SubArgs& t, uint32_t D, uint32_t B, uint32_t cus, hipStream_t s);
hipError_t sub_tables_15(const CountArgs& a, const SubArgs& t, uint32_t D, uint32_t B, uint32_t cus, hipStream_t s);
hipError_t sub_tables_20(const CountArgs& a, const SubArgs& t, uint32_t D, uint32_t B, uint32_t cus, hipStream_t s);
hipError_t sub_tables_26(const CountArgs& a, const SubArgs& t, uint32_t D, uint32_t B, uint32_t cus, hipStream_t s);

#define GERBIL_SUB_CASE(D)                                                                                       \
    case D: return B == 1024 ? sub::run<D, 1024>(a, t, cus, s) : sub::run<D, 512>(a, t, cus, s);

}  // namespace gerbil
