// The table kernel of the batched counter: every sub-table of the piece
// partition (pieces.h) counted by one workgroup in an LDS hash table
// (Sec. 2.2, Alg. 1; Sec. 2.3.2: the hasher with its own table).
//
// A workgroup copies the packed bases of its sub-table's pieces into LDS,
// rolls every k-mer of them and inserts it. A slot does not hold the key: it
// is one 64-bit word [reference 32 | tag 16 | count 16], where the tag is part
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
//
// What bounds it: vector issue (60 % of the cycles at k = 65, some 3.4 wave-wide
// instructions per key) and the barriers between the stages of the one
// workgroup a CU holds; memory would take a third of its time (21 GB of whole
// 128-byte lines that hold the pieces' bases, 3 GB of pairs). So
// - the first try of a key is straight-line code for a bucket of two slots read
//   at once; the few that find it taken go to a queue per wave, and are probed
//   on in full waves (as a loop, a wave ran on for its slowest lane);
// - k-mers are cut into segments of 6, sorted by length, so that the lanes of a
//   wave roll equally far;
// - the pieces of the next round, and of the next sub-table, are requested
//   before the current ones are processed;
// - pairs are collected per wave and written 64 at a time.
// 1.7 G 65-mer windows (3.0 G bases, 30x): 15.6 ms, against 24.4 ms for a probe
// loop over single slots, one round at a time.
#pragma once
#include "pieces.h"
#include "table.h"

namespace gerbil {
namespace sub {

// k-mers a lane rolls from one start. Six make about two rounds of segments for
// every wave of a full sub-table; with eight half of the waves had a second
// round and the others waited (k = 200 9.55 -> 9.00 ms a pass, k = 28 9.51 ->
// 9.09, k = 65 27.3 -> 27.1); with five the starts cost more than that at k >= 99.
constexpr uint32_t kSeg = 6;
constexpr uint32_t kSegLenAt = 24;       // a segment: reference of its first k-mer, k-mers - 1

// The k bases of reference ref as D left-aligned words (the bits past them
// cleared). A reference to base o is 2 (o + 15), plus one for a k-mer whose
// canonical form is its reverse complement: ref / 32 is then the word that
// holds base o - 1, counted from the word before the staged ones, and the
// funnel shifts from there are by 30 - 2 ((o - 1) mod 16), never by 32. b32
// points to the word before the staged ones, 16 bases a word.
template <int D>
__device__ __forceinline__ void window(const uint32_t* b32, uint32_t ref, uint32_t tail_mask, uint32_t (&x)[D]) {
    const uint32_t* p = b32 + (ref >> 5);
    const uint32_t s = ~(ref | 1u);   // (the low five bits count)
    uint32_t w[D + 1];
#pragma unroll
    for (int i = 0; i <= D; i++) w[i] = p[i];
#pragma unroll
    for (int i = 0; i < D; i++) x[i] = funnel(w[i], w[i + 1], s);
    x[D - 1] &= tail_mask;
}
__device__ __forceinline__ uint32_t ref_of(uint32_t o) { return 2 * o + 30; }

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

// Hash of a key: its words rotated and added up, then mixed by one
// multiplication. The top bits choose the bucket, the low ones are the tag.
// (A multiply-add per word costs four issue slots here where this takes two.)
template <int D>
__device__ __forceinline__ uint32_t hash_key(const uint32_t (&x)[D]) {
    uint32_t h = x[0];
#pragma unroll
    for (int i = 1; i < D; i++) h = funnel(h, h, 21) + x[i];
    h = (h ^ (h >> 16)) * 0x9E3779B1u;
    return h ^ (h >> 15);
}

template <uint32_t B>
struct Wg {
    using Sh = SubShape<B>;
    uint8_t* lds;
    __device__ __forceinline__ uint32_t* hist() const { return (uint32_t*)(lds + Sh::hist_at); }
    __device__ __forceinline__ uint32_t* probes() const { return (uint32_t*)(lds + Sh::probe_at); }
    __device__ __forceinline__ uint32_t* sums() const { return (uint32_t*)(lds + Sh::sum_at); }
    __device__ __forceinline__ uint64_t* base() const { return (uint64_t*)(lds + Sh::base_at); }
    __device__ __forceinline__ uint32_t* cls() const { return (uint32_t*)(lds + Sh::cls_at); }
    __device__ __forceinline__ uint32_t* segs() const { return (uint32_t*)(lds + Sh::seg_at); }
    __device__ __forceinline__ uint32_t* bases() const { return (uint32_t*)(lds + Sh::bases_at); }
    __device__ __forceinline__ uint32_t* retries() const {
        return (uint32_t*)(lds + Sh::retry_at) + Sh::retry * (threadIdx.x >> 6);
    }
    // emission queue of a wave, over the segments: 64 slots
    __device__ __forceinline__ uint64_t* queue() const {
        return (uint64_t*)(lds + Sh::seg_at) + 64u * (threadIdx.x >> 6);
    }
};

// A key ready to be inserted: its hash, and the halves of the slot word that
// claims a slot for it with a count of one.
struct Probe {
    uint32_t hash, ref, tag1;
};

// Key of a rolled k-mer (fw, its reverse complement rc, reference ref without
// the strand). False if the key is not to be inserted: another slice's, or the
// one first word that is never stored in a table in the `-d` mode (sent to the
// emergency area).
template <int D, uint32_t B>
__device__ __forceinline__ bool make_probe(const CountArgs& a, const SubArgs& t, const Wg<B>& g,
                                           const uint32_t (&fw)[D], const uint32_t (&rc)[D], uint32_t ref, uint64_t kx,
                                           uint32_t V, uint32_t v, Probe& p) {
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
    p.hash = hash_key<D>(key);
    p.ref = ref + (take ? 1u : 0u);
    p.tag1 = (p.hash << 16) | 1u;
    if (V > 1 && fastrange32(p.hash * 0x85EBCA6Bu, V) != v) return false;
    if (kx && (((fw[0] ^ (uint32_t)(kx >> 32)) & (fw[1] ^ (uint32_t)kx)) == 0xFFFFFFFFu)) {
        constexpr int W = (D + 1) / 2;
        uint64_t w[W];
        to_words<D>(fw, a.k, w);
        w[0] ^= kx;
        overflow_push<W>(a, w);
        if (t.probe_hist) atomicAdd(&g.probes()[kProbeHist - 1], 1u);
        return false;
    }
    return true;
}

enum { kSettled = 0, kNext = 1, kAgain = 2 };

// One bucket of Alg. 1: settled, on to the next bucket, or this one again. A
// bucket's first slot fills before its second. A slot found free but lost to
// another lane leaves the bucket to be read again; one whose tag agrees without
// the bases agreeing sends every occurrence of the key on to the next bucket
// (the slot keeps its content), so a key has one slot only.
template <int D>
__device__ __forceinline__ uint32_t probe_bucket(uint64_t* slots, const uint32_t* b32, const Probe& p, uint32_t bk,
                                                 const uint32_t (&fw)[D], const uint32_t (&rc)[D],
                                                 uint32_t tail_mask) {
    uint64_t* s = slots + 2 * bk;
    const uint64_t c0 = __hip_atomic_load(s, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    const uint64_t c1 = __hip_atomic_load(s + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    const bool use0 = (uint32_t)c0 == 0 || ((uint32_t)c0 ^ p.tag1) < 0x10000u;
    uint64_t cur = use0 ? c0 : c1;
    s += use0 ? 0 : 1;
    uint32_t r = kNext;
    if ((uint32_t)cur == 0) {   // claim it; cur stays 0 if that works
        cur = 0;
        __hip_atomic_compare_exchange_strong(s, &cur, ((uint64_t)p.ref << 32) | p.tag1, __ATOMIC_RELAXED,
                                             __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        r = (uint32_t)cur == 0 ? kSettled : kAgain;
    }
    if (r != kSettled && ((uint32_t)cur ^ p.tag1) < 0x10000u) {
        // the tag agrees: compare with the first occurrence, base by base
        const uint32_t ref = (uint32_t)(cur >> 32);
        uint32_t x[D];
        window<D>(b32, ref, tail_mask, x);
        const bool other = (ref ^ p.ref) & 1u;
        uint32_t diff = 0;
#pragma unroll
        for (int i = 0; i < D; i++) diff |= x[i] ^ (other ? rc[i] : fw[i]);
        r = kNext;
        if (diff == 0) {
            __hip_atomic_fetch_add((uint32_t*)s, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
            r = kSettled;
        }
    }
    return r;
}

// The whole of Alg. 1 for a key: theta buckets, then the emergency area.
template <int D, uint32_t B>
__device__ __forceinline__ void insert(const CountArgs& a, const SubArgs& t, const Wg<B>& g, uint64_t* slots,
                                       const uint32_t* b32, const Probe& p, const uint32_t (&fw)[D],
                                       const uint32_t (&rc)[D], uint32_t tail_mask, uint64_t kx) {
    const uint32_t st = 1u + (p.hash & 1023u);
    uint32_t bk = fastrange32(p.hash, t.buckets), tries = 0, r;
    do {
        r = probe_bucket<D>(slots, b32, p, bk, fw, rc, tail_mask);
        if (r != kAgain) {
            bk += st;
            bk = min(bk, bk - t.buckets);   // (wraps to a large value below)
            tries++;
        }
    } while (r != kSettled && tries < t.theta);
    if (r != kSettled) {
        constexpr int W = (D + 1) / 2;
        uint32_t key[D];
#pragma unroll
        for (int i = 0; i < D; i++) key[i] = (p.ref & 1u) ? rc[i] : fw[i];
        uint64_t w[W];
        to_words<D>(key, a.k, w);
        w[0] ^= kx;
        overflow_push<W>(a, w);
        tries = kProbeHist;
    }
    if (t.probe_hist) atomicAdd(&g.probes()[tries < kProbeHist - 1 ? tries : kProbeHist - 1], 1u);
}

// Up to 64 queued k-mers, one per lane.
template <int D, uint32_t B>
__device__ __forceinline__ void retry(const CountArgs& a, const SubArgs& t, const Wg<B>& g, uint64_t* slots,
                                      const uint32_t* b32, const uint32_t* queue, uint32_t m, uint32_t pad,
                                      uint32_t tail_mask, uint64_t kx) {
    if (__lane_id() >= m) return;
    const uint32_t ref = queue[__lane_id()];
    uint32_t fw[D], rc[D];
    window<D>(b32, ref, tail_mask, fw);
    revcomp<D>(fw, pad, tail_mask, rc);
    Probe p;
    make_probe<D, B>(a, t, g, fw, rc, ref, kx, 1, 0, p);   // (only keys to insert are queued)
    insert<D, B>(a, t, g, slots, b32, p, fw, rc, tail_mask, kx);
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
    const uint32_t ref = (uint32_t)(e >> 32);
    uint32_t x[D];
    window<D>(b32, ref, tail_mask, x);
    if (ref & 1u) {
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
    constexpr uint32_t kQuads = D <= 6 ? 2 : D <= 10 ? 3 : 4;   // 16-byte loads that hold an ordinary piece
    extern __shared__ __align__(16) uint8_t lds_raw[];
    const Wg<B> g{lds_raw};
    const uint32_t tid = threadIdx.x, lane = __lane_id(), wave = tid >> 6;
    const uint32_t k = a.k, CP = (2 * t.buckets + B - 1) / B * B;   // slots, in whole rounds of the workgroup
    const uint32_t pad = 32u * D - 2u * k;   // 0 .. 30 bits
    const uint32_t tail_mask = 0xFFFFFFFFu << pad;
    const uint64_t kx = stored_xor(a.canonical, k);
    uint32_t* hist = g.hist();
    uint32_t* cls = g.cls();
    uint32_t* bases = g.bases();
    const uint32_t* b32 = bases - 1;
    uint64_t* slots = (uint64_t*)(bases + t.halves);   // (a multiple of 16 bytes)
    uint32_t* segs = g.segs();
    for (uint32_t i = tid; i < kLdsHist; i += B) hist[i] = 0;
    if (tid < kProbeHist) g.probes()[tid] = 0;
    if (tid == 0) bases[-1] = 0;
    if (tid < 8) cls[tid] = 0;
    for (uint32_t i = tid; i < CP; i += B) slots[i] = 0;
    __syncthreads();
    uint32_t wmax = 0;
    const uint64_t tabs = *t.n_tab;   // (a bin that the last ones did not suffice for went to the fallback)
    const uint32_t n_tab = uniform(tabs < t.tab_cap ? (uint32_t)tabs : t.tab_cap), G = gridDim.x;
    // Work goes in batches of B pieces of one sub-table (and slice). While a
    // batch is counted the bases of the next one's pieces are on their way to
    // registers, the pieces of the one after that too, and the size and place
    // of the sub-table after that.
    struct Batch {
        uint32_t j, v, p0;
        uint64_t meta, off;
        __device__ __forceinline__ uint32_t pieces() const { return (uint32_t)(meta >> 32); }
    };
    auto slices = [&](uint64_t meta) -> uint32_t {
        // more k-mers than the table takes for sure: one pass per slice of the keys' hashes
        const uint32_t N = (uint32_t)meta;
        return N <= t.max_kmers ? 1u : (N + t.slice_kmers - 1) / t.slice_kmers;
    };
    auto meta_at = [&](uint32_t j) -> uint64_t { return j < n_tab ? t.tab_cnt[j] : 0ull; };
    auto off_at = [&](uint32_t j) -> uint64_t { return j < n_tab ? t.tab_off[j] : 0ull; };
    Batch cur{blockIdx.x, 0, 0, uniform(meta_at(blockIdx.x)), uniform(off_at(blockIdx.x))};
    uint64_t meta_f = meta_at(blockIdx.x + G), off_f = off_at(blockIdx.x + G);   // of the sub-table after nxt's
    auto advance = [&](Batch& x) {
        if (x.p0 + B < x.pieces()) {
            x.p0 += B;
        } else if (x.v + 1 < slices(x.meta)) {
            x.v++;
            x.p0 = 0;
        } else {
            x = Batch{x.j + G, 0, 0, uniform(meta_f), uniform(off_f)};
            meta_f = meta_at(x.j + G);
            off_f = off_at(x.j + G);
        }
    };
    auto piece_of = [&](const Batch& x) -> uint64_t {   // this thread's
        return x.p0 + tid < x.pieces() ? t.pieces[x.off + x.p0 + tid] : 0ull;
    };
    uint64_t x[2 * kQuads];
    auto request = [&](uint64_t d, bool have) {
        const uint32_t h = have ? (uint32_t)((piece_start(d) & 31) + piece_kmers(d) + k + 14) >> 4 : 0u;   // half words from its first word
        const uint64_t* src = a.packed + (piece_start(d) >> 5);
#pragma unroll
        for (uint32_t e = 0; e < kQuads; e++) {
            x[2 * e] = 4 * e < h ? src[2 * e] : 0ull;
            x[2 * e + 1] = 4 * e < h ? src[2 * e + 1] : 0ull;
        }
    };
    uint64_t d = piece_of(cur);
    request(d, cur.p0 + tid < cur.pieces());
    Batch nxt = cur;
    advance(nxt);
    uint64_t d_nxt = piece_of(nxt);
    uint32_t hbase = 0;   // half words staged so far
    while (cur.j < n_tab) {
        const uint64_t t0 = t.stage_clocks ? wall_clock64() : 0;
        const uint32_t np = cur.pieces(), V = slices(cur.meta), v = cur.v;
        const bool last = cur.p0 + B >= np;   // of the sub-table's pieces
        // one piece per thread
        const uint64_t start = piece_start(d);
        uint32_t n = cur.p0 + tid < np ? piece_kmers(d) : 0u;
        const uint32_t nh = n ? ((uint32_t)(start & 15) + n + k + 14) >> 4 : 0u;
        const uint32_t odd = (uint32_t)(start >> 4) & 1u;
        uint32_t nq = (nh + odd + 3) >> 2;   // its bases: whole words, 16 bytes at a time
        const uint64_t* src = a.packed + (start >> 5);
        // segments of kSeg k-mers, and one of the rest: ordered by length, so that
        // the lanes of a wave roll equally far
        uint32_t rest = n % kSeg;
        const uint32_t mine = nh | ((n / kSeg) << 16);
        const uint32_t incl = wave_incl_sum(mine);
        uint32_t rank = 0, add = 0;   // lane c: the wave's segments of c k-mers; lane 0: the sums
#pragma unroll
        for (uint32_t c = 1; c < kSeg; c++) {
            const uint64_t m = __ballot(rest == c);
            if (rest == c) rank = (uint32_t)__popcll(m & ((1ull << lane) - 1ull));
            if (lane == c) add = (uint32_t)__popcll(m);
        }
        if (lane == 0) add = __builtin_amdgcn_readlane(incl, 63);
        uint32_t from = 0;
        if (lane < kSeg) from = atomicAdd(&cls[lane], add);
        const uint32_t pre = __builtin_amdgcn_readlane(from, 0) + incl - mine;
        rank += __shfl(from, (int)rest);
        const uint32_t hpre = hbase + (pre & 0xFFFFu), spre = pre >> 16;
        __syncthreads();
        uint32_t total = uniform(cls[0]);
        uint32_t S = total >> 16, at = 0;
#pragma unroll
        for (uint32_t c = kSeg - 1; c > 0; c--) {
            if (c == rest) at = S + rank;
            S += cls[c];
        }
        if (hbase + (total & 0xFFFFu) > t.halves) {
            // The scan's weights rule this out. Bases past the stage would
            // overwrite slots: an error instead, and none of the batch counted.
            if (tid == 0) set_status(a.status, ST_SPIN);
            n = rest = nq = S = total = 0;
        }
        for (uint32_t q = 0; q < nq; q += kQuads) {
            if (q) {   // a longer piece than most
#pragma unroll
                for (uint32_t e = 0; e < kQuads; e++) {
                    x[2 * e] = q + e < nq ? src[2 * (q + e)] : 0ull;
                    x[2 * e + 1] = q + e < nq ? src[2 * (q + e) + 1] : 0ull;
                }
            }
#pragma unroll
            for (uint32_t e = 0; e < 4 * kQuads; e++) {
                const uint32_t i = 4 * q + e - odd;   // (wraps for the half word before the piece)
                if (i < nh) bases[hpre + i] = (uint32_t)(x[e >> 1] >> (e & 1 ? 0 : 32));
            }
        }
        d = d_nxt;
        request(d, nxt.p0 + tid < nxt.pieces());
        cur = nxt;
        advance(nxt);
        d_nxt = piece_of(nxt);
        const uint32_t ref = ref_of(16u * hpre + (uint32_t)(start & 15));
        uint32_t s0 = 0;
        do {
            if (s0) __syncthreads();
            for (uint32_t i = 0; i < n / kSeg; i++) {
                const uint32_t y = spre + i - s0;
                if (y < Sh::segs) segs[y] = (ref + 2 * i * kSeg) | ((kSeg - 1u) << kSegLenAt);
            }
            if (rest && at - s0 < Sh::segs) segs[at - s0] = (ref + 2 * (n - rest)) | ((rest - 1u) << kSegLenAt);
            __syncthreads();
            if (s0 == 0 && tid < 8) cls[tid] = 0;   // (every thread has read them)
            const uint32_t sn = S - s0 < Sh::segs ? S - s0 : Sh::segs;
            uint32_t* queue = g.retries();
            uint32_t qn = 0;   // queued k-mers of the wave
            for (uint32_t y0 = wave * 64; y0 < sn; y0 += B) {
                const uint32_t sg = segs[y0 + lane < sn ? y0 + lane : sn - 1];
                const uint32_t ref0 = sg & ((1u << kSegLenAt) - 1u);
                const uint32_t len = y0 + lane < sn ? (sg >> kSegLenAt) + 1u : 0u;
                const uint32_t most = __builtin_amdgcn_readfirstlane(len);   // (they never increase)
                uint32_t fw[D], rc[D];
                window<D>(b32, ref0, tail_mask, fw);
                revcomp<D>(fw, pad, tail_mask, rc);
                // the bases that follow the first k-mer (at most kSeg - 1)
                uint32_t nx[1];
                window<1>(b32, ref0 + 2 * k, 0xFFFFFFFFu, nx);
                for (uint32_t i = 0;;) {
                    Probe p;
                    bool left = false;
                    if (i < len && make_probe<D, B>(a, t, g, fw, rc, ref0 + 2 * i, kx, V, v, p)) {
                        left = probe_bucket<D>(slots, b32, p, fastrange32(p.hash, t.buckets), fw, rc, tail_mask) != kSettled;
                        if (t.probe_hist && !left) atomicAdd(&g.probes()[1], 1u);
                    }
                    const uint64_t m = __ballot(left);
                    if (left) {
                        const uint32_t q = qn + (uint32_t)__popcll(m & ((1ull << lane) - 1ull));
                        if (q < Sh::retry) queue[q] = ref0 + 2 * i;
                        else insert<D, B>(a, t, g, slots, b32, p, fw, rc, tail_mask, kx);
                    }
                    qn += (uint32_t)__popcll(m);
                    qn = qn < Sh::retry ? qn : Sh::retry;
                    if (++i >= most) break;
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
                if (qn >= 64) {
                    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
                    qn -= 64;
                    retry<D, B>(a, t, g, slots, b32, queue + qn, 64, pad, tail_mask, kx);
                    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
                }
            }
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            if (qn) retry<D, B>(a, t, g, slots, b32, queue, qn, pad, tail_mask, kx);
            s0 += Sh::segs;
        } while (s0 < S);
        hbase += total & 0xFFFFu;
        __syncthreads();   // the segments are done with; after the last batch, the slots are final
        if (!last) continue;
        hbase = 0;
        // (what was requested ahead has arrived: nothing that follows waits for the stores of the dump)
#pragma unroll
        for (uint32_t e = 0; e < 2 * kQuads; e++) asm volatile("" : "+v"(x[e]));
        asm volatile("" : "+v"(d_nxt), "+v"(meta_f), "+v"(off_f));
        // dump: the pairs are counted and places for them reserved; while that is on
        // its way the histogram is raised; then full waves of pairs are
        // written from a queue and the slots cleared
        uint32_t ones = 0, pairs = 0;   // of the wave (uniform)
        for (uint32_t s = tid; s < CP; s += 4 * B) {
#pragma unroll
            for (uint32_t i = 0; i < 4; i++) {
                const uint32_t c = s + i * B < CP ? ((const uint32_t*)(slots + s + i * B))[0] & 0xFFFFu : 0u;
                ones += (uint32_t)__popcll(__ballot(c == 1u));
                pairs += (uint32_t)__popcll(__ballot(c >= a.threshold));   // (a threshold is at least 1)
            }
        }
        if (lane == 0) {
            g.sums()[wave] = pairs;
            if (ones) atomicAdd(&hist[1], ones);
        }
        __syncthreads();
        if (tid == 0) {
            uint32_t all = 0;
            for (uint32_t i = 0; i < B / 64; i++) all += g.sums()[i];
            *g.base() = all ? add_dev(a.n_out, (uint64_t)all) : 0ull;
        }
        for (uint32_t s = tid; s < CP; s += 4 * B) {
#pragma unroll
            for (uint32_t i = 0; i < 4; i++) {
                const uint32_t c = s + i * B < CP ? ((const uint32_t*)(slots + s + i * B))[0] & 0xFFFFu : 0u;
                wmax = c > wmax ? c : wmax;
                if (c > 1u) {
                    if (c < kLdsHist) atomicAdd(&hist[c], 1u);
                    else add_dev(&a.hist[c], 1ull);   // at most 65535, the last bucket
                }
            }
        }
        __syncthreads();
        uint64_t pos = *g.base();
        for (uint32_t i = 0; i < wave; i++) pos += g.sums()[i];
        uint64_t* queue = g.queue();
        uint32_t qn = 0;
        for (uint32_t s = tid; s < CP; s += 4 * B) {
            uint64_t e[4];
#pragma unroll
            for (uint32_t i = 0; i < 4; i++) {
                e[i] = s + i * B < CP ? slots[s + i * B] : 0ull;
                if (s + i * B < CP) slots[s + i * B] = 0;
            }
#pragma unroll
            for (uint32_t i = 0; i < 4; i++) {
                const bool want = ((uint32_t)e[i] & 0xFFFFu) >= a.threshold;
                const uint64_t m = __ballot(want);
                if (m == 0) continue;
                const uint32_t at = qn + (uint32_t)__popcll(m & ((1ull << lane) - 1ull));
                if (want && at < 64) queue[at] = e[i];
                qn += (uint32_t)__popcll(m);
                if (qn >= 64) {
                    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
                    emit<D, B>(a, b32, queue, 64, pos, pad, tail_mask);
                    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
                    pos += 64;
                    qn -= 64;
                    if (want && at >= 64) queue[at - 64] = e[i];
                }
            }
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        if (qn) emit<D, B>(a, b32, queue, qn, pos, pad, tail_mask);
        __syncthreads();
        if (t.stage_clocks && tid == 0) {
            add_dev(&t.stage_clocks[3], wall_clock64() - t0);
            add_dev(&t.stage_clocks[7], 1ull);
        }
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
