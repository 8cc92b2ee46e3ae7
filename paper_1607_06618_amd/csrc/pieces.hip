// The partition of the bins into sub-tables by sub-minimizers (pieces.h), in
// four launches with no host synchronisation:
//   plan     groups per bin, work items (runs of descriptors of one bin);
//   split    super-mers cut into pieces, k-mers and pieces per group;
//   scan     groups to sub-tables, a contiguous run of pieces for each; heavy
//            groups (more k-mers or bases than a workgroup's LDS takes even in
//            slices: strongly repeated sub-minimizers) are set apart for the
//            fallback;
//   scatter  every piece to its sub-table's run.
// A bin whose pieces do not fit the list (which is sized for random
// sub-minimizers), or of 2^32 k-mers and more, is left to the fallback as a
// whole, so every input is counted exactly whatever its sub-minimizers look like.
#include "piece_plan.h"
#include "table.h"

namespace gerbil {

namespace {

constexpr uint32_t kPlanB = 1024;
constexpr uint32_t kScanB = 256;
constexpr uint32_t kScatB = 512;
constexpr uint32_t kBatch = 256;          // descriptors a wave takes at a time
constexpr uint32_t kScatGroups = 4096;     // groups and sub-tables of a bin that the scatter holds in LDS
constexpr uint32_t kScatTabs = 4096;

}  // namespace

// Inclusive sums of one value per thread in part[kPlanB] (all threads call it).
__device__ __forceinline__ void plan_scan(uint64_t* part, uint64_t v) {
    const uint32_t tid = threadIdx.x;
    part[tid] = v;
    __syncthreads();
    for (uint32_t off = 1; off < kPlanB; off <<= 1) {
        const uint64_t y = tid >= off ? part[tid - off] : 0ull;
        __syncthreads();
        part[tid] += y;
        __syncthreads();
    }
}

// Workgroup 0 plans; the others clear what the later launches add to (and with
// the first bins of a run the run's scalars and histogram).
__global__ void __launch_bounds__(kPlanB) k_piece_plan(PieceArgs q, uint64_t* zero_scalars, uint64_t* zero_hist) {
    const uint32_t tid = threadIdx.x;
    if (blockIdx.x > 0) {
        const uint64_t g = (uint64_t)(blockIdx.x - 1) * kPlanB + tid, G = (uint64_t)(gridDim.x - 1) * kPlanB;
        for (uint64_t i = g; i < q.grp_cap; i += G) q.grp_cnt[i] = 0;
        for (uint64_t i = g; i < q.tab_cap; i += G) {
            q.tab_cnt[i] = 0;
            q.tab_off[i] = ~0ull;
            q.tab_cur[i] = 0;
        }
        if (zero_hist)
            for (uint64_t i = g; i < kHistInternal; i += G) zero_hist[i] = 0;
        return;
    }
    __shared__ uint64_t part[kPlanB];
    if (zero_scalars && tid < 8) zero_scalars[tid] = 0;
    if (tid < kScalCount) q.scal[tid] = 0;
    const uint32_t n = q.n_bins, per = (n + kPlanB - 1) / kPlanB;
    const bool overfull = *q.n_superm > q.superm_cap;   // descriptors past the capacity were never stored
    const uint64_t S = overfull ? 0 : q.bin_off[n] - q.bin_off[0];   // (the bins of a PLAIN group are not the first)
    // k-mers per sub-table: the target, or less where that leaves workgroups without one
    uint64_t km = 0;
    for (uint32_t e = 0; e < per; e++) {
        const uint32_t b = tid * per + e;
        if (b < n && !overfull) km += q.bin_kmers[b];
    }
    plan_scan(part, km);
    const uint64_t target = plan_target(q, part[kPlanB - 1]);
    const bool many = part[kPlanB - 1] * kGroupsPerTable / target > (uint64_t)n * kManyGroups;
    const uint32_t descs = item_descs(S, many);
    __syncthreads();
    struct Planned {
        uint32_t groups, whole;
        uint64_t items;
    };
    auto planned = [&](uint32_t b) -> Planned {   // (everything is loaded before the caller stores)
        const uint64_t ns = q.bin_off[b + 1] - q.bin_off[b], K = q.bin_kmers[b];
        if (overfull || bin_left_whole(K)) return Planned{0, overfull ? 0u : 1u, 0};
        return Planned{bin_groups(q, target, ns, K), 0, (ns + descs - 1) / descs};
    };
    uint64_t sp = 0, it = 0;
    for (uint32_t e = 0; e < per; e++) {
        const uint32_t b = tid * per + e;
        if (b >= n) break;
        const Planned p = planned(b);
        sp += p.groups;
        it += p.items;
    }
    plan_scan(part, it);
    uint64_t it0 = part[tid] - it;
    const uint64_t n_items = part[kPlanB - 1];
    __syncthreads();
    plan_scan(part, sp);
    uint64_t sp0 = part[tid] - sp;
    const uint64_t n_sp = part[kPlanB - 1];
    // groups and items that do not fit their arrays (sized for any bins of
    // this many bases, so only for parameters far from the default): nothing
    // is split, and the fallback counts every bin
    const bool none = n_sp > q.grp_cap || n_items > q.items_cap;
    for (uint32_t e = 0; e < per; e++) {
        const uint32_t b = tid * per + e;
        if (b >= n) break;
        const Planned p = planned(b);
        q.ngrp[b] = none ? 0u : p.groups;
        q.grp_first[b] = none ? 0u : (uint32_t)sp0;
        q.item_first[b] = none ? 0u : (uint32_t)it0;
        q.bin_fail[b] = none ? 1u : p.whole;
        sp0 += p.groups;
        it0 += p.items;
    }
    if (tid == 0) {
        q.grp_first[n] = none ? 0u : (uint32_t)n_sp;
        q.item_first[n] = none ? 0u : (uint32_t)n_items;
        q.scal[kScalTarget] = target;
        q.scal[kScalItems] = none ? 0 : n_items;
        q.scal[kScalDescs] = descs;
        if (overfull) set_status(q.status, ST_SUPERM_CAP);
    }
}

// Bin of item `it`: last b with first[b] <= it (bins without items share their successor's start).
__device__ __forceinline__ uint32_t item_bin(const uint32_t* first, uint32_t n, uint32_t it) {
    uint32_t lo = 0, hi = n;
    while (hi - lo > 1) {
        const uint32_t mid = (lo + hi) >> 1;
        if (first[mid] <= it) lo = mid; else hi = mid;
    }
    return lo;
}

// The packed stream from base x on: requested in whole 128-bit loads, later cut
// into words of 16 bases (first base in the top bits).
typedef uint32_t Words __attribute__((ext_vector_type(16)));
struct BasesAhead {
    uint64_t w[8];
    uint32_t at;   // base before the first one, mod 32
    __device__ __forceinline__ void request(const uint64_t* packed, int64_t x, uint64_t n_bytes, uint32_t quads) {
        // from the word of base x - 1, so that no funnel shift is by 32
        const int64_t last = (int64_t)((n_bytes + 31) >> 5);   // two zero words follow the stream
        const int64_t e = (x - 1) >> 5;
        at = (uint32_t)(x - 1) & 31u;
#pragma unroll
        for (uint32_t j = 0; j < 4; j++) {
            if (j < quads) {   // (uniform)
                const int64_t i = e + 2 * (int64_t)j < last ? e + 2 * (int64_t)j : last;
                __builtin_memcpy(&w[2 * j], packed + i, 16);
            }
        }
    }
    __device__ __forceinline__ void cut(Words& v, uint32_t quads) const {
        const bool odd = at >= 16;
        const uint32_t s = 30u - 2u * (at & 15u);
        uint32_t h[16];
#pragma unroll
        for (uint32_t j = 0; j < 8; j++) {   // a word's first 16 bases are its high half
            h[2 * j] = (uint32_t)(w[j] >> 32);
            h[2 * j + 1] = (uint32_t)w[j];
        }
        uint32_t a = odd ? h[1] : h[0];
#pragma unroll
        for (uint32_t j = 0; j < 14; j++) {
            if (j % 4 == 2 && j / 4 + 1 >= quads) break;   // (uniform) nothing beyond was requested
            const uint32_t b = odd ? h[j + 2 < 16 ? j + 2 : 15] : h[j + 1];
            v[j] = funnel(a, b, s);
            a = b;
        }
    }
};

// Super-mers to pieces. A lane takes up to n0 consecutive windows of one
// super-mer and then the next descriptor of its wave's batch. All lanes of a
// wave run the steps of its longest lane, so a batch of 256 descriptors is
// taken longest first, and every branch is uniform. The descriptors are
// requested a batch ahead and the first bases a turn ahead: both come from
// places all over the stream. The n + w2 - 1 middle m2-mers of n windows (n <= w2) fall in three parts: the first n - 1 (window i holds those
// from i on: suffix minima), the w2 - n + 1 that every window holds, and the
// last n - 1 (window i holds the first i: prefix minima). Sixteen
// m2-mers at a time are cut out of two words each of the forward and the
// reverse-complement strand by constant shifts: about six instructions an
// m2-mer. The suffix minima wait in LDS, one column per lane (no conflicts);
// they are kept per block of 16 with the minima of the later blocks in rows
// of their own.
//
// Bound by vector issue (60 % of the cycles; some 1000 lane instructions a
// super-mer) and what is left of the latency of the scattered requests: 80 M
// super-mers of 1.7 G windows at k = 65 take 4.8 ms. Descriptors in stream
// order took 7.3 ms (each wave ran 48 windows for an average of 21), and
// requesting the bases word by word 6.6 ms: the waits of the ordinary words
// also waited for the next turn's.
template <bool kFull>
__global__ void __launch_bounds__(kSplitB, 3) k_split(PieceArgs q) {
    extern __shared__ uint32_t S[];                 // [n0 + 4][kSplitB]; then the group counts
    __shared__ uint64_t red[kSplitB / 64];
    __shared__ uint64_t s_start;
    __shared__ uint32_t s_item, s_n, s_cap, s_next;
    __shared__ uint8_t s_order[kSplitB / 64][kBatch];
    __shared__ uint32_t s_cls[kSplitB / 64][16];
    const uint32_t tid = threadIdx.x, lane = __lane_id(), wave = tid >> 6;
    const uint32_t k = q.k, m2 = kFull ? 16u : q.m2, w2 = q.w2, n0 = q.n0;
    const uint32_t lead = (k - m2 + 1 - w2) / 2;   // m2-mers before the middle ones
    const uint32_t n_items = (uint32_t)q.scal[kScalItems], descs = (uint32_t)q.scal[kScalDescs];
    const uint32_t cmask = 0xFFFFFFFFu << (32 - 2 * m2);   // codes are held left-aligned
    const uint32_t hist_cap = q.split_lds / 8;
    // 128-bit loads of a turn: words of 16 bases for all its steps and one more
    // (and one before), one for the funnel and one for the odd half
    const uint32_t quads = ((n0 + w2 + 14) / 16 + (kFull ? 1 : 2) + 2 + 3) / 4;
    uint64_t* hist = (uint64_t*)S;
    uint32_t* col = S + tid;
    uint32_t* block = S + n0 * kSplitB + tid;       // minima of the first part's blocks of 16
    for (;;) {
        if (tid == 0) {
            s_item = (uint32_t)add_dev(&q.scal[kScalItem], 1ull);
            s_n = 0;
            s_next = 0;
        }
        __syncthreads();
        const uint32_t item = s_item;
        if (item >= n_items) break;
        const uint64_t t0 = q.stage_clocks ? wall_clock64() : 0;
        const uint32_t b = item_bin(q.item_first, q.n_bins, item);
        const uint64_t d0 = q.bin_off[b] + (uint64_t)(item - q.item_first[b]) * descs;
        const uint64_t d1 = d0 + descs < q.bin_off[b + 1] ? d0 + descs : q.bin_off[b + 1];
        const uint32_t cnt = (uint32_t)(d1 - d0);
        // list slots for the pieces to expect
        uint64_t est = 0;
#pragma unroll 8
        for (uint32_t j = tid; j < cnt; j += kSplitB) {
            const uint32_t n = (uint32_t)(q.desc[d0 + j] & 0xFFFFFFull);
            est += (uint64_t)((n + n0 - 1) / n0) * 65536ull + (uint64_t)n * q.piece_fx;
        }
        for (int off = 32; off > 0; off >>= 1) est += __shfl_xor(est, off);
        if (lane == 0) red[wave] = est;
        __syncthreads();
        if (tid == 0) {
            uint64_t e = 0;
            for (uint32_t i = 0; i < kSplitB / 64; i++) e += red[i];
            e >>= 16;
            e += e / 16 + kItemSlack;
            const uint64_t at = add_dev(&q.scal[kScalList], e);
            s_start = at;
            s_cap = at + e <= q.cap && e < 0x7FFFFFFFull ? (uint32_t)e : 0u;
        }
        __syncthreads();
        const uint32_t cap = s_cap;
        uint64_t* out = q.list + s_start;
        // The wave's batch of descriptors and the one after it, one register a
        // lane for each 64; pos: how many of the batch are taken, in s_order's order
        const uint32_t batch = cnt >= kSplitB / 64 * kBatch ? kBatch : (cnt / (kSplitB / 64) / 64 + 1) * 64;   // every wave its share of a small item
        uint64_t d[kBatch / 64], d2[kBatch / 64];
        uint32_t pos = batch, left2 = 0;   // left2: descriptors in d2 (0: none left)
        auto request = [&]() {
            uint32_t c0 = 0;
            if (lane == 0) c0 = atomicAdd(&s_next, batch);
            c0 = uniform(c0);
            left2 = c0 < cnt ? cnt - c0 : 0u;
#pragma unroll
            for (uint32_t r = 0; r < kBatch / 64; r++) {
                const uint32_t i = c0 + 64 * r + lane;
                d2[r] = i < cnt && 64 * r < batch ? q.desc[d0 + i] : 0ull;
            }
        };
        // the next batch becomes the current one, longest super-mers first
        auto next_batch = [&]() {
            uint32_t* cls = s_cls[wave];
            if (lane < 16) cls[lane] = 0;
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            uint32_t c[kBatch / 64], rank[kBatch / 64];
#pragma unroll
            for (uint32_t r = 0; r < kBatch / 64; r++) {
                d[r] = d2[r];
                const uint32_t n = (uint32_t)(d[r] & 0xFFFFFFull);
                const uint32_t len = n <= n0 ? n >> 3 : 7 + n / n0 < 15 ? 7 + n / n0 : 15;
                c[r] = 15 - len;
                rank[r] = atomicAdd(&cls[c[r]], 1u);
            }
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            const uint32_t m = lane < 16 ? cls[lane] : 0u, first = wave_incl_sum(m) - m;
#pragma unroll
            for (uint32_t r = 0; r < kBatch / 64; r++) {
                const uint32_t at = __builtin_amdgcn_ds_bpermute((int)(4 * c[r]), (int)first) + rank[r];
                s_order[wave][at] = (uint8_t)(64 * r + lane);
            }
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            pos = 0;
        };
        // A lane's next windows: nx windows from base x of the same super-mer,
        // or if there are none the batch's next one; the first bases are requested
        uint64_t x0 = 0;
        uint32_t n = 0;
        BasesAhead ahead{};
        Words words;   // from base x0 + lead on, or for a shorter m2-mer 16 bases before it
        auto take = [&](uint64_t x, uint32_t nx, uint64_t& to_x, uint32_t& to_n, BasesAhead& f) {
            const uint64_t idle = __ballot(nx == 0);
            if (idle == ~0ull && pos >= batch && left2) {
                next_batch();
                request();
            }
            if (idle && pos < batch) {
                uint32_t at = pos + (uint32_t)__popcll(idle & ((1ull << lane) - 1ull));
                const bool got = nx == 0 && at < batch;
                const uint32_t e = s_order[wave][at < batch ? at : 0];
                uint32_t lo = 0, hi = 0;
#pragma unroll
                for (uint32_t s = 0; s < kBatch / 64; s++) {
                    const uint32_t l = __builtin_amdgcn_ds_bpermute((int)(4 * e), (int)(uint32_t)d[s]);
                    const uint32_t h = __builtin_amdgcn_ds_bpermute((int)(4 * e), (int)(uint32_t)(d[s] >> 32));
                    lo = e >> 6 == s ? l : lo;
                    hi = e >> 6 == s ? h : hi;
                }
                if (got) {
                    x = ((uint64_t)hi << 8) | (lo >> 24);
                    nx = lo & 0xFFFFFFu;
                    if (nx && x + nx - 1 + k > q.n_bytes) {   // a corrupt descriptor must not read out of range
                        set_status(q.status, ST_SPIN);
                        nx = 0;
                    }
                    x = nx ? x : 0ull;
                }
                pos += (uint32_t)__popcll(idle);
            }
            to_x = x;
            to_n = nx;
            f.request(q.packed, (int64_t)(x + lead) - (kFull ? 0 : 16), q.n_bytes, quads);
        };
        if (cap) {
            request();
            take(0, 0, x0, n, ahead);
            ahead.cut(words, quads);
        }
        while (cap) {
            if (__ballot(n > 0) == 0ull) {   // only empty descriptors were taken, or nothing is left
                if (pos >= batch && left2 == 0) break;
                take(0, 0, x0, n, ahead);
                ahead.cut(words, quads);
                continue;
            }
            uint64_t x_nxt = 0;
            uint32_t n_nxt = 0;
            const uint32_t ns = n <= n0 ? n : n <= 2 * n0 ? (n + 1) / 2 : n0;
            const uint32_t nm = wave_max(ns);
            // the m2 bases of a reverse complement end where the code's begin: 16 - m2 bases earlier
            uint32_t A = words[kFull ? 0 : 1];
            uint32_t R = revcomp16(kFull ? A : funnel(words[0], A, 32 - 2 * m2));
            col[(nm - 1) * kSplitB] = 0xFFFFFFFFu;   // the last window holds none of the first part
            uint32_t mid = 0xFFFFFFFFu, pre = 0xFFFFFFFFu, carry = 0, prev = 0;
            uint64_t cuts = 1;
            bool begun = false;   // uniform: the first part and the shared one are done
            for (uint32_t p0 = 0; p0 < nm + w2 - 1; p0 += 16) {
                const uint32_t An = words[(p0 >> 4) + (kFull ? 1 : 2)];
                const uint32_t Rn = revcomp16(kFull ? An : funnel(A, An, 32 - 2 * m2));
                uint32_t h[16];
#pragma unroll
                for (uint32_t j = 0; j < 16; j++) {
                    uint32_t fw = j ? funnel(A, An, 32u - 2u * j) : A;
                    uint32_t rc = j ? funnel(Rn, R, 2u * j) : R;
                    if (!kFull) {
                        fw &= cmask;
                        rc &= cmask;
                    }
                    const uint32_t c = fw < rc ? fw : rc;
                    h[j] = __umul24(c, 0x9E3779u) + (c ^ 0x5bd1e995u);
                }
                A = An;
                R = Rn;
                // the next turn's first bases travel while this one goes on
                if (p0 == 0) take(x0 + ns, n - ns, x_nxt, n_nxt, ahead);
                const uint32_t f = p0 + 1 >= nm ? 0u : nm - 1 - p0 < 16 ? nm - 1 - p0 : 16u;   // positions of the first part
                const uint32_t t = p0 >= w2 ? 0u : w2 - p0 < 16 ? w2 - p0 : 16u;               // first of the last part
                if (f) {
                    uint32_t run = 0xFFFFFFFFu;
#pragma unroll
                    for (int j = 15; j >= 0; j--) {
                        if ((uint32_t)j < f) {
                            run = min(run, h[j]);
                            col[(p0 + j) * kSplitB] = run;
                        }
                    }
                    block[(p0 >> 4) * kSplitB] = run;
                }
                if (f == 0 && t == 16) {
#pragma unroll
                    for (uint32_t j = 0; j < 16; j++) mid = min(mid, h[j]);
                } else {
#pragma unroll
                    for (uint32_t j = 0; j < 16; j++)
                        if (j >= f && j < t) mid = min(mid, h[j]);
                }
                if (t == 16) continue;
                if (!begun) {
                    begun = true;
                    // minima of everything after a block of the first part, the shared part included
                    uint32_t run = mid;
                    for (int c = (int)((nm - 1) >> 4); c >= 0; c--) {
                        const uint32_t m = (uint32_t)c * 16 < nm - 1 ? block[c * kSplitB] : 0xFFFFFFFFu;
                        block[c * kSplitB] = run;
                        run = min(run, m);
                    }
                    prev = run;
                    col[0] = run;   // window 0
                    carry = block[0];
                }
                uint32_t bits = 0;
#pragma unroll
                for (uint32_t j = 0; j < 16; j++) {
                    const uint32_t i = p0 + j + 1 - w2;   // (wraps below the last part)
                    if (j >= t && i < nm) {
                        if ((i & 15u) == 0) carry = block[(i >> 4) * kSplitB];
                        pre = min(pre, h[j]);
                        const uint32_t v = min(min(pre, carry), col[i * kSplitB]);
                        col[i * kSplitB] = v;
                        bits |= v != prev ? 1u << j : 0u;
                        prev = v;
                    }
                }
                const int32_t i0 = (int32_t)(p0 + 1) - (int32_t)w2;
                cuts |= i0 >= 0 ? (uint64_t)bits << i0 : (uint64_t)(bits >> -i0);
            }
            if (!begun) col[0] = mid;   // one window only
            ahead.cut(words, quads);   // (before the stores, which nothing has to wait for)
            // the lane's pieces
            cuts = ns ? cuts & (~0ull >> (64 - ns)) : 0ull;
            const uint32_t np = (uint32_t)__popcll(cuts);
            const uint32_t incl = wave_incl_sum(np);
            uint32_t at = 0;
            if (lane == 63) at = atomicAdd(&s_n, incl);
            at = (uint32_t)__builtin_amdgcn_readlane((int)at, 63) + incl - np;
            while (__ballot(cuts != 0ull) != 0ull) {
                if (cuts) {
                    const uint32_t i = (uint32_t)__builtin_ctzll(cuts);
                    cuts &= cuts - 1;
                    const uint32_t e = cuts ? (uint32_t)__builtin_ctzll(cuts) : ns;
                    const uint32_t v = col[i * kSplitB];
                    const uint32_t hh = ((v ^ (v >> 15)) * 0x85EBCA6Bu) >> (32 - kSubHashBits);
                    if (at < cap) out[at] = ((x0 + i) << 24) | ((uint64_t)hh << 6) | (e - i - 1);
                    at++;
                }
            }
            x0 = x_nxt;
            n = n_nxt;
        }
        __syncthreads();
        const uint32_t total = s_n;
        const bool fits = cap && total <= cap;
        if (tid == 0) {
            q.item_start[item] = s_start;
            q.item_n[item] = fits ? total : 0u;
            if (!fits && cnt) __hip_atomic_store(&q.bin_fail[b], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        const uint32_t P = q.ngrp[b], gb = q.grp_first[b];
        if (fits && P <= hist_cap) {
            for (uint32_t i = tid; i < P; i += kSplitB) hist[i] = 0;
            __syncthreads();
            for (uint32_t e0 = tid; e0 < total; e0 += 8 * kSplitB) {
                uint64_t p[8];
#pragma unroll
                for (uint32_t j = 0; j < 8; j++) p[j] = e0 + j * kSplitB < total ? out[e0 + j * kSplitB] : 0ull;
#pragma unroll
                for (uint32_t j = 0; j < 8; j++)
                    if (e0 + j * kSplitB < total)
                        atomicAdd((unsigned long long*)&hist[group_of_hash(piece_hash(p[j]), P)],
                                  (1ull << 32) | (unsigned long long)piece_kmers(p[j]));
            }
            __syncthreads();
            for (uint32_t i = tid; i < P; i += kSplitB)
                if (hist[i]) add_dev(&q.grp_cnt[gb + i], hist[i]);
        } else if (fits) {
            for (uint32_t e = tid; e < total; e += kSplitB) {
                const uint64_t p = out[e];
                add_dev(&q.grp_cnt[gb + group_of_hash(piece_hash(p), P)], (1ull << 32) | (uint64_t)piece_kmers(p));
            }
        }
        __syncthreads();
        if (q.stage_clocks && tid == 0) {
            add_dev(&q.stage_clocks[0], wall_clock64() - t0);
            add_dev(&q.stage_clocks[4], 1ull);
        }
    }
}

// One workgroup per bin: its groups to sub-tables, runs of pieces for the
// sub-tables from the bottom of pieces and for the heavy groups from its top,
// and the bin's fallback descriptors. A group's weight is the larger of its
// shares of a sub-table's k-mers and bases; a group belongs to the sub-table
// that the middle of its weight falls into.
__global__ void __launch_bounds__(kScanB) k_sub_scan(PieceArgs q) {
    __shared__ uint32_t wsum[32];
    __shared__ uint64_t wsum64[32];
    __shared__ uint64_t s_light, s_heavy, s_hk;
    __shared__ uint32_t s_nh, s_tab, s_fail;
    const uint32_t tid = threadIdx.x, b = blockIdx.x;
    const uint64_t t0 = q.stage_clocks ? wall_clock64() : 0;
    const uint32_t P = q.ngrp[b], gb = q.grp_first[b];
    auto leave_whole = [&]() {   // (one thread) the bin to the fallback
        const uint64_t d0 = q.bin_off[b], nd = q.bin_off[b + 1] - d0;
        q.fb_ptr[b] = (uint64_t)(q.desc + d0);
        q.fb_n[b] = nd;
        q.fb_kmers[b] = q.bin_kmers[b];
        if (nd) add_dev(&q.scal[kScalFallback], 1ull);
    };
    if (q.bin_fail[b]) {
        if (tid == 0) leave_whole();
        return;
    }
    const uint32_t target = (uint32_t)q.scal[kScalTarget];
    auto heavy = [&](uint64_t c) { return group_heavy(q, c); };
    auto weight = [&](uint64_t c) { return group_weight(q, target, c); };
    if (tid == 0) s_hk = 0, s_nh = 0;
    const uint32_t per = (P + kScanB - 1) / kScanB;
    const uint32_t i0 = tid * per, i1 = i0 + per < P ? i0 + per : P;
    uint32_t nl = 0, nh = 0;
    uint64_t w = 0, hk = 0;
    for (uint32_t i = i0; i < i1; i++) {
        const uint64_t c = q.grp_cnt[gb + i];
        if (heavy(c)) {
            nh += (uint32_t)(c >> 32);
            hk += (uint32_t)c;
        } else {
            nl += (uint32_t)(c >> 32);
            w += weight(c);
        }
    }
    uint32_t tl;
    uint64_t tw;
    const uint32_t pl = block_excl_scan(nl, wsum, tl);
    if (nh) atomicAdd(&s_nh, nh);
    uint64_t wr = block_excl_scan(w, wsum64, tw);
    const uint32_t th = s_nh;
    const uint32_t nt = tl ? bin_tables(tw) : 0u;
    if (hk) atomicAdd((unsigned long long*)&s_hk, (unsigned long long)hk);
    if (tid == 0) {
        const uint64_t tab = nt ? add_dev(&q.scal[kScalTables], (uint64_t)nt) : 0ull;
        s_tab = (uint32_t)tab;
        s_fail = tab + nt > q.tab_cap;
        if (s_fail) {
            q.bin_fail[b] = 1;
            leave_whole();
        } else {
            s_light = tl ? add_dev(&q.scal[kScalLight], (uint64_t)tl) : 0ull;
            s_heavy = th ? q.cap - add_dev(&q.scal[kScalHeavy], (uint64_t)th) - th : 0ull;
        }
    }
    __syncthreads();
    if (s_fail) return;
    const uint32_t tab = s_tab;
    uint64_t at = s_light + pl;
    // the groups of one sub-table that this thread has seen
    uint32_t cur = 0xFFFFFFFFu;
    uint64_t cnt = 0, first = 0;
    auto flush = [&]() {
        if (cnt) {
            add_dev(&q.tab_cnt[tab + cur], cnt);
            __hip_atomic_fetch_min(&q.tab_off[tab + cur], first, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        cnt = 0;
    };
    for (uint32_t i = i0; i < i1; i++) {
        const uint64_t c = q.grp_cnt[gb + i];
        const uint32_t np = (uint32_t)(c >> 32);
        if (heavy(c)) {
            q.grp_tab[gb + i] = nt;
            continue;
        }
        const uint32_t gw = weight(c);
        const uint32_t t = np ? table_of_group(wr, gw, nt) : 0u;
        q.grp_tab[gb + i] = t;
        if (np) {
            if (t != cur) {
                flush();
                cur = t;
                first = at;
            }
            cnt += c;
            at += np;
        }
        wr += gw;
    }
    flush();
    if (tid == 0) {
        q.tab_first[b] = tab;
        q.ntab[b] = nt;
        q.heavy_off[b] = s_heavy;
        q.heavy_cur[b] = 0;
        q.fb_ptr[b] = (uint64_t)(q.pieces + s_heavy);
        q.fb_n[b] = th;
        q.fb_kmers[b] = s_hk;
        if (th) add_dev(&q.scal[kScalFallback], 1ull);
        if (q.stage_clocks) {
            add_dev(&q.stage_clocks[1], wall_clock64() - t0);
            add_dev(&q.stage_clocks[5], 1ull);
        }
    }
}

// Every item's pieces to their sub-tables' runs: counted per sub-table in
// LDS, one reservation per sub-table and item, then placed. Bound by the
// scattered 8-byte stores: 150 M pieces at k = 65 take 1.6 ms, with eight
// pieces requested at a time (one at a time: 2.1 ms).
__global__ void __launch_bounds__(kScatB) k_piece_scatter(PieceArgs q) {
    __shared__ uint32_t pos[kScatTabs + 1];       // counts, then places; the last one used: the bin's heavy pieces
    __shared__ uint16_t map[kScatGroups];
    const uint32_t tid = threadIdx.x;
    const uint32_t n_items = (uint32_t)q.scal[kScalItems];
    for (uint32_t item = blockIdx.x; item < n_items; item += gridDim.x) {
        const uint32_t b = item_bin(q.item_first, q.n_bins, item);
        const uint32_t total = q.item_n[item];
        if (total == 0 || q.bin_fail[b]) continue;
        const uint64_t t0 = q.stage_clocks ? wall_clock64() : 0;
        const uint64_t* in = q.list + q.item_start[item];
        const uint32_t P = q.ngrp[b], gb = q.grp_first[b], tb = q.tab_first[b], nt = q.ntab[b];
        if (P <= kScatGroups && nt <= kScatTabs && q.cap < 1ull << 32) {
            for (uint32_t i = tid; i < P; i += kScatB) map[i] = (uint16_t)q.grp_tab[gb + i];
            for (uint32_t i = tid; i <= nt; i += kScatB) pos[i] = 0;
            __syncthreads();
            for (uint32_t e0 = tid; e0 < total; e0 += 8 * kScatB) {
                uint64_t p[8];
#pragma unroll
                for (uint32_t j = 0; j < 8; j++) p[j] = e0 + j * kScatB < total ? in[e0 + j * kScatB] : 0ull;
#pragma unroll
                for (uint32_t j = 0; j < 8; j++)
                    if (e0 + j * kScatB < total) atomicAdd(&pos[map[group_of_hash(piece_hash(p[j]), P)]], 1u);
            }
            __syncthreads();
            for (uint32_t i = tid; i <= nt; i += kScatB) {
                const uint32_t n = pos[i];
                if (n == 0) continue;
                pos[i] = i < nt ? (uint32_t)q.tab_off[tb + i] + add_dev(&q.tab_cur[tb + i], n)
                                : (uint32_t)q.heavy_off[b] + add_dev(&q.heavy_cur[b], n);
            }
            __syncthreads();
            for (uint32_t e0 = tid; e0 < total; e0 += 8 * kScatB) {
                uint64_t p[8];
#pragma unroll
                for (uint32_t j = 0; j < 8; j++) p[j] = e0 + j * kScatB < total ? in[e0 + j * kScatB] : 0ull;
#pragma unroll
                for (uint32_t j = 0; j < 8; j++) {
                    if (e0 + j * kScatB >= total) break;
                    const uint32_t t = map[group_of_hash(piece_hash(p[j]), P)], at = atomicAdd(&pos[t], 1u);
                    const bool heavy = t >= nt;
                    if (at < q.cap) q.pieces[at] = heavy ? (piece_start(p[j]) << 24) | piece_kmers(p[j]) : p[j];
                }
            }
            __syncthreads();
        } else {
            for (uint32_t e = tid; e < total; e += kScatB) {
                const uint64_t p = in[e];
                const uint32_t t = q.grp_tab[gb + group_of_hash(piece_hash(p), P)];
                const bool heavy = t >= nt;
                // (heavy pieces all go to one place: one add for those of a wave)
                const uint64_t hm = __ballot(heavy);
                uint32_t h = 0;
                if (hm) {
                    const int first = __builtin_ctzll(hm);
                    if ((int)__lane_id() == first) h = add_dev(&q.heavy_cur[b], (uint32_t)__popcll(hm));
                    h = __shfl(h, first) + (uint32_t)__popcll(hm & ((1ull << __lane_id()) - 1ull));
                }
                const uint64_t at = heavy ? q.heavy_off[b] + h : q.tab_off[tb + t] + add_dev(&q.tab_cur[tb + t], 1u);
                if (at < q.cap) q.pieces[at] = heavy ? (piece_start(p) << 24) | piece_kmers(p) : p;
            }
        }
        if (q.stage_clocks && tid == 0) {
            add_dev(&q.stage_clocks[2], wall_clock64() - t0);
            add_dev(&q.stage_clocks[6], 1ull);
        }
    }
}

hipError_t launch_piece_plan(const PieceArgs& q, uint64_t* zero_scalars, uint64_t* zero_hist, hipStream_t s) {
    const uint64_t blocks = ((uint64_t)q.grp_cap + kPlanB - 1) / kPlanB;
    const uint32_t g = 1 + (uint32_t)(blocks < 64 ? 64 : blocks > 512 ? 512 : blocks);
    hipLaunchKernelGGL(k_piece_plan, dim3(g), dim3(kPlanB), 0, s, q, zero_scalars, zero_hist);
    return hipGetLastError();
}

constexpr uint32_t kSplitStatic = kSplitB / 64 * (kBatch + 64) + 256;   // static LDS of the split kernel, rounded up

hipError_t launch_split(const PieceArgs& q, uint32_t cus, hipStream_t s) {
    const void* f = q.m2 == 16 ? (const void*)k_split<true> : (const void*)k_split<false>;
    hipError_t e = hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, (int)q.split_lds);
    if (e != hipSuccess) return e;
    uint32_t per_cu = 160u * 1024u / (q.split_lds + kSplitStatic);   // items are popped: more workgroups than fit would only wait
    per_cu = per_cu < 1 ? 1 : per_cu > 6 ? 6 : per_cu;
    if (q.m2 == 16) hipLaunchKernelGGL(k_split<true>, dim3(cus * per_cu), dim3(kSplitB), q.split_lds, s, q);
    else hipLaunchKernelGGL(k_split<false>, dim3(cus * per_cu), dim3(kSplitB), q.split_lds, s, q);
    return hipGetLastError();
}

hipError_t launch_sub_scan(const PieceArgs& q, hipStream_t s) {
    hipLaunchKernelGGL(k_sub_scan, dim3(q.n_bins), dim3(kScanB), 0, s, q);
    return hipGetLastError();
}

hipError_t launch_piece_scatter(const PieceArgs& q, uint32_t cus, hipStream_t s) {
    hipLaunchKernelGGL(k_piece_scatter, dim3(cus * 4), dim3(kScatB), 0, s, q);
    return hipGetLastError();
}

}  // namespace gerbil
