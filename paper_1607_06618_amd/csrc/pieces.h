// Pieces: the batched counter's partition of a bin into sub-tables.
//
// All occurrences of a canonical k-mer lie in one bin (Sec. 2.1). The same
// argument, repeated with a second and longer minimizer, splits a bin further:
// the sub-minimizer of a k-mer is the smallest of its middle canonical m2-mers
// under a hashed order, a piece is a run of consecutive k-mers of one super-mer
// with equal sub-minimizers, and a piece goes to the group its sub-minimizer
// hashes to. A run of groups makes a sub-table, which holds every occurrence
// of its k-mers; what is written to memory and read back is 8 bytes per piece
// (about 11 k-mers at k = 65) where a partition by the hash of the k-mer
// writes every key.
//
// A sub-minimizer brings all the k-mers of its place in the genome (some 400
// at 30x), so sub-tables of a fixed number of hash values differ widely in
// size. Groups are an eighth of a sub-table, and sub-tables are cut from their
// running total: they come out within a few per cent of what the LDS table
// takes.
#pragma once
#include "internal.h"

namespace gerbil {

// A piece: first base (40 bits) | 18 hash bits of the sub-minimizer | k-mers - 1 (6 bits).
constexpr uint32_t kPieceMax = 64;     // k-mers of a piece at most
constexpr uint32_t kSubHashBits = 18;
// Groups of a bin: their number is bounded by the hash bits; above
// kExactGroups it is a power of two, so that every group owns the same number
// of hash values.
constexpr uint32_t kMaxGroups = 1u << kSubHashBits;
constexpr uint32_t kExactGroups = 4096;
constexpr uint32_t kGroupsPerTable = 8;

__host__ __device__ inline uint64_t piece_start(uint64_t p) { return p >> 24; }
__host__ __device__ inline uint32_t piece_kmers(uint64_t p) { return (uint32_t)(p & 63u) + 1u; }
__host__ __device__ inline uint32_t piece_hash(uint64_t p) { return (uint32_t)(p >> 6) & (kMaxGroups - 1u); }
__host__ __device__ inline uint32_t group_of_hash(uint32_t h, uint32_t P) {
    return (uint32_t)(((uint64_t)h * P) >> kSubHashBits);
}

// Sub-minimizer length: 16 (a 32-bit code) for longer keys. Short keys take
// half of k, so that a window still holds about as many m2-mers as it has
// bases left: fewer would cut pieces of one or two k-mers. Below kPieceMinK
// pieces are so short, and sub-minimizers so few, that the keys themselves are
// the cheaper thing to distribute.
constexpr uint32_t kPieceMinK = 20;
inline uint32_t sub_minimizer_len(uint32_t k) { return k >= 32 ? 16u : k / 2; }
// m2-mers the sub-minimizer is taken over: those in the middle of the k-mer
// (the same ones on either strand), at most kMaxSubWindow or one more. All of
// a long key's would make runs of hundreds of k-mers, and a few of those, at
// some coverage, more than a sub-table: its size would spread too far.
constexpr uint32_t kMaxSubWindow = 96;
inline uint32_t sub_window(uint32_t k, uint32_t m2) {
    const uint32_t w = k - m2 + 1;
    return w <= kMaxSubWindow ? w : kMaxSubWindow + ((w - kMaxSubWindow) & 1u);
}

// Workgroup shapes of the table kernel: 512 threads with 80 KB of LDS (two per
// CU), or 1024 with 160 KB.
template <uint32_t B>
struct SubShape {
    static constexpr uint32_t bytes = 160u * B;
    static constexpr uint32_t hist_at = 0;                                  // u32 [kLdsHist]
    static constexpr uint32_t probe_at = 4 * kLdsHist;                      // u32 [kProbeHist]
    static constexpr uint32_t sum_at = probe_at + 4 * kProbeHist;           // u32 [16] pairs of every wave
    static constexpr uint32_t base_at = sum_at + 64;                        // u64 output base
    static constexpr uint32_t cls_at = base_at + 16;                        // u32 [8] segments by length; [0]: half words and full segments
    static constexpr uint32_t segs = 5 * B / 2;
    static constexpr uint32_t seg_at = cls_at + 32;                         // u32 [segs] segments of the round
    static constexpr uint32_t retry_at = seg_at + 4 * segs;                    // u32 [B / 64][retry] k-mers whose first bucket failed
    static constexpr uint32_t retry = 96;
    static constexpr uint32_t bases_at = (retry_at + B / 16 * retry + 31) / 16 * 16;   // u32 [halves], a pad before it
    static constexpr uint32_t pool = bytes - bases_at;                      // bytes of staged bases and slots together
};

// Half words (16 bases) that pieces of `kmers` k-mers in all need at most when
// staged: ((start & 15) + n + k - 1 + 15) / 16 each.
__host__ __device__ inline uint64_t piece_halves(uint64_t kmers, uint64_t pieces, uint32_t k) {
    return (kmers + pieces * (k + 29)) / 16;
}

struct PieceArgs {
    // input
    const uint64_t* packed;
    uint64_t n_bytes;
    const uint64_t* desc;
    const uint64_t* bin_off;
    const uint64_t* bin_kmers;
    const uint64_t* n_superm;
    uint64_t superm_cap;
    uint32_t k, m2, w2, n_bins;   // w2: m2-mers of a window (the middle ones)
    uint32_t* status;
    // sizing
    uint32_t n0;              // windows a lane splits at a time (at most kPieceMax and k - m2 + 1)
    uint32_t split_lds;       // dynamic LDS of the split kernel
    uint32_t target;          // k-mers per sub-table
    uint32_t half_target;     // staged half words (16 bases) per sub-table
    uint32_t tables_goal;     // sub-tables wanted at least: small inputs get smaller ones
    uint32_t max_kmers;       // a sub-table of more is counted in hash slices
    uint32_t slice_kmers;     // k-mers per slice
    uint32_t heavy_kmers;     // a sub-table of more goes to the fallback
    uint32_t max_halves;      // staged half words a sub-table may need
    uint32_t piece_fx;        // expected pieces per k-mer, 16.16 (over the one per super-mer)
    uint32_t turn_fx;         // turns per k-mer of a long super-mer: 65536 / n0
    uint32_t grp_cap, tab_cap, items_cap;
    uint64_t cap;             // pieces that fit in list and in pieces
    // plan
    uint32_t* ngrp;           // [n_bins]
    uint32_t* grp_first;      // [n_bins + 1] first group
    uint32_t* item_first;     // [n_bins + 1] first split item
    uint64_t* scal;           // kScal*
    uint32_t* bin_fail;       // [n_bins] 1: the bin's pieces or sub-tables did not fit, the fallback counts it whole
    // split
    uint64_t* item_start;     // [items_cap] the item's pieces in list
    uint32_t* item_n;         // [items_cap]
    uint64_t* list;           // [cap]
    uint64_t* grp_cnt;        // [grp_cap] pieces << 32 | k-mers
    // scan, scatter
    uint32_t* grp_tab;        // [grp_cap] sub-table of the group, counted from the bin's first
    uint32_t* tab_first;      // [n_bins] first sub-table of the bin
    uint32_t* ntab;           // [n_bins] sub-tables; as a group's sub-table: the group is heavy
    uint64_t* tab_cnt;        // [tab_cap] pieces << 32 | k-mers
    uint64_t* tab_off;        // [tab_cap] first piece in pieces
    uint32_t* tab_cur;        // [tab_cap]
    uint64_t* heavy_off;      // [n_bins] first heavy piece in pieces
    uint32_t* heavy_cur;      // [n_bins]
    uint64_t* pieces;         // [cap] by sub-table; those of heavy groups from the top, as descriptors
    // fallback: descriptors of every bin (heavy pieces, or the whole bin)
    uint64_t* fb_ptr;         // [n_bins] device address of the first
    uint64_t* fb_n;           // [n_bins]
    uint64_t* fb_kmers;       // [n_bins]
    uint64_t* stage_clocks;
};
// scalars
enum { kScalItem = 0, kScalList, kScalLight, kScalHeavy, kScalTables, kScalItems, kScalDescs, kScalFallback,
       kScalTarget, kScalCount };

hipError_t launch_piece_plan(const PieceArgs& q, uint64_t* zero_scalars, uint64_t* zero_hist, hipStream_t s);
hipError_t launch_split(const PieceArgs& q, uint32_t cus, hipStream_t s);
hipError_t launch_sub_scan(const PieceArgs& q, hipStream_t s);
hipError_t launch_piece_scatter(const PieceArgs& q, uint32_t cus, hipStream_t s);

// Table kernel: sub-tables [0, n) of the plan, in LDS tables of `slots` slots.
struct SubArgs {
    const uint64_t* pieces;
    const uint64_t* tab_cnt;
    const uint64_t* tab_off;
    const uint64_t* n_tab;    // scalar: sub-tables handed out, of which tab_cap are there
    uint32_t tab_cap;
    uint32_t buckets;         // of two slots
    uint32_t halves, theta, max_kmers, slice_kmers;
    uint64_t* probe_hist;
    uint64_t* stage_clocks;
};
hipError_t launch_sub_tables(const CountArgs& a, const SubArgs& t, uint32_t block, uint32_t cus, hipStream_t s);

}  // namespace gerbil
