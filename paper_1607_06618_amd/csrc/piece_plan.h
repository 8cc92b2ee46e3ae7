// Sizes and rules of the piece partition (pieces.h): how large its arrays are
// (host), and how the plan and the scan cut bins into groups and sub-tables
// (device). All of it is integer arithmetic on a few numbers, in functions that
// the host can run too, so that the bounds that the kernels rely on can be
// checked without a GPU.
#pragma once
#include <algorithm>

#include "../../include/gerbil.h"
#include "common.h"
#include "pieces.h"

namespace gerbil {

// ------------------------------------------------------------ which calls
constexpr uint64_t kShortKeyBin = 16ull << 20;   // bases per bin

// PLAIN takes the pieces too where AUTO leaves the partition to the library
// and nothing asks for the key partition's sampled run sizes: a group of bins
// at a time, as many as their pieces fit in the workspace. Four launches per
// bin left most of the chip idle: 256 bins of 0.3 M 55-mers took 23.2 ms, in
// groups 2.5 ms.
inline bool use_pieces(const gerbil_params* p, uint64_t n_bytes) {
    if (p->k < kPieceMinK || p->n_bins == 0 || n_bytes >= (1ull << 38)) return false;
    // Short keys have few sub-minimizers (4^10 or 4^11 at k < 24, and the smallest
    // dozenth of those takes most k-mers): in a large bin each brings more than a
    // sub-table's. 1.2 G bases at k = 21 in 32 bins: 65 ms by pieces, 41 by key
    // hash; 0.3 G in 32 bins 7.7 and 9.2 ms, 1.2 G in 512 bins 28.8 and 36.1 ms.
    if (p->k < 24 && n_bytes / p->n_bins > kShortKeyBin) return false;
    if (p->mode == GERBIL_BATCHED) return p->table != GERBIL_TABLE_HBM;
    return p->table == GERBIL_TABLE_AUTO && (p->k + 31) / 32 <= GERBIL_MAX_LDS_W && p->size_sample == 0;
}

// ------------------------------------------------------------ work items
constexpr uint32_t kSplitB = 256;          // threads of the split kernel
constexpr uint32_t kItemDescs = 4096;      // descriptors per item at most (at least 256); 8192 and 2048 are 1 % slower
// Where the bins have more than kManyGroups groups on average, an item of 4096
// descriptors has about one piece for each, and every piece is an atomic of its
// own: 0.6 G bases at k = 28 in 32 bins took 17.7 ms, now 10.3 ms (14.2 by key hash).
constexpr uint32_t kItemDescsMany = 16384;
constexpr uint32_t kManyGroups = 3500;
// Items of a PLAIN group, or of all bins: 2048, which even out their lengths.
// An item adds its counts to its bin's groups and reserves places in its
// sub-tables one by one, so of few super-mers each item gets 1024, as long as
// that leaves one for each of the split kernel's three workgroups a CU: a PLAIN
// pass over 125 M bases at k = 55 takes 2.54 ms with 512 items a group, 2.51
// with 768, 2.60 with 1024 and 2.82 with 2048; 100 M bases at k = 28, where the
// rule makes no difference to 768, 3.29 / 2.97 / 3.23 / 3.50 ms.
constexpr uint32_t kItemGoal = 2048;
constexpr uint32_t kItemFew = 768, kItemFewDescs = 1024;
constexpr uint32_t kItemSlack = 64;        // list slots of an item over its expected pieces
constexpr uint32_t kMinTarget = 1024;      // k-mers of a small input's sub-tables
constexpr uint32_t kUnit = 4096;           // weight of a full sub-table
constexpr uint32_t kLargeGroup = kUnit * 26 / 100;

// Descriptors per item, for S super-mers in all.
__host__ __device__ inline uint32_t item_descs(uint64_t S, bool many) {
    const uint64_t few = S / kItemFew < kItemFewDescs ? S / kItemFew : kItemFewDescs, most = many ? kItemDescsMany : kItemDescs;
    uint64_t d = S / kItemGoal > few ? S / kItemGoal : few;
    d = (d + 63) & ~63ull;
    return (uint32_t)(d < 256 ? 256 : d > most ? most : d);
}
inline uint32_t piece_items_cap(uint64_t n_superm, uint32_t n_bins) {
    return (uint32_t)(n_superm / kItemDescs + 2 * kItemGoal + n_bins + 8);
}
// List slots for this many super-mers and k-mers.
// `cut`: super-mers of more than n0 k-mers are to be expected.
inline uint64_t piece_list_slots(uint64_t n_superm, uint64_t kmers, uint32_t piece_fx, uint32_t n0, bool cut,
                                 uint32_t n_bins) {
    // a super-mer of n k-mers takes ceil(n / n0) lanes' turns: at most one more for every n0 k-mers
    const uint64_t e = n_superm + ((kmers * piece_fx) >> 16) + (cut ? kmers / n0 : 0);
    return e + e / 16 + (uint64_t)kItemSlack * piece_items_cap(n_superm, n_bins);
}
// Dynamic LDS of the split kernel.
inline uint32_t split_lds_bytes(uint32_t n0) {
    const uint32_t rows = (n0 + 4) * kSplitB * 4;
    return rows < 36864u ? 36864u : rows;   // (also the counts of up to bytes / 8 groups: at least kExactGroups)
}

// ----------------------------------------------------------------- sizes
// K-mers per slot; sub-tables are cut to within a group's size of it. 0.6
// costs 1 to 3 % (more sub-tables, each with its scan and dump), and 0.8 as much
// where probes get longer: passes of 26.8 / 26.8 / 27.5 ms for 0.8 / 0.7 / 0.6 at
// k = 65, 19.8 / 19.6 / 19.8 at k = 99, 9.20 / 9.10 / 9.18 at k = 28.
constexpr double kPieceFill = 0.7;
// Sub-tables wanted at least: one per CU. Small inputs get smaller ones for
// it. Two or more per CU even out their ends, but cost more fixed time each: 2 M
// bases at k = 55 take 191 us with one, 203 with two and 226 with four.
constexpr uint32_t kTablesGoal = 256;

struct PieceSizing {
    uint32_t block, C, target, half_target, max_kmers, slice_kmers, heavy_kmers, max_halves;
    uint32_t m2, n0, split_lds, piece_fx, items_cap;
    uint64_t grp_cap, tab_cap;
};

// For groups of bins with up to n_kmers k-mers in up to n_superm super-mers.
inline PieceSizing piece_sizing(const gerbil_params* p, uint64_t n_kmers, uint64_t n_superm) {
    PieceSizing z;
    // One workgroup of 1024 threads per CU or two of 512: the single large
    // table wastes less on the spread of group sizes and on dumps (count step
    // of 1.7 G 65-mer windows 24.5 ms against 27.6 ms; 28-mers 8.9 / 9.7, 200-mers
    // 8.5 / 9.1). Beyond k = 256 a thread of 1024 has too few registers for the
    // key's two strands.
    z.block = p->block == 512 || p->k > 256 ? 512u : 1024u;
    z.m2 = sub_minimizer_len(p->k);
    const uint32_t w2 = sub_window(p->k, z.m2), w = p->k - p->m + 1;
    // The LDS left by the fixed parts holds the staged bases and the slots. A
    // piece has about 0.8 / (2 / (w2 + 1) + 2 / (w + 1)) k-mers (cuts of either
    // minimizer, and read ends). The bases get half as much again as that, so
    // that the k-mers are what fills a sub-table, and 1.3 times their target
    // fits: a sub-table is cut to within a group's size.
    const double per_kmer = (2.0 / (w2 + 1) + 2.0 / (w + 1)) / 0.8;
    const double halves = std::min(p->k / 16.0 + 2.0, (1.0 + per_kmer * (p->k + 29)) / 16.0);
    const double pool = z.block == 1024 ? SubShape<1024>::pool : SubShape<512>::pool;
    const double n = pool / (8.0 / kPieceFill + 4.0 * 1.5 * halves);
    z.max_halves = 4 * (uint32_t)(1.5 * halves * n / 4.0);
    // whole rounds of the workgroup's threads over the slots; what that leaves goes to the bases
    uint32_t nb = ((uint32_t)pool - 4 * z.max_halves) / (8 * z.block) * z.block / 2;
    z.max_halves = ((uint32_t)pool - 16 * nb) / 16 * 4;
    for (;; nb--) {   // a prime number of buckets, so that double hashing has a full period
        bool prime = true;
        for (uint32_t d = 2; prime && d * d <= nb; d++) prime = nb % d != 0;
        if (prime) break;
    }
    z.C = 2 * nb;
    z.half_target = std::max<uint32_t>(1u, (uint32_t)(z.max_halves / 1.3));
    const double fill = p->load_factor > 0 ? p->load_factor : kPieceFill;
    z.target = std::min<uint32_t>(40000u, std::max<uint32_t>(64u, (uint32_t)(z.C * fill)));
    z.max_kmers = std::max<uint32_t>((uint32_t)(0.93 * z.C), z.target + z.target / 4);
    z.slice_kmers = std::max<uint32_t>((uint32_t)(0.75 * z.C), z.target);
    // counts are 16 bits wide; more than four tables' worth goes to the fallback
    z.heavy_kmers = std::min<uint32_t>(60000u, std::max<uint32_t>(4 * z.C, z.target + z.target / 2));
    // A turn of n windows costs n + w2 - 1 m2-mers, so long turns do less work a
    // window, but their minima take the LDS that more workgroups would need.
    // Whole passes with 32 / 40 / 48 / 64 windows at most: k = 99 19.9 / 19.6 /
    // 19.5 / 19.9 ms, k = 200 8.87 / 8.96 / 9.22 / 9.22 ms, k = 479 3.07 / 2.96 /
    // 2.91 / 2.87 ms. (Narrow windows: super-mers are seldom longer than 48.)
    // Of the last 16, the number with the most windows per step of 16 m2-mers.
    const uint32_t n_most = std::min(w2 >= kPieceMax ? 40u : 48u, w2);
    z.n0 = n_most;
    for (uint32_t n = n_most > 15 ? n_most - 15 : 1; n < n_most; n++)
        if (n * ((z.n0 + w2 + 14) / 16) > z.n0 * ((n + w2 + 14) / 16)) z.n0 = n;
    z.split_lds = split_lds_bytes(z.n0);
    // random sub-minimizers change every (w2 + 1) / 2 windows
    z.piece_fx = (uint32_t)(65536.0 * 2.15 / (w2 + 1));
    z.items_cap = piece_items_cap(n_superm, p->n_bins);
    // the number of a large bin's groups is rounded up to a power of two
    const uint64_t E = n_superm + n_kmers / z.n0 + ((n_kmers * z.piece_fx) >> 16);   // (never less than the plan's bins add up to)
    const uint64_t tabs = n_kmers / z.target + piece_halves(n_kmers, E, p->k) / z.half_target + kTablesGoal;
    z.grp_cap = 2 * kGroupsPerTable * tabs + 2ull * p->n_bins;
    // Sub-tables: no more than the groups' weights add up to (group_weight), for
    // as many pieces as the items' list slots take: the k-mers' share, twice that
    // of the bases, and what is rounded up for every group and bin. (A plan with
    // a smaller target makes at most tables_goal of them.)
    const uint64_t most = piece_list_slots(n_superm, n_kmers, z.piece_fx, z.n0, w > z.n0, p->n_bins);
    z.tab_cap = n_kmers / z.target + kTablesGoal + 2 * ((piece_halves(n_kmers, most, p->k) + z.grp_cap) / z.half_target) +
                4 * z.grp_cap / kUnit + 2ull * p->n_bins + 4;
    return z;
}

// -------------------------------------------------- rules of plan and scan
// The sizing's part of the kernels' arguments.
inline void set_rules(PieceArgs& q, const gerbil_params* p, const PieceSizing& z) {
    q.k = p->k;
    q.m2 = z.m2;
    q.w2 = sub_window(p->k, z.m2);
    q.n0 = z.n0;
    q.split_lds = z.split_lds;
    q.target = z.target;
    q.half_target = z.half_target;
    q.max_kmers = z.max_kmers;
    q.slice_kmers = z.slice_kmers;
    q.heavy_kmers = z.heavy_kmers;
    q.max_halves = z.max_halves;
    q.piece_fx = z.piece_fx;
    q.turn_fx = 65536 / z.n0;
    q.tables_goal = p->load_factor > 0 ? 1 : kTablesGoal;   // (a load that is asked for stands)
    q.grp_cap = (uint32_t)std::min<uint64_t>(z.grp_cap, 0xFFFFFFFFull);
    q.tab_cap = (uint32_t)std::min<uint64_t>(z.tab_cap, 0xFFFFFFFFull);
    q.items_cap = z.items_cap;
}

// K-mers per sub-table of a run of `total`: the target, or less where that
// leaves workgroups without one.
__host__ __device__ inline uint64_t plan_target(const PieceArgs& q, uint64_t total) {
    uint64_t target = total / q.tables_goal;
    target = target < kMinTarget ? kMinTarget : target;
    return target > q.target ? q.target : target;
}

// A group's count has 32 bits for its k-mers, and one sub-minimizer can bring all
// of a bin's (tandem repeats): bins of more go to the fallback as a whole. (By
// then their 2^18 groups are too large for LDS tables anyway.)
__host__ __device__ inline bool bin_left_whole(uint64_t K) { return K >> 32 != 0; }

// Pieces to expect from K k-mers in ns super-mers: their sub-minimizers change,
// and a super-mer is split in turns of n0 windows at most: K / n0 of them and
// half a turn more for each where they are long (half of all pieces at k = 479).
__host__ __device__ inline uint64_t expected_pieces(const PieceArgs& q, uint64_t ns, uint64_t K) {
    const uint64_t turns = ns / 2 + ((K * q.turn_fx) >> 16);
    return (turns > ns ? turns : ns) + ((K * q.piece_fx) >> 16);
}

// Groups of a bin of K k-mers in ns super-mers.
__host__ __device__ inline uint32_t bin_groups(const PieceArgs& q, uint64_t target, uint64_t ns, uint64_t K) {
    if (ns == 0) return 0;
    const uint64_t E = expected_pieces(q, ns, K);
    // an eighth of a sub-table each; of large bins more, so that an item's
    // counts of groups and sub-tables fit in LDS
    const uint64_t halves = piece_halves(K, E, q.k);
    const uint64_t Tk = (K + target - 1) / target, Th = (halves + q.half_target - 1) / q.half_target, T = Tk > Th ? Tk : Th;
    uint64_t per = kGroupsPerTable;
    if (T * per > kExactGroups) per = T < kExactGroups ? kExactGroups / T : 1;
    uint64_t P = (K * per + target - 1) / target;
    const uint64_t Ph = (halves * per + q.half_target - 1) / q.half_target;
    if (Ph > P) P = Ph;
    // Where bases are what fills the sub-tables (k above some 130), groups of about
    // one would often be heavy, and keys above 256 bases are then counted in HBM
    // tables: as many groups as LDS counts, and three for two sub-tables at
    // least. 20 M bases at k = 479 in one bin 6.07 -> 1.61 ms, 60 M at k = 300 in
    // four 11.3 -> 2.83 ms, 600 M at k = 200 in 32 10.6 -> 10.5 ms.
    if (Th > Tk && per < kGroupsPerTable) P = 3 * Th / 2 > kExactGroups ? 3 * Th / 2 : kExactGroups;
    if (P > kExactGroups) {
        uint64_t p2 = kExactGroups;
        while (p2 < P && p2 < kMaxGroups) p2 *= 2;
        P = p2;
    }
    return (uint32_t)(P ? P : 1);
}

// A group's count c: pieces << 32 | k-mers. Heavy: more than a workgroup's LDS
// takes even in slices.
__host__ __device__ inline bool group_heavy(const PieceArgs& q, uint64_t c) {
    return (uint32_t)c > q.heavy_kmers || piece_halves((uint32_t)c, c >> 32, q.k) > q.max_halves;
}

// Weight of a group that is not heavy: the larger of its shares of a
// sub-table's k-mers and bases.
__host__ __device__ inline uint32_t group_weight(const PieceArgs& q, uint32_t target, uint64_t c) {
    // Rounded up, and a large group's bases doubled: the groups whose middles
    // fall into one unit then have at most 1 + kLargeGroup units of bases
    // (1.26, where the table holds 1.3): the extents between the first and the
    // last middle add up to a unit, half of the first and half of the last lie
    // outside it, and a large group's bases are at most half of its extent.
    const uint32_t wk = (uint32_t)(((uint64_t)(uint32_t)c * kUnit + target - 1) / target);
    uint32_t wh = (uint32_t)(((piece_halves((uint32_t)c, c >> 32, q.k) + 1) * kUnit + q.half_target - 1) / q.half_target);
    if (c == 0) wh = 0;
    if (wh > kLargeGroup) wh *= 2;
    return wk > wh ? wk : wh;
}

// Sub-tables of a bin whose groups weigh `weight` together, and the one that a
// group of weight w, w0 of weight before it, belongs to: the middle of its
// weight falls into it.
// (A bin can weigh 2^32 and more: 94 M k-mers at a load factor of 0.01.)
__host__ __device__ inline uint32_t bin_tables(uint64_t weight) { return (uint32_t)(weight / kUnit) + 1; }
__host__ __device__ inline uint32_t table_of_group(uint64_t w0, uint32_t w, uint32_t n_tables) {
    const uint32_t t = (uint32_t)((w0 + w / 2) / kUnit);
    return t < n_tables ? t : n_tables - 1;
}

}  // namespace gerbil
