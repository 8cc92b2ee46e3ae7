// The plan and the scan of the piece partition (csrc/piece_plan.h) run on the
// host, over the groups that a sequence's pieces make. Prints one line of
// numbers per run; tests/test_piece_plan.py compares them with the bounds that
// the kernels rely on.
#include <stdio.h>
#include <stdlib.h>
#include <string.h>

#include <vector>

#include "../paper_1607_06618_amd/csrc/piece_plan.h"

using namespace gerbil;

static uint64_t rng_state;
static uint64_t rnd() {   // splitmix64
    uint64_t z = (rng_state += 0x9E3779B97F4A7C15ull);
    z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
    z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
    return z ^ (z >> 31);
}

// Smaller strand's code of every m-mer, left-aligned in 32 bits.
static std::vector<uint32_t> codes(const std::vector<uint8_t>& s, uint32_t m) {
    std::vector<uint32_t> c(s.size() >= m ? s.size() - m + 1 : 0);
    uint64_t fw = 0, rc = 0;
    const uint64_t mask = (1ull << (2 * m)) - 1;
    for (size_t i = 0; i < s.size(); i++) {
        fw = ((fw << 2) | s[i]) & mask;
        rc = (rc >> 2) | ((uint64_t)(3 - s[i]) << (2 * m - 2));
        if (i + 1 >= m) c[i + 1 - m] = (uint32_t)((fw < rc ? fw : rc) << (32 - 2 * m));
    }
    return c;
}

// Minima of all windows of w values.
static std::vector<uint32_t> minima(const std::vector<uint32_t>& v, uint32_t w) {
    std::vector<uint32_t> out(v.size() >= w ? v.size() - w + 1 : 0);
    std::vector<size_t> q(v.size());
    size_t head = 0, tail = 0;
    for (size_t i = 0; i < v.size(); i++) {
        while (tail > head && v[q[tail - 1]] >= v[i]) tail--;
        q[tail++] = i;
        if (q[head] + w <= i) head++;
        if (i + 1 >= w) out[i + 1 - w] = v[q[head]];
    }
    return out;
}

struct Bin {
    uint64_t ns = 0, kmers = 0;
    std::vector<uint64_t> pieces;   // hash << 8 | k-mers
};

// Pieces of one read, as the binning and the split cut them.
static void cut_read(const PieceArgs& q, uint32_t m, uint32_t n_bins, uint64_t pos, const std::vector<uint8_t>& s,
                     std::vector<Bin>& bins) {
    const uint32_t k = q.k, lead = (k - q.m2 + 1 - q.w2) / 2;
    if (s.size() < k) return;
    std::vector<uint32_t> c = codes(s, m), h = codes(s, q.m2);
    for (auto& x : c) x = x * 0x9E3779B1u;   // (any order of the minimizers)
    for (auto& x : h) x = (x & 0xFFFFFFu) * 0x9E3779u + (x ^ 0x5bd1e995u);
    const std::vector<uint32_t> mn = minima(c, k - m + 1), sub = minima(h, q.w2);
    for (size_t i = 0; i < mn.size();) {
        size_t e = i + 1;
        while (e < mn.size() && mn[e] == mn[i] && (pos + e) % 2048 != 0) e++;
        Bin& b = bins[(mn[i] >> (32 - 2 * m)) % n_bins];
        b.ns++;
        b.kmers += e - i;
        while (i < e) {   // turns
            const uint32_t left = (uint32_t)(e - i), n = left <= q.n0 ? left : left <= 2 * q.n0 ? (left + 1) / 2 : q.n0;
            for (uint32_t a = 0; a < n;) {
                uint32_t z = a + 1;
                const uint32_t v = sub[i + a + lead];
                while (z < n && sub[i + z + lead] == v) z++;
                b.pieces.push_back((uint64_t)(((v ^ (v >> 15)) * 0x85EBCA6Bu) >> (32 - kSubHashBits)) << 8 | (z - a));
                a = z;
            }
            i += n;
        }
    }
}

struct Totals {
    uint64_t groups = 0, heavy = 0, tables = 0, failed = 0, kmers = 0, heavy_kmers = 0, pieces = 0, expected = 0, lost = 0;
    uint64_t most_halves = 0, most_kmers = 0;
};

// The scan of one bin over its groups' counts.
static void scan(const PieceArgs& q, uint32_t target, const std::vector<uint64_t>& cnt, Totals& T) {
    uint64_t w = 0;
    for (uint64_t c : cnt) {
        T.groups++;
        T.pieces += c >> 32;
        if (group_heavy(q, c)) {
            T.heavy++;
            T.heavy_kmers += (uint32_t)c;
        } else {
            w += group_weight(q, target, c);
        }
    }
    const uint64_t nt = bin_tables(w);
    T.tables += nt;
    if (T.tables > q.tab_cap) {   // the bin goes to the fallback
        T.failed++;
        return;
    }
    uint64_t w0 = 0, cur = ~0ull, sum = 0;
    auto close = [&]() {
        const uint64_t h = piece_halves((uint32_t)sum, sum >> 32, q.k);
        if (h > T.most_halves) T.most_halves = h;
        if ((uint32_t)sum > T.most_kmers) T.most_kmers = (uint32_t)sum;
        sum = 0;
    };
    for (uint64_t c : cnt) {
        if (group_heavy(q, c)) continue;
        const uint64_t gw = group_weight(q, target, c), t = table_of_group(w0, gw, nt);
        if (c) {
            if (t != cur) {
                if (cur != ~0ull && t < cur) T.lost++;   // a sub-table's groups would not be in one run
                close();
                cur = t;
            }
            sum += c;
        }
        w0 += gw;
    }
    close();
}

static void print(const char* what, const PieceArgs& q, const PieceSizing& z, const Totals& T, uint64_t list) {
    printf("%s tables %llu tab_cap %llu failed %llu groups %llu grp_cap %llu heavy %llu kmers %llu heavy_kmers %llu "
           "pieces %llu expected %llu list %llu most_halves %llu max_halves %u most_kmers %llu lost %llu\n",
           what, (unsigned long long)T.tables, (unsigned long long)z.tab_cap, (unsigned long long)T.failed,
           (unsigned long long)T.groups, (unsigned long long)z.grp_cap, (unsigned long long)T.heavy,
           (unsigned long long)T.kmers, (unsigned long long)T.heavy_kmers, (unsigned long long)T.pieces,
           (unsigned long long)T.expected, (unsigned long long)list, (unsigned long long)T.most_halves, q.max_halves, (unsigned long long)T.most_kmers,
           (unsigned long long)T.lost);
}

// groups <k> <m> <load> <block> <groups> <k-mers> <pieces>: one bin of equal groups
static void groups(char** a) {
    gerbil_params p;
    memset(&p, 0, sizeof(p));
    p.k = atoi(a[0]);
    p.m = atoi(a[1]);
    p.load_factor = (float)atof(a[2]);
    p.block = atoi(a[3]);
    p.n_bins = 1;
    p.mode = GERBIL_BATCHED;
    const uint64_t n = strtoull(a[4], 0, 10), kmers = strtoull(a[5], 0, 10), pieces = strtoull(a[6], 0, 10);
    const PieceSizing z = piece_sizing(&p, n * kmers, n * pieces);
    PieceArgs q;
    memset(&q, 0, sizeof(q));
    set_rules(q, &p, z);
    Totals T;
    T.kmers = n * kmers;
    if (bin_left_whole(T.kmers)) T.failed++;
    else scan(q, (uint32_t)plan_target(q, T.kmers), std::vector<uint64_t>(n, (pieces << 32) + kmers), T);   // (as the split adds up)
    print("groups", q, z, T, 0);
}

// random <k> <load> <block> <seed>: bins of groups of all sizes up to the heavy ones'
static void random_groups(char** a) {
    gerbil_params p;
    memset(&p, 0, sizeof(p));
    p.k = atoi(a[0]);
    p.m = 9;
    p.load_factor = (float)atof(a[1]);
    p.block = atoi(a[2]);
    p.n_bins = 1;
    p.mode = GERBIL_BATCHED;
    rng_state = strtoull(a[3], 0, 10);
    const PieceSizing z = piece_sizing(&p, 1ull << 30, 1ull << 28);
    PieceArgs q;
    memset(&q, 0, sizeof(q));
    set_rules(q, &p, z);
    Totals T;
    auto unit = []() { return (double)(rnd() >> 11) / (double)(1ull << 53); };
    for (int trial = 0; trial < 3000; trial++) {
        const uint32_t target = trial % 3 ? q.target : std::min(q.target, kMinTarget);
        // a bin's own largest group, share of large ones, and k-mers a piece
        const double top = q.max_halves * (trial % 2 ? 1.0 : unit()), large = unit() * unit();
        std::vector<uint64_t> cnt(30 + rnd() % 300);
        for (auto& c : cnt) {
            const double len = 1 + 63 * unit() * unit(), halves = top * (unit() < large ? 0.2 + 0.8 * unit() : 0.15 * unit());
            const uint64_t pieces = (uint64_t)(halves * 16 / (len + q.k + 29)), kmers = (uint64_t)(pieces * len);
            c = pieces << 32 | (kmers < pieces ? pieces : kmers);
        }
        scan(q, target, cnt, T);
        T.tables = 0;   // (a bin each)
    }
    print("random", q, z, T, 0);
}

// genome <k> <m> <load> <block> <n_bins> <genome bases> <coverage, 0: one sequence> <read> <seed>
static void genome(char** a) {
    gerbil_params p;
    memset(&p, 0, sizeof(p));
    p.k = atoi(a[0]);
    p.m = atoi(a[1]);
    p.load_factor = (float)atof(a[2]);
    p.block = atoi(a[3]);
    p.n_bins = atoi(a[4]);
    p.mode = GERBIL_BATCHED;
    const uint64_t G = strtoull(a[5], 0, 10), cov = strtoull(a[6], 0, 10), read = strtoull(a[7], 0, 10);
    rng_state = strtoull(a[8], 0, 10);
    std::vector<uint8_t> g(G);
    for (auto& x : g) x = rnd() >> 62;
    const uint64_t reads = cov ? cov * G / read : 1, n_bytes = cov ? reads * read : G, w = p.k - p.m + 1;
    const uint64_t cap = std::min<uint64_t>(n_bytes * 4 / (w + 1) + n_bytes / 2048 + 4096, n_bytes + 4096);
    const PieceSizing z = piece_sizing(&p, n_bytes, cap);
    PieceArgs q;
    memset(&q, 0, sizeof(q));
    set_rules(q, &p, z);
    std::vector<Bin> bins(p.n_bins);
    uint64_t pos = 0;
    for (uint64_t r = 0; r < reads; r++) {
        const uint64_t len = cov ? read : G, at = cov ? rnd() % (G - len + 1) : 0;
        cut_read(q, p.m, p.n_bins, pos, std::vector<uint8_t>(g.begin() + at, g.begin() + at + len), bins);
        pos += len;
    }
    Totals T;
    uint64_t ns = 0;
    for (const Bin& b : bins) {
        T.kmers += b.kmers;
        ns += b.ns;
    }
    const uint64_t target = plan_target(q, T.kmers);
    for (const Bin& b : bins) {
        const uint32_t P = bin_groups(q, target, b.ns, b.kmers);
        if (P == 0) continue;
        T.expected += expected_pieces(q, b.ns, b.kmers);
        std::vector<uint64_t> cnt(P);
        for (uint64_t x : b.pieces) cnt[group_of_hash((uint32_t)(x >> 8), P)] += (1ull << 32) | (x & 255);
        scan(q, (uint32_t)target, cnt, T);
    }
    print("genome", q, z, T, piece_list_slots(ns, T.kmers, z.piece_fx, z.n0, w > z.n0, p.n_bins));
}

int main(int argc, char** argv) {
    if (argc == 11 && !strcmp(argv[1], "genome")) genome(argv + 2);
    else if (argc == 9 && !strcmp(argv[1], "groups")) groups(argv + 2);
    else if (argc == 6 && !strcmp(argv[1], "random")) random_groups(argv + 2);
    else return 2;
    return 0;
}
