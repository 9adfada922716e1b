// Cuts of random batches of trees (tree_cut.hpp) checked against what the
// kernels take for granted; prints "ok <cuts> <of them in pieces>" or the first
// property that fails.
#include <cstdio>
#include <cstdlib>
#include <random>

#include "../../paper_1812_01329_amd/csrc/tree_cut.hpp"

using namespace janus::treex;

#define NEED(x)                                                     \
    do {                                                            \
        if (!(x)) {                                                 \
            std::printf("case %d: %s (line %d)\n", the_case, #x, __LINE__); \
            std::exit(1);                                           \
        }                                                           \
    } while (0)

static int the_case = 0;
static std::mt19937 rng(23);
static int below(int n) { return int(rng() % unsigned(n)); }

struct Batch {
    std::vector<int32_t> parent, level_offsets;   // by (level, id)
    std::vector<int32_t> root;                    // by id
    int N = 0, levels = 0;
};

// parents of arbitrary node ids -> positions by (level, id)
static Batch sorted(const std::vector<int32_t>& up) {
    Batch b;
    b.N = int(up.size());
    std::vector<int32_t> level(b.N, 0), kids(b.N, 0), ready, pos(b.N);
    for (int32_t p : up)
        if (p >= 0) ++kids[p];
    for (int n = 0; n < b.N; ++n)
        if (kids[n] == 0) ready.push_back(n);
    for (size_t i = 0; i < ready.size(); ++i) {
        const int n = ready[i], p = up[n];
        b.levels = std::max(b.levels, level[n] + 1);
        if (p < 0) continue;
        level[p] = std::max(level[p], level[n] + 1);
        if (--kids[p] == 0) ready.push_back(p);
    }
    b.level_offsets.assign(b.levels + 1, 0);
    for (int n = 0; n < b.N; ++n) ++b.level_offsets[level[n] + 1];
    for (int L = 0; L < b.levels; ++L) b.level_offsets[L + 1] += b.level_offsets[L];
    std::vector<int32_t> next(b.level_offsets.begin(), b.level_offsets.end());
    for (int n = 0; n < b.N; ++n) pos[n] = next[level[n]]++;
    b.parent.assign(b.N, -1);
    for (int n = 0; n < b.N; ++n)
        if (up[n] >= 0)
            b.parent[pos[n]] = pos[up[n]];
        else
            b.root.push_back(pos[n]);
    return b;
}

// kind 0: random binary, 1: caterpillars, 2: random recursive (any arity), 3: stars, 4: chains
static Batch draw(int trees, int most, int kind) {
    std::vector<int32_t> up;
    for (int k = 0; k < trees; ++k) {
        const int n = 1 + below(most);
        if (kind <= 1) {   // n leaves joined two by two
            std::vector<int32_t> open;
            for (int i = 0; i < n; ++i) {
                open.push_back(int32_t(up.size()));
                up.push_back(-1);
            }
            while (open.size() > 1) {
                const int i = kind == 1 ? 0 : below(int(open.size()) - 1);
                up[open[i]] = up[open[i + 1]] = int32_t(up.size());
                open[i] = int32_t(up.size());
                open.erase(open.begin() + i + 1);
                up.push_back(-1);
            }
        } else {
            const int32_t r = int32_t(up.size());
            for (int i = 0; i < n; ++i) up.push_back(i == 0 ? -1 : kind == 2 ? r + below(i) : kind == 3 ? r : r + i - 1);
        }
    }
    return sorted(up);
}

// `count` trees of n leaves each, the first of `first` leaves
Batch equal_trees(int count, int n, int first) {
    std::vector<int32_t> up;
    for (int k = 0; k < count; ++k) {
        std::vector<int32_t> open;
        for (int i = 0; i < (k == 0 ? first : n); ++i) {
            open.push_back(int32_t(up.size()));
            up.push_back(-1);
        }
        while (open.size() > 1) {
            const int i = below(int(open.size()) - 1);
            up[open[i]] = up[open[i + 1]] = int32_t(up.size());
            open[i] = int32_t(up.size());
            open.erase(open.begin() + i + 1);
            up.push_back(-1);
        }
    }
    return sorted(up);
}
std::vector<int32_t> sizes(const Batch& b) {
    std::vector<int32_t> n(b.N, 1);
    for (int i = 0; i < b.N; ++i)
        if (b.parent[i] >= 0) n[b.parent[i]] += n[i];
    return n;
}
bool cuts_trees(const Batch& b, int nu, bool leaves) {
    CutShape s;
    s.nu = nu;
    s.per_xcd = 32;
    s.xccs = 8;
    s.leaves = leaves;
    s.capacity = 4000;
    Cut c;
    c.take(b.N, 0);
    std::copy(b.parent.begin(), b.parent.end(), c.parent);
    c.root = b.root;
    NEED(cut_batch(b.N, b.level_offsets, b.levels, s, c));
    NEED(c.split || c.piece.empty());   // none are made to be dropped
    bool equal = !c.split;              // equal trees go to the groups in turn
    for (size_t k = 1; k < b.root.size(); ++k) equal &= sizes(b)[b.root[k]] == sizes(b)[b.root[0]];
    for (size_t k = 0; equal && k < b.root.size(); ++k)
        NEED(c.bin[b.root[k]] == int(k) % std::min(int(b.root.size()), s.most_groups()));
    return c.split;
}

int main() {
    // pieces only where one tree keeps the other groups waiting for more than they cost
    for (bool leaves : {false, true}) {
        NEED(!cuts_trees(equal_trees(30, 120, 120), 8, leaves));
        NEED(!cuts_trees(equal_trees(25, 50, 50), 19, leaves));
        NEED(cuts_trees(equal_trees(9, 100, 400), 19, leaves));
        NEED(cuts_trees(equal_trees(1, 600, 600), 19, leaves));
    }
    int pieces = 0;
    for (the_case = 0; the_case < 1500; ++the_case) {
        const int trees = the_case % 3 == 0 ? 1 + below(3) : 1 + below(300);
        const Batch b = draw(trees, trees < 4 ? 1 + below(4000) : 1 + below(60), the_case % 5);
        CutShape s;
        s.nu = 1 + below(32);
        s.per_xcd = 32;
        s.xccs = the_case % 7 == 6 ? 1 : 8;
        s.leaves = the_case % 2 == 0;
        s.capacity = the_case % 4 == 3 ? 20 + below(100) : 300 + below(4000);
        Cut c;
        c.take(b.N, 0);
        std::copy(b.parent.begin(), b.parent.end(), c.parent);
        c.root = b.root;
        if (!cut_batch(b.N, b.level_offsets, b.levels, s, c)) {
            NEED(b.N > s.capacity);   // a batch that fits one group is never refused
            continue;
        }
        pieces += c.split;
        const int bins = int(c.group.size()), M0 = b.level_offsets[1];
        NEED(c.launch.size() <= size_t(kMaxParts) && sizeof(Group) * bins <= kGroupBytes && int(c.tile.size()) <= b.N);
        std::vector<int> launch_of(bins, -1), group_of(b.N, -1), level_of(b.N);
        int first = 0;
        for (size_t l = 0; l < c.launch.size(); ++l) {
            NEED(c.launch[l].first == first && c.launch[l].groups >= 1 && c.launch[l].groups <= s.most_groups());
            NEED(c.blocks(c.launch[l], s.nu) <= s.per_xcd * s.xccs && c.blocks(c.launch[l], s.nu) >= c.launch[l].groups * s.nu);
            for (int g = 0; g < c.launch[l].groups; ++g) launch_of[first++] = int(l);
        }
        NEED(first == bins);
        for (int L = 0; L < b.levels; ++L)
            for (int i = b.level_offsets[L]; i < b.level_offsets[L + 1]; ++i) {
                NEED(c.pos[i] >= 0 && c.pos[i] < b.N && c.order[c.pos[i]] == i && (c.pos[i] < M0) == (L == 0));
                level_of[c.pos[i]] = L;
            }
        int leaf = 0, inner = M0, tile = 0;
        for (int g = 0; g < bins; ++g) {
            const Group& q = c.group[g];
            NEED(q.leaf0 == leaf && q.int0 == inner && q.t0 == tile && q.t1 >= q.t0);
            NEED(q.nleaf + q.nint <= s.capacity && q.nleaf + q.nint <= c.most_nodes);
            for (int p = q.leaf0; p < q.leaf0 + q.nleaf; ++p) group_of[p] = g;
            for (int p = q.int0; p < q.int0 + q.nint; ++p) group_of[p] = g;
            int at = q.leaf0, level = -1;
            for (int t = q.t0; t < q.t1; ++t) {
                if (t == q.t0 + q.leaf_tiles) {
                    NEED(at == q.leaf0 + q.nleaf);
                    at = q.int0;
                }
                const int rows = c.tile[t].rows_level & 0xff, L = c.tile[t].rows_level >> 8;
                NEED(c.tile[t].p0 == at && rows >= 1 && rows <= kRows && L >= level && (L == 0) == (t < q.t0 + q.leaf_tiles));
                for (int p = at; p < at + rows; ++p) NEED(level_of[p] == L);
                level = L;
                at += rows;
            }
            NEED(at == (q.leaf_tiles == q.t1 - q.t0 ? q.leaf0 + q.nleaf : q.int0 + q.nint));
            leaf += q.nleaf;
            inner += q.nint;
            tile = q.t1;
        }
        NEED(leaf == M0 && inner == b.N && tile == int(c.tile.size()));
        std::vector<int> holds(bins, 0);
        for (int i = 0; i < b.N; ++i) {
            const int up = b.parent[i], g = group_of[c.pos[i]];
            NEED(g >= 0);
            const bool apart = up >= 0 && group_of[c.pos[up]] != g;
            NEED(!apart || (c.split && launch_of[g] < launch_of[group_of[c.pos[up]]]));
            if (c.split) {
                NEED(bool(c.piece[i]) == apart);
                if (apart) holds[g] = 1;
            }
        }
        for (int g = 0; g < bins; ++g) NEED(c.group[g].pieces == holds[g]);
    }
    std::printf("ok %d %d\n", the_case, pieces);
    return 0;
}
