// How a batch of trees is cut into groups that each run on one XCD, and the
// tiles and order of positions that follow.  Host code without device parts.
//
// Positions in: nodes by (level, id), a level being the height above the
// leaves, so children come before their parents; `parent` gives the position
// of each node's parent (-1 for a root).  Positions out: all leaves, then all
// internal nodes, in each by (launch and group, level, id).
#pragma once

#include <algorithm>
#include <cstddef>
#include <cstdint>
#include <memory>
#include <numeric>
#include <utility>
#include <vector>

namespace janus {
namespace treex {

constexpr int kRows = 16;             // nodes of a tile
constexpr int kMaxGroups = 64;        // groups of one launch
constexpr int kMaxParts = 16;         // launches of a batch at most

// One group's part of the launch: nodes by position (leaves first, then the
// internal nodes; both contiguous per group), its tiles in order.  The tiles
// [t0, t1) start with the `leaf_tiles` tiles of leaves.  A launch may have
// groups without nodes (t0 == t1).
struct Group {
    int leaf0, nleaf, int0, nint;
    int t0, t1, leaf_tiles;
    int pieces;            // holds roots of pieces whose parents run in a later launch
};
// A tile: first position and (rows | level << 8).
struct Tile {
    int p0, rows_level;
};
constexpr size_t kGroupBytes = sizeof(Group) * kMaxGroups * kMaxParts;

// What a launch can hold: workgroups of a group, CUs of an XCD, XCDs, and nodes
// of a group (its cells' LDS).
struct CutShape {
    int nu = 0, per_xcd = 0, xccs = 0, capacity = 0;
    bool leaves = true;    // tiles of leaves are worked (the TreeRNN's are not)
    int most_groups() const { return std::min(xccs * (per_xcd / nu), kMaxGroups); }
};
// Groups [first, first + groups) of the cut run in one launch.
struct CutLaunch {
    int first, groups;
};
struct Cut {
    // The arrays by node, and `more` integers for the caller, in one block.
    int32_t* parent = nullptr;         // position in -> position in of the parent, set by the caller
    int32_t* order = nullptr;          // position out -> position in
    int32_t* pos = nullptr;            // position in -> position out
    int32_t* bin = nullptr;            // position in -> group
    int32_t* more = nullptr;
    // Positions in of the roots, set by the caller in the order of its trees:
    // ties of the deal go by it.  (By height the tallest of equal trees would
    // share a group: 25 trees of 50 leaves, TreeRNN of H 150, forward kernel 39.4
    // us so, 42.3 by height, the mean of 12 batches.)
    std::vector<int32_t> root;
    std::vector<CutLaunch> launch;     // in the order of the forward
    int xccs = 0;
    int most_nodes = 0;                // nodes of the largest group
    bool split = false;                // trees are cut: links between launches
    std::vector<Group> group;
    std::vector<Tile> tile;
    std::vector<char> piece;           // by position in, if split: a root of a piece
    void take(int N, size_t n_more) {
        store.reset(new int32_t[size_t(4) * N + n_more]);
        parent = store.get();
        order = parent + N;
        pos = order + N;
        bin = pos + N;
        more = bin + N;
    }
    int blocks(const CutLaunch& l, int nu) const { return xccs * nu * ((l.groups + xccs - 1) / xccs); }

  private:
    std::unique_ptr<int32_t[]> store;
};

// Groups of a plan: the group of each node, and the launches.
struct CutPlan {
    int32_t* bin = nullptr;
    std::vector<CutLaunch> launch;
    int bins = 0, most_nodes = 0;
};

// Units of `size` nodes each to the least loaded of `groups` groups, the
// largest first (ties by index), in as few launches as hold them.  Appends the
// launches; unit_bin receives the groups.
inline bool deal_units(const std::vector<int32_t>& size, int groups, int capacity, CutPlan& p,
                       std::vector<int32_t>& unit_bin) {
    const int n = int(size.size());
    int64_t total = 0;
    int32_t top = 0;
    for (int32_t v : size) {
        total += v;
        top = std::max(top, v);
    }
    if (n == 0 || top > capacity) return false;
    // by size, largest first
    std::vector<int32_t> by(n), at(size_t(top) + 2, 0);
    for (int32_t v : size) ++at[top - v + 1];
    for (int32_t v = 0; v <= top; ++v) at[v + 1] += at[v];
    for (int k = 0; k < n; ++k) by[at[top - size[k]]++] = k;
    unit_bin.resize(n);
    std::vector<std::pair<int64_t, int>> heap;   // (-load, -bin): the least loaded, lowest bin on top
    const int64_t room = int64_t(capacity) * groups;
    for (int64_t parts = std::max<int64_t>(1, (total + room - 1) / room);; ++parts) {
        if (int64_t(p.launch.size()) + parts > kMaxParts) return false;
        heap.clear();
        for (int b = 0; b < int(parts) * groups; ++b) heap.push_back({0, -b});
        int64_t most = 0;
        for (int k : by) {
            std::pop_heap(heap.begin(), heap.end());
            auto& low = heap.back();
            unit_bin[k] = p.bins - low.second;
            low.first -= size[k];
            most = std::max(most, -low.first);
            std::push_heap(heap.begin(), heap.end());
        }
        if (most > capacity) continue;
        p.most_nodes = std::max(p.most_nodes, int(most));
        for (int q = 0; q < int(parts); ++q) p.launch.push_back({p.bins + q * groups, groups});
        p.bins += int(parts) * groups;
        return true;
    }
}

// Nodes of the subtree of each position.
inline std::vector<int32_t> subtree_sizes(int N, const int32_t* parent) {
    std::vector<int32_t> size(N, 1);
    for (int i = 0; i < N; ++i)
        if (parent[i] >= 0) size[parent[i]] += size[i];
    return size;
}

// Whole trees of tree_size nodes: the groups of their roots.
inline bool plan_trees(const std::vector<int32_t>& root, const std::vector<int32_t>& tree_size, const CutShape& s,
                       CutPlan& p) {
    std::vector<int32_t> tree_bin;
    if (!deal_units(tree_size, std::min(int(root.size()), s.most_groups()), s.capacity, p, tree_bin)) return false;
    for (size_t k = 0; k < root.size(); ++k) p.bin[root[k]] = tree_bin[k];
    return true;
}

// Pieces of trees.  A round takes the largest subtrees of at most `most` nodes
// of what is left, deals them to all groups and leaves their parents to a later
// round, whose launches find the pieces' results in memory.  The first round
// makes pieces of a 2 G-th of the nodes, for balance; a second takes all that is
// above them, unless a tree of that is still larger than a group.
// left: subtree_sizes.  One loop over all nodes finds the first round's pieces,
// parents before children, the later rounds only visit what is left (9 trees of
// 999 to 1399 nodes: 63 us with loops over all nodes for each round and their
// tiles counted, 31 so).
inline bool plan_pieces(int N, const int32_t* parent, std::vector<int32_t> left, const CutShape& s, CutPlan& p,
                        std::vector<char>& piece) {
    std::vector<int32_t> id(size_t(N) + 1, -1);   // unit of a node
    std::vector<int32_t> rest, above, unit, unit_size, unit_bin, bin;
    piece.assign(N, 0);
    int64_t most = std::min<int64_t>(s.capacity, std::max<int64_t>(kRows, N / (2 * s.most_groups())));
    const auto visit = [&](int i) {
        const int up = parent[i] < 0 ? N : parent[i];
        id[i] = id[up];
        if (id[up] >= 0) return;
        if (left[i] <= most) {
            id[i] = int32_t(bin.size() + unit.size());
            piece[i] = up < N;
            unit.push_back(i);
            unit_size.push_back(left[i]);
        } else {
            above.push_back(i);
        }
    };
    for (int i = N; i-- > 0;) visit(i);
    for (;;) {
        if (!deal_units(unit_size, std::min(int(unit.size()), s.most_groups()), s.capacity, p, unit_bin)) return false;
        bin.insert(bin.end(), unit_bin.begin(), unit_bin.end());
        if (above.empty()) break;
        rest.swap(above);
        above.clear();
        unit.clear();
        unit_size.clear();
        most = s.capacity;
        for (int i : rest) left[i] = 1;
        for (size_t k = rest.size(); k-- > 0;)
            if (parent[rest[k]] >= 0) left[parent[rest[k]]] += left[rest[k]];
        for (int i : rest) visit(i);
    }
    for (int i = 0; i < N; ++i) p.bin[i] = bin[id[i]];
    return true;
}

// Calls node(i, group) for every position in order, and level(L, group, nodes)
// for the groups that have nodes at a level, after the nodes of that level.
template <class NodeFn, class LevelFn>
inline void each_level(int num_levels, const std::vector<int32_t>& level_offsets, const CutPlan& p, NodeFn node,
                       LevelFn level) {
    std::vector<int32_t> rows(p.bins, 0), touched(p.bins);
    for (int L = 0; L < num_levels; ++L) {
        int n = 0;
        for (int i = level_offsets[L]; i < level_offsets[L + 1]; ++i) {
            const int b = p.bin[i];
            node(i, b);
            if (rows[b]++ == 0) touched[n++] = b;
        }
        for (int k = 0; k < n; ++k) {
            level(L, touched[k], rows[touched[k]]);
            rows[touched[k]] = 0;
        }
    }
}

// Nodes and tiles of each group of a plan, and what its launches take together in units
// of a tile: each as long as its longest group, and a start worth kStart tiles.
// (`leaves`: tiles of leaves are worked, too.)
constexpr int kStart = 8;
inline int64_t plan_cost(int num_levels, const std::vector<int32_t>& level_offsets, bool leaves, const CutPlan& p,
                         std::vector<Group>& group) {
    group.assign(p.bins, Group{});
    each_level(num_levels, level_offsets, p, [](int, int) {}, [&](int L, int b, int rows) {
        Group& g = group[b];
        g.t1 += (rows + kRows - 1) / kRows;
        if (L == 0) g.leaf_tiles = g.t1;
        (L == 0 ? g.nleaf : g.nint) += rows;
    });
    int64_t cost = 0;
    for (const CutLaunch& l : p.launch) {
        int most = 0;
        for (int b = l.first; b < l.first + l.groups; ++b)
            most = std::max(most, group[b].t1 - (leaves ? 0 : group[b].leaf_tiles));
        cost += kStart + most;
    }
    return cost;
}

// The cut of a batch (c.take, c.parent and c.root are the caller's): its trees
// whole, or in pieces where a tree is larger than a group may be, or so large a
// part of the batch that the other XCDs would wait for it and the pieces take
// less time (one tree of 1199 nodes of a TreeLSTM of H 150, step: 531 us whole,
// 249 in pieces).  Pieces are only made where the wait could hold a second start
// and the host's work for them, about 3 ns a node, a tile of 16 taking 1.5 us
// and more (30 trees of 239 nodes of a TreeRNN of H 64: step 270 us with pieces
// made and dropped, 214 without; 8 trees of 199 and one of 799, H 150: 192 us
// whole, 160 in pieces).
// False when the batch does not fit kMaxParts launches.
inline bool cut_batch(int N, const std::vector<int32_t>& level_offsets, int num_levels, const CutShape& s, Cut& c) {
    if (s.nu <= 0 || s.per_xcd < s.nu || s.xccs <= 0 || s.capacity <= 0) return false;
    const std::vector<int32_t> size = subtree_sizes(N, c.parent);
    std::vector<int32_t> tree_size;
    for (int32_t r : c.root) tree_size.push_back(size[r]);
    const int32_t largest = *std::max_element(tree_size.begin(), tree_size.end());
    std::vector<int32_t> bin;
    std::vector<Group> other;
    CutPlan p, q;   // whole and in pieces
    p.bin = c.bin;
    const bool whole = plan_trees(c.root, tree_size, s, p);
    // nodes whose tiles are worked, of n nodes (without leaves: of a binary tree)
    const auto worked = [&](int64_t n) { return s.leaves ? n : n / 2; };
    c.split = !whole;
    int64_t cost = INT64_MAX;
    // nodes of the longest groups above an even share
    const int64_t above = int64_t(p.most_nodes) * int64_t(p.launch.size()) - N / s.most_groups();
    if (!whole || worked(above) > kStart * kRows + N / 40) {
        bin.resize(N);
        q.bin = bin.data();
        if (plan_pieces(N, c.parent, size, s, q, c.piece))
            cost = plan_cost(num_levels, level_offsets, s.leaves, q, other);
        else if (!whole)
            return false;
        // about what the largest tree alone takes whole, every other level with a tile that is not full
        c.split |= cost < kStart + worked(largest) / kRows + num_levels / 2;
    }
    if (!c.split) {
        for (int i = N; i-- > 0;)
            if (c.parent[i] >= 0) c.bin[i] = c.bin[c.parent[i]];
        c.split = cost < plan_cost(num_levels, level_offsets, s.leaves, p, c.group);
    }
    if (c.split) {
        std::copy(bin.begin(), bin.end(), c.bin);
        p = std::move(q);
        p.bin = c.bin;
        c.group.swap(other);
    }
    c.xccs = s.xccs;
    c.launch = std::move(p.launch);
    c.most_nodes = p.most_nodes;
    std::vector<int32_t> next(p.bins), tile(p.bins);   // next position and tile of each group
    int leaf = 0, inner = level_offsets[1], first = 0;
    for (int b = 0; b < p.bins; ++b) {
        Group& g = c.group[b];
        g.leaf0 = leaf;
        g.int0 = inner;
        next[b] = g.nleaf > 0 ? leaf : inner;
        g.t0 = tile[b] = first;
        g.t1 += first;
        leaf += g.nleaf;
        inner += g.nint;
        first = g.t1;
    }
    c.tile.resize(first);
    each_level(
        num_levels, level_offsets, p,
        [&](int i, int b) {
            const int q = next[b]++;
            c.order[q] = i;
            c.pos[i] = q;
        },
        [&](int L, int b, int rows) {
            for (int q = next[b] - rows; q < next[b]; q += kRows)
                c.tile[tile[b]++] = {q, std::min(kRows, next[b] - q) | L << 8};
            if (L == 0) next[b] = c.group[b].int0;
        });
    if (c.split)
        for (int i = 0; i < N; ++i)
            if (c.piece[i]) c.group[p.bin[i]].pieces = 1;
    return true;
}

}  // namespace treex
}  // namespace janus
