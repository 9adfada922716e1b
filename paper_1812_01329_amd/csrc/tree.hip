// Binary TreeLSTM over a batch of trees, evaluated as level-wise frontiers.
//
// The recursive TreeNN program (Section 6.1, footnote 6; recursion turned
// into graph invocations, Section 4.2.1) visits a node after both of its
// subtrees.  Grouping nodes by height gives frontiers of independent cell
// applications: every node of level k depends only on levels < k, so a
// level is one batched contraction plus one pointwise kernel, across all
// trees of the batch at once (the paper's largest gain on TreeNNs comes from
// running independent nodes together, Section 6.3.1 "+PARL").
//
// Node state is stored by level-ordered position p (nodes of a level are
// contiguous), so each level's contraction reads a dense block of rows:
//   level 0 (all leaves):  A_0 = emb[word] W^T + b   (row gather of emb)
//   level k >= 1:          A_k = HLR_k U^T + b       (HLR row = [h_L; h_R])
// The pointwise kernel of a level writes each node's h straight into its
// parent's HLR row (left or right half) or into h_root, so the next level's
// operand is ready without a gather.
//
// Backward, levels from the top down: the pointwise backward of a level
// writes its da rows and its children's dc; the contraction da U sends
// [dh_L; dh_R] to the two children (each node has one parent, so these are
// plain stores).  After the loop: dU = da_int^T HLR, dW = da_leaf^T X_leaf,
// db = column sums of da, dx_leaf = da_leaf W, then the embedding gradient.
#include <algorithm>
#include <cstdlib>
#include <mutex>
#include <vector>

#include "device.hpp"
#include "ops.hpp"
#include "simt.hpp"
#include "tree_common.hpp"
#include "tree_tail.hpp"
#include "tree_xcd.hpp"

namespace janus {

namespace {

using tpersist::TreeDev;
using tpersist::tree_dev;
using tpersist::tree_persistent_launch;

struct TreeWs {
    // level-ordered device schedule
    int32_t* lword = nullptr;    // [N] word of a leaf, -1 otherwise
    int32_t* lchild = nullptr;   // [N] position of left child, -1 for leaves
    int32_t* rchild = nullptr;   // [N]
    int32_t* parent = nullptr;   // [N] 2 * position of parent + side, -1 for roots
    int32_t* rootk = nullptr;    // [N] tree index of a root, -1 otherwise
    int32_t* rootpos = nullptr;  // [K] position of root k
    float* A = nullptr;          // [N x ld5] pre-activations (forward), da (backward)
    float* G = nullptr;          // [N x ld5] gates (i, f_L, f_R, o, u) after activation
    float* C = nullptr;          // [N x H]   cell memory
    float* HLR = nullptr;        // [N x 2H]  children's h of internal nodes (row p - M0)
    float* dh = nullptr;         // [N x H]
    float* dc = nullptr;         // [N x H]
    float* dxl = nullptr;        // [N x E]   gradient of leaf inputs
    float* Wt = nullptr;         // [E x 5H]  W transposed (forward)
    float* Ut = nullptr;         // [2H x 5H] U transposed (forward)
    float* part = nullptr;
    int32_t* seg = nullptr;      // the leaves grouped by word, for the embedding gradient
    int64_t ld5 = 0;
    // groups of trees per XCD (tree_xcd.hpp): the groups, followed by their
    // tiles (carved after the schedule arrays, so that one copy uploads both),
    // the counters, and node rows padded to whole 128-byte lines
    tpersist::TreeSync* tsync = nullptr;
    treex::Group* xgroup = nullptr;  // the groups of every launch, then up to N tiles
    float* xl = nullptr;         // [N x ldx] leaf inputs
    float* hx = nullptr;         // [N x ldc] h of every node
    float* Gp = nullptr;         // [N x ldg] gates
    float* Cp = nullptr;         // [N x ldc]
    float* HLRp = nullptr;       // [N x ldl]
    float* dAp = nullptr;        // [N x lda]
    float* dxp = nullptr;        // [3][N x E] parts of the leaves' input gradient
    float* tpart = nullptr;      // parts of dU and dW
    float* tsum = nullptr;       // parts of db
    int64_t ldg = 0, ldc = 0, ldl = 0, lda = 0, ldx = 0;
};

// the groups of every launch and the tiles of N nodes
treex::Group* take_cut(Carver& c, int32_t N) {
    return reinterpret_cast<treex::Group*>(c.take<char>(treex::kGroupBytes + size_t(N) * sizeof(treex::Tile)));
}

size_t carve(const janus_treelstm_desc& d, int32_t N, int32_t K, void* base, TreeWs& w) {
    Carver c(base);
    const int H = d.H;
    w.ld5 = round_up(int64_t(5) * H, 4);
    w.lword = c.take<int32_t>(N);
    w.lchild = c.take<int32_t>(N);
    w.rchild = c.take<int32_t>(N);
    w.parent = c.take<int32_t>(N);
    w.rootk = c.take<int32_t>(N);
    w.rootpos = c.take<int32_t>(K);
    w.xgroup = take_cut(c, N);
    w.tsync = c.take<tpersist::TreeSync>(1);
    w.seg = c.take<int32_t>(int64_t(embed_seg_ints(N)));   // the leaves grouped by word
    w.A = c.take<float>(int64_t(N) * w.ld5);
    w.G = c.take<float>(int64_t(N) * w.ld5);
    w.C = c.take<float>(int64_t(N) * H);
    w.HLR = c.take<float>(int64_t(N) * 2 * H);
    w.dh = c.take<float>(int64_t(N) * H);
    w.dc = c.take<float>(int64_t(N) * H);
    w.dxl = c.take<float>(int64_t(N) * d.E);
    w.Wt = c.take<float>(int64_t(d.E) * 5 * H);
    w.Ut = c.take<float>(int64_t(2) * H * 5 * H);
    w.part = c.take<float>(colsum_partial_floats(5 * H));
    w.ldg = w.lda = round_up(int64_t(5) * H, 32);
    w.ldc = round_up(H, 32);
    w.ldl = round_up(int64_t(2) * H, 32);
    w.ldx = round_up(d.E, 32);
    w.Gp = c.take<float>(int64_t(N) * w.ldg);
    w.Cp = c.take<float>(int64_t(N) * w.ldc);
    w.HLRp = c.take<float>(int64_t(N) * w.ldl);
    w.dAp = c.take<float>(int64_t(N) * w.lda);
    w.dxp = c.take<float>(int64_t(3) * N * d.E);
    w.tpart = c.take<float>(tail_part_floats(5 * H, 2 * H) + tail_part_floats(5 * H, d.E));
    w.tsum = c.take<float>(tail_sum_floats(N, 5 * H));
    w.xl = c.take<float>(int64_t(N) * w.ldx);
    w.hx = c.take<float>(int64_t(N) * w.ldc);
    return c.off + 256;
}

// one schedule array set per call, in level order or in that of a cut
struct TreeHost {
    int32_t *lword, *lchild, *rchild, *parent, *rootk, *rootpos;
    static size_t ints(int32_t N, int32_t K) { return size_t(5) * N + K; }
    TreeHost(int32_t* store, int32_t N)
        : lword(store), lchild(lword + N), rchild(lchild + N), parent(rchild + N), rootk(parent + N), rootpos(rootk + N) {}
};

// The schedule's arrays; pos: where each of its positions goes (NULL: it stays).
void build_host(const janus_tree_batch* t, const TreeSchedule& s, const int32_t* pos, const TreeHost& h) {
    const int32_t N = s.N, M0 = s.level_offsets[1];
    std::fill(h.lword, h.lword + size_t(5) * N, -1);
    auto at = [&](int32_t n) { return pos ? pos[s.pos[n]] : s.pos[n]; };
    for (int32_t i = 0; i < M0; ++i) h.lword[pos ? pos[i] : i] = t->word[s.level_nodes[i]];
    for (int32_t i = M0; i < N; ++i) {
        const int32_t n = s.level_nodes[i], p = pos ? pos[i] : i, l = at(t->left[n]), r = at(t->right[n]);
        h.lchild[p] = l;
        h.rchild[p] = r;
        h.parent[l] = 2 * p;
        h.parent[r] = 2 * p + 1;
    }
    for (int32_t k = 0; k < t->num_trees; ++k) {
        const int32_t p = at(t->root[k]);
        h.rootk[p] = k;
        h.rootpos[k] = p;
    }
}

__device__ __forceinline__ float sig(float x) { return sigmoidf_(x); }

__global__ void tree_fwd_point_kernel(int p0, int rows, int H, int M0, int64_t ld5, const float* A, float* G,
                                      float* C, const int32_t* lchild, const int32_t* rchild, const int32_t* parent,
                                      const int32_t* rootk, float* HLR, float* h_root) {
    const int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
    if (i >= int64_t(rows) * H) return;
    const int p = p0 + int(i / H), j = int(i % H);
    const float* a = A + int64_t(p) * ld5 + j;
    const float gi = sig(a[0]), gl = sig(a[H]), gr = sig(a[2 * H]), go = sig(a[3 * H]), gu = tanhf_(a[4 * H]);
    const int lc = lchild[p], rc = rchild[p];
    const float cl = lc >= 0 ? C[int64_t(lc) * H + j] : 0.f;
    const float cr = rc >= 0 ? C[int64_t(rc) * H + j] : 0.f;
    const float c = gi * gu + gl * cl + gr * cr;
    const float h = go * tanhf_(c);
    C[int64_t(p) * H + j] = c;
    float* g = G + int64_t(p) * ld5 + j;
    g[0] = gi;
    g[H] = gl;
    g[2 * H] = gr;
    g[3 * H] = go;
    g[4 * H] = gu;
    const int par = parent[p];
    if (par >= 0) HLR[int64_t((par >> 1) - M0) * 2 * H + (par & 1) * H + j] = h;
    else h_root[int64_t(rootk[p]) * H + j] = h;
}

__global__ void tree_bwd_init_kernel(int K, int H, const int32_t* rootpos, const float* dh_root, float* dh, float* dc) {
    const int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
    if (i >= int64_t(K) * H) return;
    const int k = int(i / H), j = int(i % H);
    const int p = rootpos[k];
    dh[int64_t(p) * H + j] = dh_root[i];
    dc[int64_t(p) * H + j] = 0.f;
}

__global__ void tree_bwd_point_kernel(int p0, int rows, int H, int64_t ld5, const float* G, const float* C,
                                      const float* dh, float* dc, const int32_t* lchild, const int32_t* rchild,
                                      float* dA) {
    const int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
    if (i >= int64_t(rows) * H) return;
    const int p = p0 + int(i / H), j = int(i % H);
    const float* g = G + int64_t(p) * ld5 + j;
    const float gi = g[0], gl = g[H], gr = g[2 * H], go = g[3 * H], gu = g[4 * H];
    const int lc = lchild[p], rc = rchild[p];
    const float cl = lc >= 0 ? C[int64_t(lc) * H + j] : 0.f;
    const float cr = rc >= 0 ? C[int64_t(rc) * H + j] : 0.f;
    const float c = C[int64_t(p) * H + j];
    const float dhv = dh[int64_t(p) * H + j];
    const float tau = tanhf_(c);
    const float d_o = dhv * tau;
    const float dct = dc[int64_t(p) * H + j] + dhv * go * (1.f - tau * tau);
    float* da = dA + int64_t(p) * ld5 + j;
    da[0] = dct * gu * gi * (1.f - gi);
    da[H] = dct * cl * gl * (1.f - gl);
    da[2 * H] = dct * cr * gr * (1.f - gr);
    da[3 * H] = d_o * go * (1.f - go);
    da[4 * H] = dct * gi * (1.f - gu * gu);
    if (lc >= 0) {
        dc[int64_t(lc) * H + j] = dct * gl;
        dc[int64_t(rc) * H + j] = dct * gr;
    }
}

// One backward level k >= 1 in one launch: block (x, y) first applies the
// cell backward to the 8 rows y*8.. of the level (all 5H gate columns; every
// column block does this, block x = 0 also writes da and the children's dc
// to memory), straight into the LDS slab, then computes columns x*64.. of
// [dh_L; dh_R] = da U with K = 5H split over its waves, as simt_gemm_kernel.
__global__ __launch_bounds__(64 * kSimtWaves) void tree_bwd_level_kernel(int p0, int rows, int H, int64_t ld5,
                                                                         const float* G, const float* C,
                                                                         const float* dh_in, float* dc,
                                                                         const int32_t* lchild, const int32_t* rchild,
                                                                         float* dA, const float* U, float* dh) {
    __shared__ __align__(16) float sA[kSimtKc][kSimtRows];
    __shared__ float red[kSimtWaves][kSimtRows][kSimtCols];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int N = 2 * H, K = 5 * H;
    const int n = blockIdx.x * kSimtCols + lane;
    const int m0 = blockIdx.y * kSimtRows;
    const bool writer = blockIdx.x == 0;
    for (int i = tid; i < kSimtRows * H; i += 64 * kSimtWaves) {
        const int r = i / H, j = i - r * H, m = m0 + r;
        float da[5] = {0.f, 0.f, 0.f, 0.f, 0.f};
        if (m < rows) {
            const int p = p0 + m;
            const float* g = G + int64_t(p) * ld5 + j;
            const float gi = g[0], gl = g[H], gr = g[2 * H], go = g[3 * H], gu = g[4 * H];
            const int lc = lchild[p], rc = rchild[p];
            const float cl = C[int64_t(lc) * H + j], cr = C[int64_t(rc) * H + j];
            const float c = C[int64_t(p) * H + j];
            const float dhv = dh_in[int64_t(p) * H + j];
            const float tau = tanhf_(c);
            const float d_o = dhv * tau;
            const float dct = dc[int64_t(p) * H + j] + dhv * go * (1.f - tau * tau);
            da[0] = dct * gu * gi * (1.f - gi);
            da[1] = dct * cl * gl * (1.f - gl);
            da[2] = dct * cr * gr * (1.f - gr);
            da[3] = d_o * go * (1.f - go);
            da[4] = dct * gi * (1.f - gu * gu);
            if (writer) {
                float* dst = dA + int64_t(p) * ld5 + j;
#pragma unroll
                for (int q = 0; q < 5; ++q) dst[q * H] = da[q];
                dc[int64_t(lc) * H + j] = dct * gl;
                dc[int64_t(rc) * H + j] = dct * gr;
            }
        }
#pragma unroll
        for (int q = 0; q < 5; ++q) sA[q * H + j][r] = da[q];
    }
    __syncthreads();
    float acc[kSimtRows];
#pragma unroll
    for (int r = 0; r < kSimtRows; ++r) acc[r] = 0.f;
    const int kb = wave * K / kSimtWaves, ke = (wave + 1) * K / kSimtWaves;
    if (n < N) {
#pragma unroll 16
        for (int k = kb; k < ke; ++k) {
            const float bv = U[int64_t(k) * N + n];
            const float4 a0 = *reinterpret_cast<const float4*>(&sA[k][0]);
            const float4 a1 = *reinterpret_cast<const float4*>(&sA[k][4]);
            acc[0] += a0.x * bv; acc[1] += a0.y * bv; acc[2] += a0.z * bv; acc[3] += a0.w * bv;
            acc[4] += a1.x * bv; acc[5] += a1.y * bv; acc[6] += a1.z * bv; acc[7] += a1.w * bv;
        }
    }
#pragma unroll
    for (int r = 0; r < kSimtRows; ++r) red[wave][r][lane] = acc[r];
    __syncthreads();
    const int r = wave, m = m0 + r;
    if (m >= rows || n >= N) return;
    float sum = 0.f;
#pragma unroll
    for (int w = 0; w < kSimtWaves; ++w) sum += red[w][r][lane];
    const int p = p0 + m;
    if (n < H) dh[int64_t(lchild[p]) * H + n] = sum;
    else dh[int64_t(rchild[p]) * H + n - H] = sum;
}

janus_status check(const janus_treelstm_desc* d) {
    if (!d || d->E <= 0 || d->H <= 0 || d->V <= 0) return JANUS_ERR_INVALID_ARG;
    if (d->dtype != JANUS_F32) return JANUS_ERR_UNSUPPORTED;
    return JANUS_OK;
}

// `words`: receives the leaves' words (the backward groups the leaves by them)
janus_status upload_tree(const janus_tree_batch* t, const TreeSchedule& s, const TreeWs& w, hipStream_t st,
                         std::vector<int32_t>* words = nullptr) {
    std::vector<int32_t> store(TreeHost::ints(s.N, t->num_trees));
    const TreeHost h(store.data(), s.N);
    build_host(t, s, nullptr, h);
    if (words) words->assign(h.lword, h.lword + s.level_offsets[1]);
    const size_t nb = sizeof(int32_t) * s.N;
    // The error flag is zeroed too, so the device report of a call on this
    // path reads no stale one.
    const std::vector<char> zero_sync(tpersist::kTreeSyncCounters, 0);
    const UploadPiece pieces[] = {{w.lword, h.lword, nb},   {w.lchild, h.lchild, nb},
                                  {w.rchild, h.rchild, nb}, {w.parent, h.parent, nb},
                                  {w.rootk, h.rootk, nb},
                                  {w.rootpos, h.rootpos, sizeof(int32_t) * t->num_trees},
                                  {w.tsync, zero_sync.data(), zero_sync.size()}};
    return upload_pieces(pieces, 7, st);
}

janus_status prepare(const janus_treelstm_desc* d, const janus_tree_batch* t, void* ws, size_t ws_bytes,
                     TreeSchedule& s, TreeWs& w) {
    janus_status e = check(d);
    if (e != JANUS_OK) return e;
    if ((e = build_tree_schedule(t, d->V, s)) != JANUS_OK) return e;
    if (!ws || ws_bytes < carve(*d, s.N, t->num_trees, nullptr, w) || reinterpret_cast<uintptr_t>(ws) % 256 != 0)
        return JANUS_ERR_WORKSPACE;
    carve(*d, s.N, t->num_trees, ws, w);
    return JANUS_OK;
}


// ------------------------------------------------------- persistent path

// ------------------------------------------------- groups of trees per XCD

bool tree_env(const char* name, char v) {
    const char* e = getenv(name);
    return e && e[0] == v;
}

bool cut_trees(const janus_tree_batch* t, const TreeSchedule& s, const treex::CutShape& shape, treex::Cut& c) {
    c.take(s.N, TreeHost::ints(s.N, t->num_trees));
    std::fill(c.parent, c.parent + s.N, -1);
    for (int32_t i = s.level_offsets[1]; i < s.N; ++i) {
        const int32_t n = s.level_nodes[i];
        c.parent[s.pos[t->left[n]]] = c.parent[s.pos[t->right[n]]] = i;
    }
    for (int32_t k = 0; k < t->num_trees; ++k) c.root.push_back(s.pos[t->root[k]]);
    return treex::cut_batch(s.N, s.level_offsets, s.num_levels, shape, c);
}

// The binary TreeLSTM in groups of trees per XCD: row tiles of the forward
// (5 gates of 16 NT / 5 units) and of the backward ([dh_L; dh_R] of 8 MT
// units) by H, so that a group's workgroups fit one XCD (32 CUs) and their
// weights its VGPRs; each direction cuts the batch the same way, with the
// larger workgroup count and the backward's LDS (dh and dc of every node).
struct TreeXcdPlan {
    bool on = false;
    int NT = 0, MT = 0, fwd_nu = 0, bwd_nu = 0;
    treex::Cut cut;
    size_t fwd_lds = 0, bwd_lds = 0;
};
size_t tree_xcd_fwd_lds(int NT, int nodes) {
    return NT == 1   ? treex::LstmFwdCfg<1>::lds(nodes)
           : NT == 2 ? treex::LstmFwdCfg<2>::lds(nodes)
           : NT == 3 ? treex::LstmFwdCfg<3>::lds(nodes)
                     : treex::LstmFwdCfg<4>::lds(nodes);
}
size_t tree_xcd_bwd_lds(int MT, int nodes) {
    return MT == 1 ? treex::LstmBwdCfg<1>::lds(nodes) : treex::LstmBwdCfg<2>::lds(nodes);
}
TreeXcdPlan tree_xcd_plan(const janus_treelstm_desc& d, const janus_tree_batch* t, const TreeSchedule& s) {
    TreeXcdPlan p;
    if (tree_env("JANUS_TREE_PERSIST", '0')) return p;
    const TreeDev dev = tree_dev();
    if (dev.cus <= 0 || dev.lds == 0 || d.H > 384 || d.E > tpersist::kMaxE) return p;
    // 32-bit byte offsets into the exchanged rows
    if (int64_t(s.N) * round_up(5 * d.H, 32) * 4 >= (int64_t(1) << 31) ||
        int64_t(s.N) * round_up(d.E, 32) * 4 >= (int64_t(1) << 31))
        return p;
    p.NT = d.H <= 96 ? 1 : d.H <= 192 ? 2 : d.H <= 288 ? 3 : 4;
    p.MT = d.H <= 256 ? 1 : 2;
    const int fu = 16 * p.NT / 5, bu = 8 * p.MT;
    p.fwd_nu = (d.H + fu - 1) / fu;
    p.bwd_nu = (d.H + bu - 1) / bu;
    const int capacity = treex::node_capacity(
        dev.lds, [&](int n) { return std::max(tree_xcd_fwd_lds(p.NT, n), tree_xcd_bwd_lds(p.MT, n)); });
    p.on = cut_trees(t, s, treex::cut_shape(dev, std::max(p.fwd_nu, p.bwd_nu), capacity), p.cut);
    p.fwd_lds = tree_xcd_fwd_lds(p.NT, p.cut.most_nodes);
    p.bwd_lds = tree_xcd_bwd_lds(p.MT, p.cut.most_nodes);
    return p;
}
treex::Tile* cut_tiles(const TreeWs& w, const treex::Cut& c) {
    return reinterpret_cast<treex::Tile*>(w.xgroup + c.group.size());
}

// The schedule in the order of a cut, with its groups and tiles: one copy.
janus_status upload_cut(const janus_tree_batch* t, const TreeSchedule& s, const TreeWs& w, const treex::Cut& c,
                        hipStream_t st) {
    const TreeHost h(c.more, s.N);
    build_host(t, s, c.pos, h);
    if (c.split)
        for (int32_t i = 0; i < s.N; ++i)
            if (c.piece[i]) h.rootk[c.pos[i]] = treex::kPieceRoot;
    const size_t nb = sizeof(int32_t) * s.N;
    const UploadPiece pieces[] = {{w.lword, h.lword, nb},
                                  {w.lchild, h.lchild, nb},
                                  {w.rchild, h.rchild, nb},
                                  {w.parent, h.parent, nb},
                                  {w.rootk, h.rootk, nb},
                                  {w.rootpos, h.rootpos, sizeof(int32_t) * t->num_trees},
                                  {w.xgroup, c.group.data(), sizeof(treex::Group) * c.group.size()},
                                  {cut_tiles(w, c), c.tile.data(), sizeof(treex::Tile) * c.tile.size()}};
    return upload_pieces(pieces, 8, st);
}
// The leaves grouped by word, in the order of a cut.
int leaf_segments(const janus_tree_batch* t, const TreeSchedule& s, int32_t V, const treex::Cut& c,
                  std::vector<int32_t>& seg) {
    const int32_t M0 = s.level_offsets[1];
    int32_t* word = c.more;
    for (int32_t i = 0; i < M0; ++i) word[i] = t->word[s.level_nodes[c.order[i]]];
    return embed_segments(word, M0, V, seg);
}

unsigned fill_blocks(int64_t n) { return unsigned(std::min<int64_t>((n + 1023) / 1024, 1024)); }

template <int NT, bool PIECES>
janus_status launch_tree_fwd(int blocks, size_t lds, const treex::LstmFwd& a, hipStream_t st) {
    static size_t attr = 0;
    return tree_persistent_launch(treex::treelstm_fwd_xcd<NT, PIECES>, blocks, lds, a, st, attr, treex::kThreads);
}
template <int NT>
janus_status launch_tree_fwd(const TreeXcdPlan& p, int blocks, const treex::LstmFwd& a, hipStream_t st) {
    return p.cut.split ? launch_tree_fwd<NT, true>(blocks, p.fwd_lds, a, st)
                       : launch_tree_fwd<NT, false>(blocks, p.fwd_lds, a, st);
}
template <int MT, bool PIECES>
janus_status launch_tree_bwd(int blocks, size_t lds, const treex::LstmBwd& a, hipStream_t st) {
    static size_t attr = 0;
    return tree_persistent_launch(treex::treelstm_bwd_xcd<MT, PIECES>, blocks, lds, a, st, attr, treex::kThreads);
}
template <int MT>
janus_status launch_tree_bwd(const TreeXcdPlan& p, int blocks, const treex::LstmBwd& a, hipStream_t st) {
    return p.cut.split ? launch_tree_bwd<MT, true>(blocks, p.bwd_lds, a, st)
                       : launch_tree_bwd<MT, false>(blocks, p.bwd_lds, a, st);
}

janus_status treelstm_fwd_xcd_call(const janus_treelstm_desc& d, const janus_tree_batch* t, const TreeSchedule& s,
                                   const TreeWs& w, const TreeXcdPlan& p, const void* emb, const void* W, const void* U,
                                   const void* b, void* h_root, hipStream_t st) {
    janus_status e = upload_cut(t, s, w, p.cut, st);
    if (e != JANUS_OK) return e;
    const int M0 = s.level_offsets[1];
    treex::LstmFwd a = {};
    a.E = d.E;
    a.H = d.H;
    a.M0 = M0;
    a.nu = p.fwd_nu;
    a.xccs = tree_env("JANUS_XCD_REMOTE", '1') ? 0 : p.cut.xccs;
    a.tile = cut_tiles(w, p.cut);
    a.lchild = w.lchild;
    a.rchild = w.rchild;
    a.parent = w.parent;
    a.rootk = w.rootk;
    a.W = static_cast<const float*>(W);
    a.U = static_cast<const float*>(U);
    a.b = static_cast<const float*>(b);
    a.x = w.xl;
    a.ldx = w.ldx;
    a.x_bytes = uint32_t(int64_t(M0) * w.ldx * 4);
    a.hx = w.hx;
    a.ldh = w.ldc;
    a.hx_bytes = uint32_t(int64_t(s.N) * w.ldc * 4);
    a.G = w.Gp;
    a.ldg = w.ldg;
    a.C = w.Cp;
    a.ldc = w.ldc;
    a.HLR = w.HLRp;
    a.ldl = w.ldl;
    a.h_root = static_cast<float*>(h_root);
    a.sync = w.tsync;
    const int parts = int(p.cut.launch.size());
    for (int part = 0; part < parts; ++part) {
        if (part == 0) {
            TraceScope trace("tree_fwd_init", 0.0, 4.0 * (double(s.N) * w.ldc + 2.0 * M0 * w.ldx), st);
            hipLaunchKernelGGL(treex::fwd_init_kernel, dim3(fill_blocks(int64_t(s.N) * w.ldc + int64_t(M0) * w.ldx)),
                               dim3(256), 0, st, s.N, M0, d.E, w.lword, static_cast<const float*>(emb), w.xl, w.ldx,
                               w.hx, w.ldc, d.H, w.tsync);
        } else {   // the counters of the next launch
            hipLaunchKernelGGL(treex::fill_kernel, dim3(4), dim3(256), 0, st, w.hx, w.ldc, int64_t(0), int64_t(0), d.H,
                               w.tsync);
        }
        JANUS_LAUNCH_CHECK();
        const treex::CutLaunch& l = p.cut.launch[part];
        a.group = w.xgroup + l.first;
        a.groups = l.groups;
        const int blocks = p.cut.blocks(l, p.fwd_nu);
        const double flops = 2.0 * 5.0 * d.H * (double(M0) * d.E + double(s.N - M0) * 2.0 * d.H) / parts;
        TraceScope trace("treelstm_fwd_persistent", flops, 0.0, st);
        e = p.NT == 1   ? launch_tree_fwd<1>(p, blocks, a, st)
            : p.NT == 2 ? launch_tree_fwd<2>(p, blocks, a, st)
            : p.NT == 3 ? launch_tree_fwd<3>(p, blocks, a, st)
                        : launch_tree_fwd<4>(p, blocks, a, st);
        if (e != JANUS_OK) return e;
    }
    return JANUS_OK;
}

// The backward's levels in groups of trees per XCD: dA of every node.
janus_status treelstm_bwd_xcd_levels(const janus_treelstm_desc& d, const TreeSchedule& s, const TreeWs& w,
                                     const TreeXcdPlan& p, const void* U, const void* dh_root, hipStream_t st) {
    const int M0 = s.level_offsets[1];
    treex::LstmBwd a = {};
    a.H = d.H;
    a.M0 = M0;
    a.nu = p.bwd_nu;
    a.xccs = tree_env("JANUS_XCD_REMOTE", '1') ? 0 : p.cut.xccs;
    a.tile = cut_tiles(w, p.cut);
    a.lchild = w.lchild;
    a.rchild = w.rchild;
    a.rootk = w.rootk;
    a.U = static_cast<const float*>(U);
    a.G = w.Gp;
    a.ldg = w.ldg;
    a.C = w.Cp;
    a.ldc = w.ldc;
    a.dh_root = static_cast<const float*>(dh_root);
    a.dhx = w.dh;
    a.dcx = w.dc;
    a.dA = w.dAp;
    a.lda = w.lda;
    a.dA_bytes = uint32_t(int64_t(s.N) * w.lda * 4);
    a.sync = w.tsync;
    const int parts = int(p.cut.launch.size());
    for (int part = parts; part-- > 0;) {   // parents before the pieces below them
        const int64_t rows = part == parts - 1 ? s.N - M0 : 0;
        {
            TraceScope trace("tree_bwd_init", 0.0, 4.0 * double(rows) * w.lda, st);
            hipLaunchKernelGGL(treex::fill_kernel, dim3(fill_blocks(rows * w.lda + 4096)), dim3(256), 0, st, w.dAp, w.lda,
                               int64_t(M0), rows, 5 * d.H, w.tsync);
            JANUS_LAUNCH_CHECK();
        }
        const treex::CutLaunch& l = p.cut.launch[part];
        a.group = w.xgroup + l.first;
        a.groups = l.groups;
        const int blocks = p.cut.blocks(l, p.bwd_nu);
        TraceScope trace("treelstm_bwd_persistent", 2.0 * 5.0 * d.H * double(s.N - M0) * 2.0 * d.H / parts, 0.0, st);
        const janus_status e = p.MT == 1 ? launch_tree_bwd<1>(p, blocks, a, st) : launch_tree_bwd<2>(p, blocks, a, st);
        if (e != JANUS_OK) return e;
    }
    return JANUS_OK;
}

// Backward: the schedule is the forward's (the workspace is unchanged between
// the two calls); the leaves grouped by word go over in one copy, then the
// levels, the contractions over nodes and the embedding gradient.
janus_status treelstm_bwd_xcd_call(const janus_treelstm_desc& d, const janus_tree_batch* t, const TreeSchedule& s,
                                   const TreeWs& w, const TreeXcdPlan& p, const void* W, const void* U,
                                   const void* dh_root, float* demb, float* dW, float* dU, float* db, hipStream_t st) {
    const int M0 = s.level_offsets[1], Nint = s.N - M0, H = d.H, E = d.E;
    std::vector<int32_t> seg;
    const int nseg = leaf_segments(t, s, d.V, p.cut, seg);
    janus_status e;
    if ((e = upload(w.seg, seg.data(), seg.size() * sizeof(int32_t), st)) != JANUS_OK) return e;
    if ((e = treelstm_bwd_xcd_levels(d, s, w, p, U, dh_root, st)) != JANUS_OK) return e;
    TailArgs a;
    GemmDesc g;
    g.dtype = JANUS_F32;
    // dU = dA_int^T [h_L; h_R]
    g.M = 5 * H;
    g.N = 2 * H;
    g.K = Nint;
    g.a_t = g.b_t = true;
    g.A = w.dAp + int64_t(M0) * w.lda;
    g.lda = w.lda;
    g.B = w.HLRp;
    g.ldb = w.ldl;
    g.C = dU;
    g.ldc = 2 * H;
    tail_add(a, g, w.tpart);
    // dW = dA_leaf^T x
    g.N = E;
    g.K = M0;
    g.A = w.dAp;
    g.B = w.xl;
    g.ldb = w.ldx;
    g.C = dW;
    g.ldc = E;
    tail_add(a, g, w.tpart + tail_part_floats(5 * H, 2 * H));
    // dx = dA_leaf W, in up to three parts that the embedding rows add up
    g.M = M0;
    g.K = 5 * H;
    g.a_t = false;
    g.B = W;
    g.ldb = E;
    g.C = nullptr;
    tail_add(a, g, w.dxp, 3);
    TailProblem& dx = a.p[a.n - 1];
    if (dx.splits == 1) {
        dx.g.C = w.dxp;
        dx.g.ldc = E;
    }
    a.dx = w.dxp;
    a.ldx = E;
    a.dx_parts = dx.splits;
    a.dx_stride = int64_t(M0) * E;
    a.src = w.dAp;
    a.ld = w.lda;
    a.rows = s.N;
    a.cols = 5 * H;
    a.sum_part = w.tsum;
    a.sum_out = db;
    a.demb = demb;
    a.demb_n = int64_t(d.V) * E;
    a.E = E;
    a.leaves = M0;
    a.nseg = nseg;
    a.seg = w.seg;
    return tail_run(a, "treelstm_bwd_tail", st);
}

// ------------------------------------------------------------------ TreeRNN
// Binary TreeRNN on the same frontier schedule: a leaf's h is its word
// vector (embedding width = H), an internal node h = tanh(W [h_L; h_R] + b).
// Forward: the leaves copy their embedding rows into their parents' [h_L;
// h_R] rows; each internal level is one contraction with W^T whose epilogue
// adds the bias, applies tanh, saves h and sends it to the parent.
// Backward, levels from the top down, one contraction per level: its a slab
// is da = dh (1 - h^2) (column block 0 also stores da) and its epilogue sends
// [dh_L; dh_R] = da W to the two children; after the loop dW = da^T HLR and
// db = column sums of da over the internal nodes, and the leaves' dh is the
// gradient of their word vectors.
struct TreeRnnWs {
    TreeWs s;                    // schedule arrays (lword .. rootpos, xgroup, tsync, seg) only
    float* A = nullptr;          // [N x H] pre-activations (forward), da (backward)
    float* Hn = nullptr;         // [N x H] h of every node
    float* HLR = nullptr;        // [N - M0 x 2H] children's h of internal nodes
    float* dh = nullptr;         // [N x H]
    float* Wt = nullptr;         // [2H x H] W transposed
    float* part = nullptr;
    // groups of trees per XCD: node rows padded to whole 128-byte lines
    float* hx = nullptr;         // [N x ldh] h of every node
    float* dAp = nullptr;        // [N x ldh]
    float* dx = nullptr;         // [N x H] gradient of the leaves' word vectors
    float* tpart = nullptr;      // parts of the two halves of dW
    float* tsum = nullptr;       // parts of db
    int64_t ldh = 0;
};

size_t carve_rnn(const janus_treelstm_desc& d, int32_t N, int32_t K, void* base, TreeRnnWs& w) {
    Carver c(base);
    const int H = d.H;
    w.s.lword = c.take<int32_t>(N);
    w.s.lchild = c.take<int32_t>(N);
    w.s.rchild = c.take<int32_t>(N);
    w.s.parent = c.take<int32_t>(N);
    w.s.rootk = c.take<int32_t>(N);
    w.s.rootpos = c.take<int32_t>(K);
    w.s.xgroup = take_cut(c, N);
    w.s.tsync = c.take<tpersist::TreeSync>(1);
    w.s.seg = c.take<int32_t>(int64_t(embed_seg_ints(N)));
    w.A = c.take<float>(int64_t(N) * H);
    w.Hn = c.take<float>(int64_t(N) * H);
    w.HLR = c.take<float>(int64_t(N) * 2 * H);
    w.dh = c.take<float>(int64_t(N) * H);
    w.Wt = c.take<float>(int64_t(2) * H * H);
    w.part = c.take<float>(colsum_partial_floats(H));
    w.ldh = round_up(H, 32);
    w.hx = c.take<float>(int64_t(N) * w.ldh);
    w.dAp = c.take<float>(int64_t(N) * w.ldh);
    w.dx = c.take<float>(int64_t(N) * H);
    w.tpart = c.take<float>(2 * tail_part_floats(H, H));
    w.tsum = c.take<float>(tail_sum_floats(N, H));
    return c.off + 256;
}

// h of node p (level-ordered) to its parent's [h_L; h_R] row or to h_root
__device__ __forceinline__ void rnn_send(int p, int j, int H, int M0, float h, const int32_t* parent,
                                         const int32_t* rootk, float* HLR, float* h_root) {
    const int par = parent[p];
    if (par >= 0) HLR[int64_t((par >> 1) - M0) * 2 * H + (par & 1) * H + j] = h;
    else h_root[int64_t(rootk[p]) * H + j] = h;
}

__global__ void treernn_leaf_kernel(int rows, int H, int M0, const int32_t* lword, const float* emb,
                                    const int32_t* parent, const int32_t* rootk, float* Hn, float* HLR,
                                    float* h_root) {
    const int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
    if (i >= int64_t(rows) * H) return;
    const int p = int(i / H), j = int(i % H);
    const float h = emb[int64_t(lword[p]) * H + j];
    Hn[i] = h;
    rnn_send(p, j, H, M0, h, parent, rootk, HLR, h_root);
}

janus_status check_rnn(const janus_treelstm_desc* d) {
    janus_status e = check(d);
    if (e != JANUS_OK) return e;
    return d->E == d->H ? JANUS_OK : JANUS_ERR_INVALID_ARG;
}

janus_status prepare_rnn(const janus_treelstm_desc* d, const janus_tree_batch* t, void* ws, size_t ws_bytes,
                         TreeSchedule& s, TreeRnnWs& w) {
    janus_status e = check_rnn(d);
    if (e != JANUS_OK) return e;
    if ((e = build_tree_schedule(t, d->V, s)) != JANUS_OK) return e;
    if (!ws || ws_bytes < carve_rnn(*d, s.N, t->num_trees, nullptr, w) || reinterpret_cast<uintptr_t>(ws) % 256 != 0)
        return JANUS_ERR_WORKSPACE;
    carve_rnn(*d, s.N, t->num_trees, ws, w);
    return JANUS_OK;
}

}  // namespace

}  // namespace janus

using namespace janus;

extern "C" size_t janus_treelstm_workspace_bytes(const janus_treelstm_desc* d, int32_t max_nodes,
                                                 int32_t max_trees) {
    if (check(d) != JANUS_OK || max_nodes <= 0 || max_trees <= 0) return 0;
    TreeWs w;
    return carve(*d, max_nodes, max_trees, nullptr, w);
}

extern "C" janus_status janus_treelstm_fwd(const janus_treelstm_desc* d, const janus_tree_batch* t, const void* emb,
                                           const void* W, const void* U, const void* b, void* h_root, void* ws,
                                           size_t ws_bytes, void* stream) {
    if (!emb || !W || !U || !b || !h_root) return JANUS_ERR_INVALID_ARG;
    TreeSchedule s;
    TreeWs w;
    janus_status e = prepare(d, t, ws, ws_bytes, s, w);
    if (e != JANUS_OK) return e;
    hipStream_t st = static_cast<hipStream_t>(stream);
    const TreeXcdPlan xp = tree_xcd_plan(*d, t, s);
    if (xp.on) return treelstm_fwd_xcd_call(*d, t, s, w, xp, emb, W, U, b, h_root, st);
    if ((e = upload_tree(t, s, w, st)) != JANUS_OK) return e;
    const int H = d->H, E = d->E;
    const int M0 = s.level_offsets[1];
    // the level contractions read W and U transposed (N = 5H contiguous)
    if ((e = transpose_f32(static_cast<const float*>(W), 5 * H, E, w.Wt, st)) != JANUS_OK) return e;
    if ((e = transpose_f32(static_cast<const float*>(U), 5 * H, 2 * H, w.Ut, st)) != JANUS_OK) return e;
    const float* bias = static_cast<const float*>(b);
    for (int k = 0; k < s.num_levels; ++k) {
        const int p0 = s.level_offsets[k], rows = s.level_offsets[k + 1] - p0;
        // A_k = a . W^T + b over the rows of level k: leaves gather their
        // embedding rows, internal nodes read [h_L; h_R]
        if (k == 0)
            e = simt_gemm<false, kSimtStore>("tree_level_gemm", rows, 5 * H, E, static_cast<const float*>(emb), E,
                                             w.lword, w.Wt, 5 * H, nullptr, bias, w.A, w.ld5, st);
        else
            e = simt_gemm<false, kSimtStore>("tree_level_gemm", rows, 5 * H, 2 * H,
                                             w.HLR + int64_t(p0 - M0) * 2 * H, 2 * H, nullptr, w.Ut, 5 * H, nullptr,
                                             bias, w.A + int64_t(p0) * w.ld5, w.ld5, st);
        if (e != JANUS_OK) return e;
        const int64_t n = int64_t(rows) * H;
        TraceScope trace("tree_fwd_point", 0.0, 4.0 * n * 14.0, st);
        hipLaunchKernelGGL(tree_fwd_point_kernel, dim3(unsigned((n + 255) / 256)), dim3(256), 0, st, p0, rows, H, M0,
                           w.ld5, w.A, w.G, w.C, w.lchild, w.rchild, w.parent, w.rootk, w.HLR,
                           static_cast<float*>(h_root));
        JANUS_LAUNCH_CHECK();
    }
    return JANUS_OK;
}

extern "C" janus_status janus_treelstm_bwd(const janus_treelstm_desc* d, const janus_tree_batch* t, const void* emb,
                                           const void* W, const void* U, void* ws, size_t ws_bytes,
                                           const void* dh_root, float* demb, float* dW, float* dU, float* db,
                                           void* stream) {
    if (!emb || !W || !U || !dh_root || !demb || !dW || !dU || !db) return JANUS_ERR_INVALID_ARG;
    TreeSchedule s;
    TreeWs w;
    janus_status e = prepare(d, t, ws, ws_bytes, s, w);
    if (e != JANUS_OK) return e;
    const int M0 = s.level_offsets[1];
    hipStream_t st = static_cast<hipStream_t>(stream);
    const TreeXcdPlan xp = tree_xcd_plan(*d, t, s);
    if (xp.on) return treelstm_bwd_xcd_call(*d, t, s, w, xp, W, U, dh_root, demb, dW, dU, db, st);
    std::vector<int32_t> words;
    if ((e = upload_tree(t, s, w, st, &words)) != JANUS_OK) return e;
    const int H = d->H, E = d->E, N = s.N;
    const int64_t kh = int64_t(t->num_trees) * H;
    {
    TraceScope trace("tree_bwd_init", 0.0, 12.0 * kh, st);
    hipLaunchKernelGGL(tree_bwd_init_kernel, dim3(unsigned((kh + 255) / 256)), dim3(256), 0, st, t->num_trees, H,
                       w.rootpos, static_cast<const float*>(dh_root), w.dh, w.dc);
    JANUS_LAUNCH_CHECK();
    }
    for (int k = s.num_levels - 1; k >= 0; --k) {
        const int p0 = s.level_offsets[k], rows = s.level_offsets[k + 1] - p0;
        const int64_t n = int64_t(rows) * H;
        if (k == 0) {
            TraceScope trace("tree_bwd_point", 0.0, 4.0 * n * 17.0, st);
            hipLaunchKernelGGL(tree_bwd_point_kernel, dim3(unsigned((n + 255) / 256)), dim3(256), 0, st, p0, rows, H,
                               w.ld5, w.G, w.C, w.dh, w.dc, w.lchild, w.rchild, w.A);
            JANUS_LAUNCH_CHECK();
            break;
        }
        if (5 * H > kSimtKc) {
            // gate columns do not fit one LDS slab: pointwise, then the contraction
            {
                TraceScope trace("tree_bwd_point", 0.0, 4.0 * n * 17.0, st);
                hipLaunchKernelGGL(tree_bwd_point_kernel, dim3(unsigned((n + 255) / 256)), dim3(256), 0, st, p0, rows,
                                   H, w.ld5, w.G, w.C, w.dh, w.dc, w.lchild, w.rchild, w.A);
                JANUS_LAUNCH_CHECK();
            }
            e = simt_gemm<false, kSimtChildren>("tree_dh_gemm", rows, 2 * H, 5 * H, w.A + int64_t(p0) * w.ld5, w.ld5,
                                                nullptr, static_cast<const float*>(U), 2 * H, nullptr, nullptr, w.dh,
                                                0, st, w.lchild + p0, w.rchild + p0, H);
            if (e != JANUS_OK) return e;
            continue;
        }
        // cell backward of the level and [dh_L; dh_R] = da U to the children
        dim3 grid(unsigned((2 * H + kSimtCols - 1) / kSimtCols), unsigned((rows + kSimtRows - 1) / kSimtRows));
        TraceScope trace("tree_bwd_level", 2.0 * rows * 2.0 * H * 5.0 * H,
                         4.0 * (double(rows) * 17.0 * H + 10.0 * H * H + 2.0 * rows * H), st);
        hipLaunchKernelGGL(tree_bwd_level_kernel, grid, dim3(64 * kSimtWaves), 0, st, p0, rows, H, w.ld5, w.G, w.C,
                           w.dh, w.dc, w.lchild, w.rchild, w.A, static_cast<const float*>(U), w.dh);
        JANUS_LAUNCH_CHECK();
    }
    // dU = da_int^T HLR  (K = internal nodes)
    e = simt_gemm<true, kSimtStore>("tree_dU_gemm", 5 * H, 2 * H, N - M0, w.A + int64_t(M0) * w.ld5, w.ld5, nullptr,
                                    w.HLR, 2 * H, nullptr, nullptr, dU, 2 * H, st);
    if (e != JANUS_OK) return e;
    // dW = da_leaf^T emb[word]  (K = leaves, gathered rows of emb)
    e = simt_gemm<true, kSimtStore>("tree_dW_gemm", 5 * H, E, M0, w.A, w.ld5, nullptr, static_cast<const float*>(emb),
                                    E, w.lword, nullptr, dW, E, st);
    if (e != JANUS_OK) return e;
    if ((e = colsum(JANUS_F32, w.A, N, 5 * H, w.ld5, db, w.part, st)) != JANUS_OK) return e;
    // dx_leaf = da_leaf W, then the embedding gradient
    e = simt_gemm<false, kSimtStore>("tree_dx_gemm", M0, E, 5 * H, w.A, w.ld5, nullptr, static_cast<const float*>(W), E,
                                     nullptr, nullptr, w.dxl, E, st);
    if (e != JANUS_OK) return e;
    return embed_backward(JANUS_F32, w.dxl, words.data(), M0, E, demb, d->V, w.seg, st);
}

extern "C" janus_status janus_treelstm_device_report(const janus_treelstm_desc* d, const janus_tree_batch* t,
                                                     const void* ws, size_t ws_bytes, int32_t* timed_out,
                                                     void* stream) {
    if (!timed_out) return JANUS_ERR_INVALID_ARG;
    TreeSchedule s;
    TreeWs w;
    janus_status e = prepare(d, t, const_cast<void*>(ws), ws_bytes, s, w);
    if (e != JANUS_OK) return e;
    unsigned flag = 0;
    JANUS_HIP(hipStreamSynchronize(static_cast<hipStream_t>(stream)));
    JANUS_HIP(hipMemcpy(&flag, &w.tsync->error, sizeof(flag), hipMemcpyDeviceToHost));
    *timed_out = flag != 0u ? 1 : 0;
    return flag != 0u ? JANUS_ERR_DEVICE : JANUS_OK;
}

namespace janus {
namespace {

// The TreeRNN in groups of trees per XCD: 16 units per forward workgroup (H up
// to 512 in the 32 workgroups of an XCD), [dh_L; dh_R] of 8 or 16 in the
// backward.  Off with JANUS_TREE_PERSIST=0; wider models run level by level.
struct RnnXcdPlan {
    bool on = false;
    int MT = 0, fwd_nu = 0, bwd_nu = 0;
    treex::Cut cut;
    size_t bwd_lds = 0;
};
size_t rnn_bwd_lds(int MT, int nodes) {
    return MT == 1 ? treex::RnnBwdCfg<1>::lds(nodes) : treex::RnnBwdCfg<2>::lds(nodes);
}
RnnXcdPlan rnn_xcd_plan(const janus_treelstm_desc& d, const janus_tree_batch* t, const TreeSchedule& s) {
    RnnXcdPlan p;
    if (tree_env("JANUS_TREE_PERSIST", '0')) return p;
    const TreeDev dev = tree_dev();
    if (dev.cus <= 0 || dev.lds == 0 || d.H > 512) return p;
    if (int64_t(s.N) * round_up(d.H, 32) * 4 >= (int64_t(1) << 31)) return p;   // 32-bit byte offsets
    p.MT = d.H <= 256 ? 1 : 2;
    p.fwd_nu = (d.H + treex::kRnnU - 1) / treex::kRnnU;
    p.bwd_nu = (d.H + 8 * p.MT - 1) / (8 * p.MT);
    const int capacity = treex::node_capacity(dev.lds, [&](int n) { return rnn_bwd_lds(p.MT, n); });
    p.on = cut_trees(t, s, treex::cut_shape(dev, std::max(p.fwd_nu, p.bwd_nu), capacity, false), p.cut);
    p.bwd_lds = rnn_bwd_lds(p.MT, p.cut.most_nodes);
    return p;
}

janus_status treernn_fwd_xcd_call(const janus_treelstm_desc& d, const janus_tree_batch* t, const TreeSchedule& s,
                                  const TreeRnnWs& w, const RnnXcdPlan& p, const void* emb, const void* W,
                                  const void* b, void* h_root, hipStream_t st) {
    janus_status e = upload_cut(t, s, w.s, p.cut, st);
    if (e != JANUS_OK) return e;
    const int M0 = s.level_offsets[1];
    treex::RnnFwd a = {};
    a.H = d.H;
    a.M0 = M0;
    a.nu = p.fwd_nu;
    a.xccs = tree_env("JANUS_XCD_REMOTE", '1') ? 0 : p.cut.xccs;
    a.tile = cut_tiles(w.s, p.cut);
    a.lchild = w.s.lchild;
    a.rchild = w.s.rchild;
    a.rootk = w.s.rootk;
    a.W = static_cast<const float*>(W);
    a.b = static_cast<const float*>(b);
    a.hx = w.hx;
    a.ldh = w.ldh;
    a.hx_bytes = uint32_t(int64_t(s.N) * w.ldh * 4);
    a.h_root = static_cast<float*>(h_root);
    a.sync = w.s.tsync;
    const int parts = int(p.cut.launch.size());
    for (int part = 0; part < parts; ++part) {
        if (part == 0) {
            TraceScope trace("tree_fwd_init", 0.0, 4.0 * double(s.N + M0) * w.ldh, st);
            hipLaunchKernelGGL(treex::rnn_fwd_init_kernel, dim3(fill_blocks(int64_t(s.N) * w.ldh)), dim3(256), 0, st,
                               s.N, M0, d.H, w.s.lword, w.s.rootk, static_cast<const float*>(emb), w.hx, w.ldh,
                               static_cast<float*>(h_root), w.s.tsync);
        } else {
            hipLaunchKernelGGL(treex::fill_kernel, dim3(4), dim3(256), 0, st, w.hx, w.ldh, int64_t(0), int64_t(0), d.H,
                               w.s.tsync);
        }
        JANUS_LAUNCH_CHECK();
        const treex::CutLaunch& l = p.cut.launch[part];
        a.group = w.s.xgroup + l.first;
        a.groups = l.groups;
        static size_t attr = 0;
        TraceScope trace("treernn_fwd_persistent", 2.0 * d.H * 2.0 * d.H * double(s.N - M0) / parts, 0.0, st);
        e = tree_persistent_launch(treex::treernn_fwd_xcd, p.cut.blocks(l, p.fwd_nu), treex::kRnnFwdLds, a, st, attr,
                                   treex::kThreads);
        if (e != JANUS_OK) return e;
    }
    return JANUS_OK;
}

template <int MT, bool PIECES>
janus_status launch_rnn_bwd(int blocks, size_t lds, const treex::RnnBwd& a, hipStream_t st) {
    static size_t attr = 0;
    return tree_persistent_launch(treex::treernn_bwd_xcd<MT, PIECES>, blocks, lds, a, st, attr, treex::kThreads);
}
template <int MT>
janus_status launch_rnn_bwd(const RnnXcdPlan& p, int blocks, const treex::RnnBwd& a, hipStream_t st) {
    return p.cut.split ? launch_rnn_bwd<MT, true>(blocks, p.bwd_lds, a, st)
                       : launch_rnn_bwd<MT, false>(blocks, p.bwd_lds, a, st);
}

// The schedule is the forward's (the workspace is unchanged between the calls).
janus_status treernn_bwd_xcd_call(const janus_treelstm_desc& d, const janus_tree_batch* t, const TreeSchedule& s,
                                  const TreeRnnWs& w, const RnnXcdPlan& p, const void* W, const void* dh_root,
                                  float* demb, float* dW, float* db, hipStream_t st) {
    const int M0 = s.level_offsets[1], Nint = s.N - M0, H = d.H;
    std::vector<int32_t> seg;
    const int nseg = leaf_segments(t, s, d.V, p.cut, seg);
    janus_status e = upload(w.s.seg, seg.data(), seg.size() * sizeof(int32_t), st);
    if (e != JANUS_OK) return e;
    treex::RnnBwd a = {};
    a.H = H;
    a.M0 = M0;
    a.nu = p.bwd_nu;
    a.xccs = tree_env("JANUS_XCD_REMOTE", '1') ? 0 : p.cut.xccs;
    a.tile = cut_tiles(w.s, p.cut);
    a.lchild = w.s.lchild;
    a.rchild = w.s.rchild;
    a.rootk = w.s.rootk;
    a.W = static_cast<const float*>(W);
    a.hx = w.hx;
    a.ldh = w.ldh;
    a.dh_root = static_cast<const float*>(dh_root);
    a.dhx = w.dh;
    a.dA = w.dAp;
    a.dA_bytes = uint32_t(int64_t(s.N) * w.ldh * 4);
    a.dx = w.dx;
    a.sync = w.s.tsync;
    const int parts = int(p.cut.launch.size());
    for (int part = parts; part-- > 0;) {   // parents before the pieces below them
        if (part == parts - 1) {
            TraceScope trace("tree_bwd_init", 0.0, 4.0 * double(Nint) * w.ldh, st);
            hipLaunchKernelGGL(treex::rnn_bwd_init_kernel, dim3(fill_blocks(int64_t(Nint) * w.ldh + 4096)), dim3(256), 0,
                               st, s.N, M0, H, w.s.rootpos, t->num_trees, a.dh_root, w.dAp, w.ldh, w.dx, w.s.tsync);
        } else {
            hipLaunchKernelGGL(treex::fill_kernel, dim3(4), dim3(256), 0, st, w.dAp, w.ldh, int64_t(0), int64_t(0), H,
                               w.s.tsync);
        }
        JANUS_LAUNCH_CHECK();
        const treex::CutLaunch& l = p.cut.launch[part];
        a.group = w.s.xgroup + l.first;
        a.groups = l.groups;
        const int blocks = p.cut.blocks(l, p.bwd_nu);
        TraceScope trace("treernn_bwd_persistent", 2.0 * H * 2.0 * H * double(Nint) / parts, 0.0, st);
        e = p.MT == 1 ? launch_rnn_bwd<1>(p, blocks, a, st) : launch_rnn_bwd<2>(p, blocks, a, st);
        if (e != JANUS_OK) return e;
    }
    // dW = dA_int^T [h_L; h_R], the children's rows gathered; db; demb
    TailArgs q;
    GemmDesc g;
    g.dtype = JANUS_F32;
    g.M = g.N = H;
    g.K = Nint;
    g.a_t = g.b_t = true;
    g.A = w.dAp + int64_t(M0) * w.ldh;
    g.lda = w.ldh;
    g.B = w.hx;
    g.ldb = w.ldh;
    g.b_idx = w.s.lchild + M0;
    g.C = dW;
    g.ldc = 2 * H;
    tail_add(q, g, w.tpart);
    g.b_idx = w.s.rchild + M0;
    g.C = dW + H;
    tail_add(q, g, w.tpart + tail_part_floats(H, H));
    q.src = w.dAp + int64_t(M0) * w.ldh;
    q.ld = w.ldh;
    q.rows = Nint;
    q.cols = H;
    q.sum_part = w.tsum;
    q.sum_out = db;
    q.demb = demb;
    q.demb_n = int64_t(d.V) * H;
    q.dx = w.dx;
    q.ldx = H;
    q.E = H;
    q.leaves = M0;
    q.nseg = nseg;
    q.seg = w.s.seg;
    return tail_run(q, "treernn_bwd_tail", st);
}

}  // namespace
}  // namespace janus

extern "C" size_t janus_treernn_workspace_bytes(const janus_treernn_desc* d, int32_t max_nodes, int32_t max_trees) {
    if (check_rnn(d) != JANUS_OK || max_nodes <= 0 || max_trees <= 0) return 0;
    TreeRnnWs w;
    return carve_rnn(*d, max_nodes, max_trees, nullptr, w);
}

extern "C" janus_status janus_treernn_fwd(const janus_treernn_desc* d, const janus_tree_batch* t, const void* emb,
                                          const void* W, const void* b, void* h_root, void* ws, size_t ws_bytes,
                                          void* stream) {
    if (!emb || !W || !b || !h_root) return JANUS_ERR_INVALID_ARG;
    TreeSchedule s;
    TreeRnnWs w;
    janus_status e = prepare_rnn(d, t, ws, ws_bytes, s, w);
    if (e != JANUS_OK) return e;
    hipStream_t st = static_cast<hipStream_t>(stream);
    const RnnXcdPlan xp = rnn_xcd_plan(*d, t, s);
    if (xp.on) return treernn_fwd_xcd_call(*d, t, s, w, xp, emb, W, b, h_root, st);
    if ((e = upload_tree(t, s, w.s, st)) != JANUS_OK) return e;
    const int H = d->H;
    const int M0 = s.level_offsets[1];
    float* hr = static_cast<float*>(h_root);
    // the level contractions read W transposed (N = H contiguous)
    if ((e = transpose_f32(static_cast<const float*>(W), H, 2 * H, w.Wt, st)) != JANUS_OK) return e;
    {
        const int64_t n = int64_t(M0) * H;
        TraceScope trace("treernn_leaf", 0.0, 12.0 * n, st);
        hipLaunchKernelGGL(treernn_leaf_kernel, dim3(unsigned((n + 255) / 256)), dim3(256), 0, st, M0, H, M0,
                           w.s.lword, static_cast<const float*>(emb), w.s.parent, w.s.rootk, w.Hn, w.HLR, hr);
        JANUS_LAUNCH_CHECK();
    }
    SimtExtra send;
    send.HLR = w.HLR;
    send.root = hr;
    send.M0 = M0;
    for (int k = 1; k < s.num_levels; ++k) {
        const int p0 = s.level_offsets[k], rows = s.level_offsets[k + 1] - p0;
        // h = tanh([h_L; h_R] W^T + b), saved and sent on (parent slot and tree
        // index of each row through the epilogue's index arguments)
        e = simt_gemm<false, kSimtTanhSend>("treernn_level", rows, H, 2 * H, w.HLR + int64_t(p0 - M0) * 2 * H, 2 * H,
                                            nullptr, w.Wt, H, nullptr, static_cast<const float*>(b),
                                            w.Hn + int64_t(p0) * H, H, st, w.s.parent + p0, w.s.rootk + p0, H, send);
        if (e != JANUS_OK) return e;
    }
    return JANUS_OK;
}

extern "C" janus_status janus_treernn_bwd(const janus_treernn_desc* d, const janus_tree_batch* t, const void* W,
                                          void* ws, size_t ws_bytes, const void* dh_root, float* demb, float* dW,
                                          float* db, void* stream) {
    if (!W || !dh_root || !demb || !dW || !db) return JANUS_ERR_INVALID_ARG;
    TreeSchedule s;
    TreeRnnWs w;
    janus_status e = prepare_rnn(d, t, ws, ws_bytes, s, w);
    if (e != JANUS_OK) return e;
    const int M0 = s.level_offsets[1];
    hipStream_t st = static_cast<hipStream_t>(stream);
    const RnnXcdPlan xp = rnn_xcd_plan(*d, t, s);
    if (xp.on) return treernn_bwd_xcd_call(*d, t, s, w, xp, W, dh_root, demb, dW, db, st);
    std::vector<int32_t> words;
    if ((e = upload_tree(t, s, w.s, st, &words)) != JANUS_OK) return e;
    const int H = d->H, N = s.N;
    const int64_t kh = int64_t(t->num_trees) * H;
    {
        // dh of the roots (the dc half of this kernel's output is unused here)
        TraceScope trace("tree_bwd_init", 0.0, 12.0 * kh, st);
        hipLaunchKernelGGL(tree_bwd_init_kernel, dim3(unsigned((kh + 255) / 256)), dim3(256), 0, st, t->num_trees, H,
                           w.s.rootpos, static_cast<const float*>(dh_root), w.dh, w.A);
        JANUS_LAUNCH_CHECK();
    }
    for (int k = s.num_levels - 1; k >= 1; --k) {
        const int p0 = s.level_offsets[k], rows = s.level_offsets[k + 1] - p0;
        // da = dh (1 - h^2) as the a slab (stored by column block 0), and
        // [dh_L; dh_R] = da W to the children (W rows are N = 2H contiguous)
        SimtExtra tg;
        tg.S = w.Hn + int64_t(p0) * H;
        tg.D = w.A + int64_t(p0) * H;
        e = simt_gemm<false, kSimtChildren, kSimtTanhGrad>("treernn_level_bwd", rows, 2 * H, H, w.dh + int64_t(p0) * H,
                                                           H, nullptr, static_cast<const float*>(W), 2 * H, nullptr,
                                                           nullptr, w.dh, 0, st, w.s.lchild + p0, w.s.rchild + p0, H,
                                                           tg);
        if (e != JANUS_OK) return e;
    }
    // dW = da_int^T HLR  (K = internal nodes), db = column sums of da_int
    e = simt_gemm<true, kSimtStore>("treernn_dW_gemm", H, 2 * H, N - M0, w.A + int64_t(M0) * H, H, nullptr, w.HLR,
                                    2 * H, nullptr, nullptr, dW, 2 * H, st);
    if (e != JANUS_OK) return e;
    if (N > M0) {
        if ((e = colsum(JANUS_F32, w.A + int64_t(M0) * H, N - M0, H, H, db, w.part, st)) != JANUS_OK) return e;
    } else if ((e = zero_fill(db, sizeof(float) * H, st)) != JANUS_OK) {
        return e;
    }
    // the leaves' dh is the gradient of their word vectors
    return embed_backward(JANUS_F32, w.dh, words.data(), M0, H, demb, d->V, w.s.seg, st);
}

extern "C" janus_status janus_treernn_device_report(const janus_treernn_desc* d, const janus_tree_batch* t,
                                                    const void* ws, size_t ws_bytes, int32_t* timed_out,
                                                    void* stream) {
    if (!timed_out) return JANUS_ERR_INVALID_ARG;
    TreeSchedule s;
    TreeRnnWs w;
    janus_status e = prepare_rnn(d, t, const_cast<void*>(ws), ws_bytes, s, w);
    if (e != JANUS_OK) return e;
    unsigned flag = 0;
    JANUS_HIP(hipStreamSynchronize(static_cast<hipStream_t>(stream)));
    JANUS_HIP(hipMemcpy(&flag, &w.s.tsync->error, sizeof(flag), hipMemcpyDeviceToHost));
    *timed_out = flag != 0u ? 1 : 0;
    return flag != 0u ? JANUS_ERR_DEVICE : JANUS_OK;
}
