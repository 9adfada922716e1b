// Tree level programs whose groups of trees each live on one XCD.
//
// Trees of a batch are independent, so a level's exchange of h (forward) or
// of the pre-activation gradients (backward) is needed only among the
// workgroups that work the same trees.  The batch is cut in groups of whole
// trees, one per XCD, worked by NU workgroups (at most the CUs of an XCD) of
// that XCD; workgroup m owns units [U m, U m + U), keeps their weights in
// VGPRs for the whole launch, and handles them for every node of its group.
// The nodes go through in tiles of 16, level by level.
//
// What bounds a level is the chain "publish -> load -> MFMA -> sum over the
// waves -> cell"; its MFMA work is under 1 us at H 150.  A device-wide barrier
// per level (about 2 us, after write-through stores) is replaced by the data
// itself, as in the LSTM recurrence: a row that other workgroups read is
// prefilled with a pattern no result takes, stored once, and loaded until no
// word holds the pattern, all in the XCD's L2.  Everything else a node needs
// from its children or parent (c, dc, dh of the owned units) stays in the LDS
// of the workgroup that owns the unit.
//
// A tree that is larger than a group may be, or so large that the other XCDs
// would wait for it, runs in pieces (tree_cut.hpp): subtrees in one launch, what
// is above them in the next, the backward in the opposite order.  At the cuts a
// node's values go through memory (`PIECES`): c, and G of the Child-Sum, up; dh
// and dc down.  Step of one tree, whole (level by level where it fits no
// group), and in pieces, against the kernels with a device-wide barrier:
// TreeLSTM H 150, 600 leaves 531 and 249 against 435 us, 1200 leaves 778 and
// 333 against 567; TreeRNN H 300, 1200 leaves 635 and 215 against 401;
// Child-Sum H 150, 1200 nodes 677 and 289 against 506.
//
// Measured, forward and backward levels of the binary TreeLSTM against the
// kernels with a device-wide barrier per level: 25 trees of 5-50 leaves, H
// 150: 61 and 58 us against 116 and about 120; 100 trees, H 300, against one
// launch per level: 282 and 252 us against 950 and 720.
#pragma once

#include "lstm_xcd.hpp"
#include "tree_common.hpp"
#include "tree_cut.hpp"

namespace janus {
namespace treex {

using persist::kOutOfRange;
using persist::make_rsrc;
using tpersist::TreeSync;
using xcd::f32x4_t;
using xcd::kEmpty;
using xcd::not_empty;

constexpr int kThreads = xcd::kThreads;
constexpr int kWaves = xcd::kWaves;
constexpr int kPieceRoot = -2;   // in place of a root's tree index: the parent runs in another launch

__device__ __forceinline__ int tile_rows(Tile t) { return t.rows_level & 0xff; }
__device__ __forceinline__ int tile_level(Tile t) { return t.rows_level >> 8; }
// The tiles of a group, read 64 at a time into one register of the wave, so
// that a tile's extent costs no load when its turn comes.
struct TileWindow {
    const Tile* tile;
    int base, end;     // tiles [base, base + 64) of those below `end` are held
    int p0, rl;        // this lane's tile
    __device__ __forceinline__ void load(int first) {
        base = first;
        const int i = min(max(first + int(threadIdx.x & 63), 0), end - 1);
        p0 = tile[i].p0;
        rl = tile[i].rows_level;
    }
    __device__ __forceinline__ void init(const Tile* t, int e, int first) {
        tile = t;
        end = e;
        load(first);
    }
    // tile i (the same for every lane); `down`: a miss loads the 64 tiles that end with it
    __device__ __forceinline__ Tile at(int i, bool down = false) {
        if (i < base || i >= base + 64) load(down ? max(i - 63, 0) : i);
        Tile r;
        r.p0 = __builtin_amdgcn_readlane(p0, i - base);
        r.rows_level = __builtin_amdgcn_readlane(rl, i - base);
        return r;
    }
};
// Whether a position is one of the group's nodes (in a launch of pieces of
// trees a child or parent may have run, or run later, in another one).
__device__ __forceinline__ bool inside(const Group& g, int M0, int p) {
    return p < M0 ? unsigned(p - g.leaf0) < unsigned(g.nleaf) : unsigned(p - g.int0) < unsigned(g.nint);
}
// index of a position among its group's nodes
__device__ __forceinline__ int local_of(const Group& g, int M0, int p) {
    return p < M0 ? p - g.leaf0 : g.nleaf + p - g.int0;
}

// ------------------------------------------------------------------ set-up
// Rows [r0, r0 + rows) of a row array of pitch ld: columns below `cols` hold
// the pattern, the padding zero.
__device__ __forceinline__ void fill_empty(float* a, int64_t ld, int64_t r0, int64_t rows, int cols, int64_t i0,
                                           int64_t stride) {
    const int q = int(ld / 4);   // 16-byte pieces of a row
    uint4* d = reinterpret_cast<uint4*>(a + r0 * ld);
    for (int64_t i = i0; i < rows * q; i += stride) {
        const int c = 4 * int(i % q);
        d[i] = make_uint4(c < cols ? kEmpty : 0u, c + 1 < cols ? kEmpty : 0u, c + 2 < cols ? kEmpty : 0u,
                          c + 3 < cols ? kEmpty : 0u);
    }
}
__device__ __forceinline__ void zero_counters(TreeSync* s, int64_t i0, int64_t stride) {
    uint32_t* c = reinterpret_cast<uint32_t*>(reinterpret_cast<char*>(s) + tpersist::kTreeSyncCounters);
    for (int64_t i = i0; i < int64_t((sizeof(TreeSync) - tpersist::kTreeSyncCounters) / 4); i += stride) c[i] = 0u;
}
// Empty rows and zero counters (not the error flag).
static __global__ __launch_bounds__(256) void fill_kernel(float* a, int64_t ld, int64_t r0, int64_t rows, int cols,
                                                   TreeSync* s) {
    const int64_t i0 = int64_t(blockIdx.x) * 256 + threadIdx.x, stride = int64_t(gridDim.x) * 256;
    zero_counters(s, i0, stride);
    fill_empty(a, ld, r0, rows, cols, i0, stride);
}
// Forward: the leaves' word vectors gathered into padded rows x (pitch ldx,
// zero past E), every node's row of h empty, counters and error flag zero.
static __global__ __launch_bounds__(256) void fwd_init_kernel(int N, int M0, int E, const int32_t* lword, const float* emb,
                                                       float* x, int64_t ldx, float* hx, int64_t ldh, int H,
                                                       TreeSync* s) {
    const int64_t i0 = int64_t(blockIdx.x) * 256 + threadIdx.x, stride = int64_t(gridDim.x) * 256;
    zero_counters(s, i0, stride);
    if (i0 == 0) s->error = 0u;
    fill_empty(hx, ldh, 0, N, H, i0, stride);
    for (int64_t i = i0; i < int64_t(M0) * ldx; i += stride) {
        const int p = int(i / ldx), e = int(i % ldx);
        x[i] = e < E ? emb[int64_t(lword[p]) * E + e] : 0.f;
    }
}

// Sum of the waves' partial values of element (m, n) of the row tiles: the
// partial tiles lie [wave][tile][lane][4], lane l holding rows 4 (l / 16) + v,
// column l % 16.
template <int NT>
__device__ __forceinline__ float sum_waves(const float* red, int m, int n) {
    const int o = ((m >> 4) * 64 + ((m & 15) >> 2) * 16 + n) * 4 + (m & 3);
    float s = 0.f;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) s += red[w * NT * 256 + o];
    return s;
}

// A weight fragment: row r of a [rows x K] matrix of pitch ld, columns k ..
// k + 3, zero for r < 0 and past K.
__device__ __forceinline__ uint4 weight4(const float* W, int64_t ld, int r, int k, int K) {
    uint4 v = make_uint4(0, 0, 0, 0);
    if (r >= 0 && k < K) {
        const float* p = W + int64_t(r) * ld + k;
        v.x = __float_as_uint(p[0]);
        if (k + 1 < K) v.y = __float_as_uint(p[1]);
        if (k + 2 < K) v.z = __float_as_uint(p[2]);
        if (k + 3 < K) v.w = __float_as_uint(p[3]);
    }
    return v;
}

// ------------------------------------------------------- TreeLSTM, forward
struct LstmFwd {
    int E, H, M0;
    int groups, nu, xccs;
    const Group* group;        // of this launch
    const Tile* tile;
    const int32_t* lchild;
    const int32_t* rchild;
    const int32_t* parent;     // 2 * position + side, -1 for roots
    const int32_t* rootk;
    const float* W;            // [5H x E]
    const float* U;            // [5H x 2H]
    const float* b;
    const float* x;            // [M0 x ldx] leaf inputs
    int64_t ldx;
    uint32_t x_bytes;
    float* hx;                 // [N x ldh] h of every node (exchange)
    int64_t ldh;
    uint32_t hx_bytes;
    float* G;                  // [N x ldg] gates after activation, gate-major
    int64_t ldg;
    float* C;                  // [N x ldc]
    int64_t ldc;
    float* HLR;                // [(N - M0) x ldl]
    int64_t ldl;
    float* h_root;
    TreeSync* sync;
};

// NT 16-row tiles hold the 5 gates of U = floor(16 NT / 5) units.  The waves
// split the k-groups of 16 (left child's h, right child's h; or the leaf
// input): at most J per wave.
template <int NT>
struct LstmFwdCfg {
    static constexpr int U = 16 * NT / 5;
    static constexpr int J = NT <= 2 ? 4 : NT == 3 ? 5 : 6;
    static constexpr int RED = kWaves * NT * 256;   // floats of one set of partial tiles
    // cells' c of the group's nodes follow the two sets
    static size_t lds(int nodes) { return sizeof(float) * (2 * size_t(RED) + size_t(nodes) * U); }
};

template <int NT, bool PIECES>
__global__ __launch_bounds__(kThreads) void treelstm_fwd_xcd(LstmFwd a) {
    using C = LstmFwdCfg<NT>;
    constexpr int U = C::U, J = C::J;
    extern __shared__ __align__(16) float sm[];
    float* cl = sm + 2 * C::RED;   // [nodes][U]
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int lr = lane & 15, lq = lane >> 4;
    const xcd::Place pl = xcd::take_place(a.sync, a.nu, a.groups, a.xccs);
    const int g = __builtin_amdgcn_readfirstlane(pl.g), m = __builtin_amdgcn_readfirstlane(pl.m);
    const bool local = __builtin_amdgcn_readfirstlane(pl.local) != 0;
    if (g < 0) return;
    const Group gr = a.group[g];
    if (gr.t0 >= gr.t1) return;   // a group without trees
    const int H = a.H, E = a.E, v0 = m * U;
    const int KH = (H + 15) / 16;   // k-groups of one child

    // row m of tile i: gate r % 5 of unit v0 + r / 5, r = 16 i + lr
    uint4 w[NT][J];
    auto gate_row = [&](int i) -> int {
        const int r = 16 * i + lr, u = v0 + r / 5;
        return r < 5 * U && u < H ? (r % 5) * H + u : -1;
    };
    // this wave's k-groups of nk: [kw0, kw1), at most J
    auto share = [&](int nk, int& k0, int& k1) {
        k0 = wave * nk / kWaves;
        k1 = (wave + 1) * nk / kWaves;
    };
    int kw0, kw1;
    share((E + 15) / 16, kw0, kw1);
#pragma unroll
    for (int i = 0; i < NT; ++i)
#pragma unroll
        for (int j = 0; j < J; ++j)
            w[i][j] = kw0 + j < kw1 ? weight4(a.W, E, gate_row(i), 16 * (kw0 + j) + 4 * lq, E) : make_uint4(0, 0, 0, 0);

    // cells: thread (unit cu, node cn) of the tile
    const int cu = tid >> 4, cn = tid & 15, cj = v0 + cu;
    const bool cell_thread = cu < U && cj < H;
    float bias[5];
#pragma unroll
    for (int q = 0; q < 5; ++q) bias[q] = cell_thread ? a.b[q * H + cj] : 0.f;

    bool dead = false;
    unsigned phase = 0;
    TileWindow win;
    win.init(a.tile, gr.t1, gr.t0);
    // a tile's links, loaded while the tile before it is worked: the operand
    // rows of this lane's node, and the cell's children, parent and root slot
    struct Links {
        int ql, qr, lc, rc, par, rk;
    };
    auto links = [&](int t) {
        const Tile tl = win.at(t);
        Links k;
        const int q = tl.p0 + min(lr, tile_rows(tl) - 1), p = tl.p0 + min(cn, tile_rows(tl) - 1);
        k.ql = a.lchild[q];
        k.qr = a.rchild[q];
        k.lc = a.lchild[p];
        k.rc = a.rchild[p];
        k.par = a.parent[p];
        k.rk = a.rootk[p];
        return k;
    };
    Links next = links(gr.t0);
    for (int t = gr.t0; t < gr.t1; ++t) {
        const Tile tl = win.at(t);
        const int rows = tile_rows(tl), ti = t - gr.t0;
        const bool leaf = ti < gr.leaf_tiles;
        if (ti == gr.leaf_tiles) {   // the internal nodes' weights
            share(2 * KH, kw0, kw1);
#pragma unroll
            for (int i = 0; i < NT; ++i)
#pragma unroll
                for (int j = 0; j < J; ++j) {
                    const int kg = kw0 + j, side = kg >= KH;
                    const int k = 16 * (kg - side * KH) + 4 * lq;
                    w[i][j] = kg < kw1 ? weight4(a.U + side * H, 2 * H, gate_row(i), k, H) : make_uint4(0, 0, 0, 0);
                }
        }
        const Links k = next;
        const int p = tl.p0 + cn;
        const bool cell = cell_thread && cn < rows;
        f32x4_t acc[NT];
#pragma unroll
        for (int i = 0; i < NT; ++i) acc[i] = f32x4_t{0.f, 0.f, 0.f, 0.f};
        // c of children that an earlier launch worked
        float xl = 0.f, xr = 0.f;
        if (PIECES && cell && !leaf) {
            if (!inside(gr, a.M0, k.lc)) xl = a.C[int64_t(k.lc) * a.ldc + cj];
            if (!inside(gr, a.M0, k.rc)) xr = a.C[int64_t(k.rc) * a.ldc + cj];
        }
        uint4 f[J];
        if (leaf) {
            const auto rs = make_rsrc(a.x, a.x_bytes);
            xcd::load_operand<float>(f, rs, [&](int j) {
                const int kg = kw0 + j;
                return lr < rows && kg < kw1
                           ? (uint32_t(tl.p0 + lr) * uint32_t(a.ldx) + uint32_t(16 * kg + 4 * lq)) * 4u
                           : kOutOfRange;
            }, false, a.sync, dead);
        } else {
            if (!local) xcd::remote_barrier(a.sync, g, phase, unsigned(a.nu));
            const auto rs = make_rsrc(a.hx, a.hx_bytes);
            const uint32_t ol = uint32_t(k.ql) * uint32_t(a.ldh), orr = uint32_t(k.qr) * uint32_t(a.ldh);
            xcd::load_operand<float>(f, rs, [&](int j) {
                const int kg = kw0 + j;
                const uint32_t o = kg < KH ? ol + uint32_t(16 * kg) : orr + uint32_t(16 * (kg - KH));
                return lr < rows && kg < kw1 ? (o + uint32_t(4 * lq)) * 4u : kOutOfRange;
            }, local, a.sync, dead);
        }
        if (t + 1 < gr.t1) next = links(t + 1);
#pragma unroll
        for (int j = 0; j < J; ++j)
#pragma unroll
            for (int i = 0; i < NT; ++i) acc[i] = xcd::mma(w[i][j], f[j], acc[i], static_cast<const float*>(nullptr));
        float* red = sm + (t & 1) * C::RED;
#pragma unroll
        for (int i = 0; i < NT; ++i) reinterpret_cast<f32x4_t*>(red)[(wave * NT + i) * 64 + lane] = acc[i];
        __syncthreads();
        if (cell) {
            float z[5];
#pragma unroll
            for (int q = 0; q < 5; ++q) z[q] = bias[q] + sum_waves<NT>(red, 5 * cu + q, cn);
            const float gi = sigmoidf_(z[0]), gl = sigmoidf_(z[1]), gr_ = sigmoidf_(z[2]), go = sigmoidf_(z[3]);
            const float gu = tanhf_(z[4]);
            float c = gi * gu;
            if (!leaf) {
                if (!PIECES || inside(gr, a.M0, k.lc)) xl = cl[local_of(gr, a.M0, k.lc) * U + cu];
                if (!PIECES || inside(gr, a.M0, k.rc)) xr = cl[local_of(gr, a.M0, k.rc) * U + cu];
                c += gl * xl + gr_ * xr;
            }
            const float h = go * tanhf_(c);
            // published for the tiles above
            if (k.par >= 0)
                xcd::store_b32(make_rsrc(a.hx, a.hx_bytes), (uint32_t(p) * uint32_t(a.ldh) + uint32_t(cj)) * 4u,
                               not_empty(__float_as_uint(h)));
            cl[local_of(gr, a.M0, p) * U + cu] = c;
            a.C[int64_t(p) * a.ldc + cj] = c;
            float* gp = a.G + int64_t(p) * a.ldg + cj;
            gp[0] = gi;
            gp[H] = gl;
            gp[2 * H] = gr_;
            gp[3 * H] = go;
            gp[4 * H] = gu;
            if (k.par >= 0) a.HLR[int64_t((k.par >> 1) - a.M0) * a.ldl + (k.par & 1) * H + cj] = h;
            else a.h_root[int64_t(k.rk) * H + cj] = h;
        }
    }
}

// ------------------------------------------------------ TreeLSTM, backward
struct LstmBwd {
    int H, M0;
    int groups, nu, xccs;
    const Group* group;
    const Tile* tile;          // the forward's tiles, walked backwards
    const int32_t* lchild;
    const int32_t* rchild;
    const int32_t* rootk;
    const float* U;
    const float* G;
    int64_t ldg;
    const float* C;
    int64_t ldc;
    const float* dh_root;
    float* dhx;                // [N x H] dh and dc of the roots of pieces, from the parents' launch
    float* dcx;
    float* dA;                 // [N x lda] gate-major; internal rows are the exchange
    int64_t lda;
    uint32_t dA_bytes;
    TreeSync* sync;
};

// MT 16-row tiles hold [dh_L; dh_R] of U = 8 MT units (row 2 u + side); K =
// 5H gate columns in k-groups of 16, at most J per wave.
template <int MT>
struct LstmBwdCfg {
    static constexpr int U = 8 * MT;
    static constexpr int J = MT == 1 ? 10 : 15;
    static constexpr int RED = kWaves * MT * 256;
    // then dh and dc of the group's nodes, [nodes][U] each
    static size_t lds(int nodes) { return sizeof(float) * (2 * size_t(RED) + 2 * size_t(nodes) * U); }
};

template <int MT, bool PIECES>
__global__ __launch_bounds__(kThreads) void treelstm_bwd_xcd(LstmBwd a) {
    using C = LstmBwdCfg<MT>;
    constexpr int U = C::U, J = C::J;
    extern __shared__ __align__(16) float sm[];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int lr = lane & 15, lq = lane >> 4;
    const xcd::Place pl = xcd::take_place(a.sync, a.nu, a.groups, a.xccs);
    const int g = __builtin_amdgcn_readfirstlane(pl.g), m = __builtin_amdgcn_readfirstlane(pl.m);
    const bool local = __builtin_amdgcn_readfirstlane(pl.local) != 0;
    if (g < 0) return;
    const Group gr = a.group[g];
    if (gr.t0 >= gr.t1) return;   // a group without trees
    float* dhl = sm + 2 * C::RED;                          // [nodes][U]
    float* dcl = dhl + int64_t(gr.nleaf + gr.nint) * U;    // [nodes][U]
    const int H = a.H, K = 5 * H, v0 = m * U;
    const int nk = (K + 15) / 16, kw0 = wave * nk / kWaves, kw1 = (wave + 1) * nk / kWaves;

    // row r = 16 i + lr: column side * H + unit of U, unit v0 + r / 2, side r % 2
    uint4 w[MT][J];
#pragma unroll
    for (int i = 0; i < MT; ++i)
#pragma unroll
        for (int j = 0; j < J; ++j) {
            const int r = 16 * i + lr, u = v0 + (r >> 1), k = 16 * (kw0 + j) + 4 * lq;
            float tmp[4];
#pragma unroll
            for (int e = 0; e < 4; ++e)
                tmp[e] = u < H && kw0 + j < kw1 && k + e < K ? a.U[int64_t(k + e) * 2 * H + (r & 1) * H + u] : 0.f;
            w[i][j] = make_uint4(__float_as_uint(tmp[0]), __float_as_uint(tmp[1]), __float_as_uint(tmp[2]),
                                 __float_as_uint(tmp[3]));
        }

    // cells: thread (unit cu, node cn); their inputs are loaded a tile ahead
    const int cu = tid >> 4, cn = tid & 15, cj = v0 + cu;
    const bool cell_thread = cu < U && cj < H;
    struct In {
        int p, lc, rc, rk;
        int ch;                          // child of this thread's element of [dh_L; dh_R]
        float g[5], c, cl, cr, dhr, dcr;
    } in;
    TileWindow win;
    win.init(a.tile, gr.t1, max(gr.t1 - 64, gr.t0));
    auto fetch = [&](int t, In& x) {
        const Tile tl = win.at(t, true);
        {
            const int q = tl.p0 + min(tid & 15, tile_rows(tl) - 1);
            x.ch = (tid >> 4 & 1) ? a.rchild[q] : a.lchild[q];
        }
        const bool ok = cell_thread && cn < tile_rows(tl);
        x.p = ok ? tl.p0 + cn : -1;
        const int p = ok ? x.p : tl.p0, j = cell_thread ? cj : 0;
        x.lc = a.lchild[p];
        x.rc = a.rchild[p];
        x.rk = a.rootk[p];
        const float* gp = a.G + int64_t(p) * a.ldg + j;
#pragma unroll
        for (int q = 0; q < 5; ++q) x.g[q] = gp[q * H];
        x.c = a.C[int64_t(p) * a.ldc + j];
        x.cl = a.C[int64_t(x.lc >= 0 ? x.lc : p) * a.ldc + j];
        x.cr = a.C[int64_t(x.rc >= 0 ? x.rc : p) * a.ldc + j];
        x.dhr = x.rk >= 0 ? a.dh_root[int64_t(x.rk) * H + j] : 0.f;
        x.dcr = 0.f;
        if (PIECES && x.rk == kPieceRoot) {
            x.dhr = a.dhx[int64_t(p) * H + j];
            x.dcr = a.dcx[int64_t(p) * H + j];
        }
    };
    // cell backward of a tile: dA published (internal) or stored (leaves),
    // the children's dc into LDS
    auto cells = [&](const In& x) {
        if (x.p < 0) return;
        const int lo = local_of(gr, a.M0, x.p) * U + cu;
        const bool leaf = x.p < a.M0;
        const float dh = x.rk != -1 ? x.dhr : dhl[lo], dc = x.rk != -1 ? x.dcr : dcl[lo];
        const float gi = x.g[0], gl = x.g[1], gr_ = x.g[2], go = x.g[3], gu = x.g[4];
        const float tau = tanhf_(x.c);
        const float d_o = dh * tau;
        const float dct = dc + dh * go * (1.f - tau * tau);
        float da[5];
        da[0] = dct * gu * gi * (1.f - gi);
        da[1] = leaf ? 0.f : dct * x.cl * gl * (1.f - gl);
        da[2] = leaf ? 0.f : dct * x.cr * gr_ * (1.f - gr_);
        da[3] = d_o * go * (1.f - go);
        da[4] = dct * gi * (1.f - gu * gu);
        const auto rs = make_rsrc(a.dA, a.dA_bytes);
        const uint32_t o = (uint32_t(x.p) * uint32_t(a.lda) + uint32_t(cj)) * 4u;
#pragma unroll
        for (int q = 0; q < 5; ++q)
            xcd::store_b32(rs, o + uint32_t(q) * uint32_t(H) * 4u, not_empty(__float_as_uint(da[q])));
        if (!leaf) {
            if (!PIECES || inside(gr, a.M0, x.lc)) dcl[local_of(gr, a.M0, x.lc) * U + cu] = dct * gl;
            else a.dcx[int64_t(x.lc) * H + cj] = dct * gl;
            if (!PIECES || inside(gr, a.M0, x.rc)) dcl[local_of(gr, a.M0, x.rc) * U + cu] = dct * gr_;
            else a.dcx[int64_t(x.rc) * H + cj] = dct * gr_;
        }
    };
    static_assert(2 * U * 16 <= kThreads, "one element of a tile's [dh_L; dh_R] per thread: row 2 u + side, node");

    bool dead = false;
    unsigned phase = 0;
    const int first_int = gr.t0 + gr.leaf_tiles;
    int t = gr.t1 - 1;
    fetch(t, in);
    cells(in);
    for (; t >= first_int; --t) {
        const Tile tl = win.at(t, true);
        const int rows = tile_rows(tl);
        const bool more = t - 1 >= gr.t0;
        const bool same = more && t - 1 >= first_int && tile_level(win.at(t - 1, true)) == tile_level(tl);
        In nx = in;
        if (more) fetch(t - 1, nx);
        if (same) cells(nx);   // a tile of the same level needs nothing of this one
        if (!local) xcd::remote_barrier(a.sync, g, phase, unsigned(a.nu));
        f32x4_t acc[MT];
#pragma unroll
        for (int i = 0; i < MT; ++i) acc[i] = f32x4_t{0.f, 0.f, 0.f, 0.f};
        uint4 f[J];
        const auto rs = make_rsrc(a.dA, a.dA_bytes);
        xcd::load_operand<float>(f, rs, [&](int j) {
            return lr < rows && kw0 + j < kw1
                       ? (uint32_t(tl.p0 + lr) * uint32_t(a.lda) + uint32_t(16 * (kw0 + j) + 4 * lq)) * 4u
                       : kOutOfRange;
        }, local, a.sync, dead);
#pragma unroll
        for (int j = 0; j < J; ++j)
#pragma unroll
            for (int i = 0; i < MT; ++i) acc[i] = xcd::mma(w[i][j], f[j], acc[i], static_cast<const float*>(nullptr));
        float* red = sm + (t & 1) * C::RED;
#pragma unroll
        for (int i = 0; i < MT; ++i) reinterpret_cast<f32x4_t*>(red)[(wave * MT + i) * 64 + lane] = acc[i];
        __syncthreads();
        {
            const int r = tid >> 4, n = tid & 15;
            if (r < 2 * U && n < rows && v0 + (r >> 1) < H) {
                const float v = sum_waves<MT>(red, r, n);
                if (!PIECES || inside(gr, a.M0, in.ch)) dhl[local_of(gr, a.M0, in.ch) * U + (r >> 1)] = v;
                else a.dhx[int64_t(in.ch) * H + v0 + (r >> 1)] = v;
            }
        }
        __syncthreads();   // the children's dh and dc
        if (more && !same) cells(nx);
        in = nx;
    }
    // the remaining tiles of leaves (the first one is done above)
    for (--t; t >= gr.t0; --t) {
        fetch(t, in);
        cells(in);
    }
}

// ----------------------------------------------------------------- TreeRNN
// h = tanh(W [h_L; h_R] + b) of the internal nodes; a leaf's h is its word
// vector, which the set-up kernel puts in its row of hx, so only the tiles of
// internal nodes run.
struct RnnFwd {
    int H, M0;
    int groups, nu, xccs;
    const Group* group;
    const Tile* tile;
    const int32_t* lchild;
    const int32_t* rchild;
    const int32_t* rootk;
    const float* W;            // [H x 2H]
    const float* b;
    float* hx;                 // [N x ldh]
    int64_t ldh;
    uint32_t hx_bytes;
    float* h_root;
    TreeSync* sync;
};
// Set-up of the forward: leaf rows of hx (and of h_root for a leaf that is a
// root), empty rows of the internal nodes, counters and error flag zero.  A
// word vector's NaN of the pattern's bits is stored as another NaN, so that no
// wait takes the leaf for one not stored yet.
static __global__ __launch_bounds__(256) void rnn_fwd_init_kernel(int N, int M0, int H, const int32_t* lword,
                                                                  const int32_t* rootk, const float* emb, float* hx,
                                                                  int64_t ldh, float* h_root, TreeSync* s) {
    const int64_t i0 = int64_t(blockIdx.x) * 256 + threadIdx.x, stride = int64_t(gridDim.x) * 256;
    zero_counters(s, i0, stride);
    if (i0 == 0) s->error = 0u;
    fill_empty(hx, ldh, M0, N - M0, H, i0, stride);
    for (int64_t i = i0; i < int64_t(M0) * ldh; i += stride) {
        const int p = int(i / ldh), j = int(i % ldh);
        const float v = j < H ? emb[int64_t(lword[p]) * H + j] : 0.f;
        hx[i] = __uint_as_float(not_empty(__float_as_uint(v)));
        if (j < H && rootk[p] >= 0) h_root[int64_t(rootk[p]) * H + j] = v;
    }
}

constexpr int kRnnU = 16;      // units of a forward workgroup: one row tile
constexpr int kRnnJ = 8;       // k-groups of a wave at most: H up to 512
constexpr int kRnnFwdLds = 2 * kWaves * 256 * 4;

static __global__ __launch_bounds__(kThreads) void treernn_fwd_xcd(RnnFwd a) {
    extern __shared__ __align__(16) float sm[];
    constexpr int U = kRnnU, J = kRnnJ;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int lr = lane & 15, lq = lane >> 4;
    const xcd::Place pl = xcd::take_place(a.sync, a.nu, a.groups, a.xccs);
    const int g = __builtin_amdgcn_readfirstlane(pl.g), m = __builtin_amdgcn_readfirstlane(pl.m);
    const bool local = __builtin_amdgcn_readfirstlane(pl.local) != 0;
    if (g < 0) return;
    const Group gr = a.group[g];
    if (gr.t0 >= gr.t1) return;   // a group without trees
    const int H = a.H, v0 = m * U, KH = (H + 15) / 16;
    const int kw0 = wave * 2 * KH / kWaves, nj = (wave + 1) * 2 * KH / kWaves - kw0;
    uint4 w[J];
#pragma unroll
    for (int j = 0; j < J; ++j) {
        const int kg = kw0 + j, side = kg >= KH, k = 16 * (kg - side * KH) + 4 * lq;
        w[j] = j < nj ? weight4(a.W + side * H, 2 * H, v0 + lr < H ? v0 + lr : -1, k, H) : make_uint4(0, 0, 0, 0);
    }
    // cells: thread (unit cu, node cn)
    const int cu = tid >> 4, cn = tid & 15, cj = v0 + cu;
    const bool cell_thread = cu < U && cj < H;
    const float bias = cell_thread ? a.b[cj] : 0.f;
    bool dead = false;
    unsigned phase = 0;
    const int t0 = gr.t0 + gr.leaf_tiles;
    if (t0 >= gr.t1) return;
    TileWindow win;
    win.init(a.tile, gr.t1, t0);
    struct Links {
        int ql, qr, rk;
    };
    auto links = [&](int t) {
        const Tile tl = win.at(t);
        Links k;
        const int q = tl.p0 + min(lr, tile_rows(tl) - 1), p = tl.p0 + min(cn, tile_rows(tl) - 1);
        k.ql = a.lchild[q];
        k.qr = a.rchild[q];
        k.rk = a.rootk[p];
        return k;
    };
    Links next = links(t0);
    for (int t = t0; t < gr.t1; ++t) {
        const Tile tl = win.at(t);
        const int rows = tile_rows(tl);
        const Links k = next;
        if (!local && t > t0) xcd::remote_barrier(a.sync, g, phase, unsigned(a.nu));
        const auto rs = make_rsrc(a.hx, a.hx_bytes);
        const uint32_t ol = uint32_t(k.ql) * uint32_t(a.ldh), orr = uint32_t(k.qr) * uint32_t(a.ldh);
        uint4 f[J];
        xcd::load_operand<float>(f, rs, [&](int j) {
            const int kg = kw0 + j;
            const uint32_t o = kg < KH ? ol + uint32_t(16 * kg) : orr + uint32_t(16 * (kg - KH));
            return lr < rows && j < nj ? (o + uint32_t(4 * lq)) * 4u : kOutOfRange;
        }, local, a.sync, dead);
        if (t + 1 < gr.t1) next = links(t + 1);
        f32x4_t acc = f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int j = 0; j < J; ++j)
            if (j < nj) acc = xcd::mma(w[j], f[j], acc, static_cast<const float*>(nullptr));
        float* red = sm + (t & 1) * kWaves * 256;
        reinterpret_cast<f32x4_t*>(red)[wave * 64 + lane] = acc;
        __syncthreads();
        if (cell_thread && cn < rows) {
            const int p = tl.p0 + cn;
            const float h = tanhf_(bias + sum_waves<1>(red, cu, cn));
            xcd::store_b32(rs, (uint32_t(p) * uint32_t(a.ldh) + uint32_t(cj)) * 4u, not_empty(__float_as_uint(h)));
            if (k.rk >= 0) a.h_root[int64_t(k.rk) * H + cj] = h;
        }
    }
}

struct RnnBwd {
    int H, M0;
    int groups, nu, xccs;
    const Group* group;
    const Tile* tile;
    const int32_t* lchild;
    const int32_t* rchild;
    const int32_t* rootk;
    const float* W;
    const float* hx;
    int64_t ldh;
    const float* dh_root;
    float* dhx;                // [N x H] dh of the roots of pieces, from the parents' launch
    float* dA;                 // [N x ldh], internal rows
    uint32_t dA_bytes;
    float* dx;                 // [M0 x H] gradient of the leaves' word vectors
    TreeSync* sync;
};
// Set-up of the backward: empty rows of dA, the gradient of a leaf that is a
// root, counters zero.
static __global__ __launch_bounds__(256) void rnn_bwd_init_kernel(int N, int M0, int H, const int32_t* rootpos,
                                                                  int trees, const float* dh_root, float* dA,
                                                                  int64_t ldh, float* dx, TreeSync* s) {
    const int64_t i0 = int64_t(blockIdx.x) * 256 + threadIdx.x, stride = int64_t(gridDim.x) * 256;
    zero_counters(s, i0, stride);
    fill_empty(dA, ldh, M0, N - M0, H, i0, stride);
    for (int64_t i = i0; i < int64_t(trees) * H; i += stride) {
        const int p = rootpos[i / H];
        if (p < M0) dx[int64_t(p) * H + i % H] = dh_root[i];
    }
}

// MT row tiles hold [dh_L; dh_R] of 8 MT units; K = H, at most 4 k-groups a wave.
template <int MT>
struct RnnBwdCfg {
    static constexpr int U = 8 * MT, J = 4;
    static constexpr int RED = kWaves * MT * 256;
    static size_t lds(int nodes) { return sizeof(float) * (2 * size_t(RED) + size_t(nodes) * U); }
};
template <int MT, bool PIECES>
__global__ __launch_bounds__(kThreads) void treernn_bwd_xcd(RnnBwd a) {
    using C = RnnBwdCfg<MT>;
    constexpr int U = C::U, J = C::J;
    extern __shared__ __align__(16) float sm[];
    float* dhl = sm + 2 * C::RED;   // [internal nodes][U]
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int lr = lane & 15, lq = lane >> 4;
    const xcd::Place pl = xcd::take_place(a.sync, a.nu, a.groups, a.xccs);
    const int g = __builtin_amdgcn_readfirstlane(pl.g), m = __builtin_amdgcn_readfirstlane(pl.m);
    const bool local = __builtin_amdgcn_readfirstlane(pl.local) != 0;
    if (g < 0) return;
    const Group gr = a.group[g];
    if (gr.t0 >= gr.t1) return;   // a group without trees
    const int first = gr.t0 + gr.leaf_tiles;
    if (first >= gr.t1) return;
    const int H = a.H, v0 = m * U, nk = (H + 15) / 16;
    const int kw0 = wave * nk / kWaves, nj = (wave + 1) * nk / kWaves - kw0;
    uint4 w[MT][J];
#pragma unroll
    for (int i = 0; i < MT; ++i)
#pragma unroll
        for (int j = 0; j < J; ++j) {
            const int r = 16 * i + lr, u = v0 + (r >> 1), k = 16 * (kw0 + j) + 4 * lq;
            float tmp[4];
#pragma unroll
            for (int e = 0; e < 4; ++e)
                tmp[e] = u < H && j < nj && k + e < H ? a.W[int64_t(k + e) * 2 * H + (r & 1) * H + u] : 0.f;
            w[i][j] = make_uint4(__float_as_uint(tmp[0]), __float_as_uint(tmp[1]), __float_as_uint(tmp[2]),
                                 __float_as_uint(tmp[3]));
        }
    const int cu = tid >> 4, cn = tid & 15, cj = v0 + cu;
    const bool cell_thread = cu < U && cj < H;
    const auto rs = make_rsrc(a.dA, a.dA_bytes);
    struct In {
        int p, rk, ch;
        float h, dhr;
    } in;
    TileWindow win;
    win.init(a.tile, gr.t1, max(gr.t1 - 64, gr.t0));
    auto fetch = [&](int t, In& x) {
        const Tile tl = win.at(t, true);
        const int q = tl.p0 + min(cn, tile_rows(tl) - 1);
        x.ch = (tid >> 4 & 1) ? a.rchild[q] : a.lchild[q];
        x.p = cell_thread && cn < tile_rows(tl) ? q : -1;
        const int j = cell_thread ? cj : 0;
        x.rk = a.rootk[q];
        x.h = a.hx[int64_t(q) * a.ldh + j];
        x.dhr = x.rk >= 0 ? a.dh_root[int64_t(x.rk) * H + j] : 0.f;
        if (PIECES && x.rk == kPieceRoot) x.dhr = a.dhx[int64_t(q) * H + j];
    };
    auto cells = [&](const In& x) {
        if (x.p < 0) return;
        const float dh = x.rk != -1 ? x.dhr : dhl[(x.p - gr.int0) * U + cu];
        xcd::store_b32(rs, (uint32_t(x.p) * uint32_t(a.ldh) + uint32_t(cj)) * 4u,
                       not_empty(__float_as_uint(dh * (1.f - x.h * x.h))));
    };
    bool dead = false;
    unsigned phase = 0;
    int t = gr.t1 - 1;
    fetch(t, in);
    cells(in);
    for (; t >= first; --t) {
        const Tile tl = win.at(t, true);
        const int rows = tile_rows(tl);
        const bool more = t - 1 >= first;
        const bool same = more && tile_level(win.at(t - 1, true)) == tile_level(tl);
        In nx = in;
        if (more) fetch(t - 1, nx);
        if (same) cells(nx);   // a tile of the same level needs nothing of this one
        if (!local) xcd::remote_barrier(a.sync, g, phase, unsigned(a.nu));
        uint4 f[J];
        xcd::load_operand<float>(f, rs, [&](int j) {
            return lr < rows && j < nj
                       ? (uint32_t(tl.p0 + lr) * uint32_t(a.ldh) + uint32_t(16 * (kw0 + j) + 4 * lq)) * 4u
                       : kOutOfRange;
        }, local, a.sync, dead);
        f32x4_t acc[MT];
#pragma unroll
        for (int i = 0; i < MT; ++i) acc[i] = f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int j = 0; j < J; ++j)
            if (j < nj) {
#pragma unroll
                for (int i = 0; i < MT; ++i) acc[i] = xcd::mma(w[i][j], f[j], acc[i], static_cast<const float*>(nullptr));
            }
        float* red = sm + (t & 1) * C::RED;
#pragma unroll
        for (int i = 0; i < MT; ++i) reinterpret_cast<f32x4_t*>(red)[(wave * MT + i) * 64 + lane] = acc[i];
        __syncthreads();
        {
            const int r = tid >> 4, n = tid & 15, u = r >> 1;
            if (r < 2 * U && n < rows && v0 + u < H) {
                const float v = sum_waves<MT>(red, r, n);
                if (in.ch < a.M0) a.dx[int64_t(in.ch) * H + v0 + u] = v;
                else if (!PIECES || inside(gr, a.M0, in.ch)) dhl[(in.ch - gr.int0) * U + u] = v;
                else a.dhx[int64_t(in.ch) * H + v0 + u] = v;
            }
        }
        __syncthreads();   // the children's dh
        if (more && !same) cells(nx);
        in = nx;
    }
}

// --------------------------------------------------------------- Child-Sum
// A node's i, o, u take U (sum of its children's h) and each child its own
// forget gate, so by linearity a node needs its children's rows G = U h.  The
// owner of a unit computes the four gate rows of G for every node of the group
// (from the exchanged h) and keeps them in LDS for the parent's cell.  Forward
// and backward are each a serial chain of one exchange per tile, like the
// binary trees'; the step of 25 trees of 5-50 nodes (E 300, H 150) went from
// 352 us, with barriers over the whole device around each level, to 173 us.
struct CsFwd {
    int E, H, M0;
    int groups, nu, xccs;
    const Group* group;
    const Tile* tile;
    const int32_t* coff;       // [N + 1] children of position p: kids[coff[p] .. coff[p + 1])
    const int32_t* kids;       // child positions
    const int32_t* rootk;
    const float* W;            // [4H x E], blocks (i, o, u, f)
    const float* U;            // [4H x H]
    const float* b;
    const float* x;            // [N x ldx] inputs
    int64_t ldx;
    uint32_t x_bytes;
    float* hx;                 // [N x ldh]
    int64_t ldh;
    uint32_t hx_bytes;
    float* Gt;                 // [N x ld3] gates i, o, u
    int64_t ld3;
    float* F;                  // [N x ldh] forget gate of each node towards its parent
    float* C;                  // [N x ldh]
    float* Gx;                 // [N x ld4] G of the roots of pieces, [unit][gate]
    int64_t ld4;
    float* h_root;
    TreeSync* sync;
};

// The children of a cell, the first two prefetched, the others eight at a time.
struct Kids {
    int n, c0, k[2];
};
template <class F>
__device__ __forceinline__ void each_kid(const Kids& q, const int32_t* kids, F f) {
#pragma unroll
    for (int e = 0; e < 2; ++e)
        if (e < q.n) f(e, q.k[e]);
    for (int e = 2; e < q.n; e += 8) {
        int k[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) k[i] = e + i < q.n ? kids[q.c0 + e + i] : 0;
#pragma unroll
        for (int i = 0; i < 8; ++i)
            if (e + i < q.n) f(e + i, k[i]);
    }
}

// NT row tiles hold the four gates of U = 4 NT units (row 4 u + gate), so a
// lane's four accumulators are the gates of one (unit, node).
template <int NT>
struct CsFwdCfg {
    static constexpr int U = 4 * NT;
    static constexpr int JE = 4, JH = NT;             // k-groups of a wave: E up to 512, H up to 128 NT
    static constexpr int RED = kWaves * NT * 256;     // floats of one set of partial tiles
    // two sets for x W, one for G; then G and c of the group's nodes
    static size_t lds(int nodes) { return sizeof(float) * (3 * size_t(RED) + size_t(nodes) * 5 * U); }
};
template <int NT, bool PIECES>
__global__ __launch_bounds__(kThreads) void childsum_fwd_xcd(CsFwd a) {
    using C = CsFwdCfg<NT>;
    constexpr int U = C::U, JE = C::JE, JH = C::JH;
    extern __shared__ __align__(16) float sm[];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int lr = lane & 15, lq = lane >> 4;
    const xcd::Place pl = xcd::take_place(a.sync, a.nu, a.groups, a.xccs);
    const int g = __builtin_amdgcn_readfirstlane(pl.g), m = __builtin_amdgcn_readfirstlane(pl.m);
    const bool local = __builtin_amdgcn_readfirstlane(pl.local) != 0;
    if (g < 0) return;
    const Group gr = a.group[g];
    if (gr.t0 >= gr.t1) return;   // a group without trees
    f32x4_t* gl = reinterpret_cast<f32x4_t*>(sm + 3 * C::RED);                              // [nodes][U] gates
    float* cl = sm + 3 * C::RED + int64_t(gr.nleaf + gr.nint) * 4 * U;                     // [nodes][U]
    const int H = a.H, E = a.E, v0 = m * U;
    const int ne = (E + 15) / 16, nh = (H + 15) / 16;
    const int ke0 = wave * ne / kWaves, nje = (wave + 1) * ne / kWaves - ke0;
    const int kh0 = wave * nh / kWaves, njh = (wave + 1) * nh / kWaves - kh0;
    uint4 we[NT][JE], wh[NT][JH];
#pragma unroll
    for (int i = 0; i < NT; ++i) {
        const int u = v0 + 4 * i + (lr >> 2), row = u < H ? (lr & 3) * H + u : -1;
#pragma unroll
        for (int j = 0; j < JE; ++j)
            we[i][j] = j < nje ? weight4(a.W, E, row, 16 * (ke0 + j) + 4 * lq, E) : make_uint4(0, 0, 0, 0);
#pragma unroll
        for (int j = 0; j < JH; ++j)
            wh[i][j] = j < njh ? weight4(a.U, H, row, 16 * (kh0 + j) + 4 * lq, H) : make_uint4(0, 0, 0, 0);
    }
    const int cu = tid >> 4, cn = tid & 15, cj = v0 + cu;
    const bool cell_thread = cu < U && cj < H;
    float bias[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) bias[q] = cell_thread ? a.b[q * H + cj] : 0.f;
    // partial tiles of a unit's four gates: tile cu / 4, lane 16 (cu % 4) + cn
    const int po = (cu >> 2) * 64 + (cu & 3) * 16 + cn;
    auto sum4 = [&](const f32x4_t* red) {
        f32x4_t s = f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int w = 0; w < kWaves; ++w) s += red[w * NT * 64 + po];
        return s;
    };
    f32x4_t* redx = reinterpret_cast<f32x4_t*>(sm);
    f32x4_t* redg = reinterpret_cast<f32x4_t*>(sm + 2 * C::RED);
    const auto rx = make_rsrc(a.x, a.x_bytes), rh = make_rsrc(a.hx, a.hx_bytes);
    TileWindow win;
    win.init(a.tile, gr.t1, gr.t0);
    bool dead = false;
    unsigned phase = 0;

    auto load_x = [&](int t, uint4 (&f)[JE]) {
        const Tile tl = win.at(t);
        xcd::load_operand<float>(f, rx, [&](int j) {
            return lr < tile_rows(tl) && j < nje
                       ? (uint32_t(tl.p0 + lr) * uint32_t(a.ldx) + uint32_t(16 * (ke0 + j) + 4 * lq)) * 4u
                       : kOutOfRange;
        }, false, a.sync, dead);
    };
    auto mma_x = [&](int t, const uint4 (&f)[JE]) {
        f32x4_t acc[NT];
#pragma unroll
        for (int i = 0; i < NT; ++i) acc[i] = f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int j = 0; j < JE; ++j)
            if (j < nje) {
#pragma unroll
                for (int i = 0; i < NT; ++i) acc[i] = xcd::mma(we[i][j], f[j], acc[i], static_cast<const float*>(nullptr));
            }
#pragma unroll
        for (int i = 0; i < NT; ++i) redx[(t & 1) * kWaves * NT * 64 + (wave * NT + i) * 64 + lane] = acc[i];
    };
    // a cell's children and root slot: the list's ends first, the first ids later
    struct Cell {
        int p, rk, c0, c1;
    };
    auto fetch = [&](int t) {
        const Tile tl = win.at(t);
        Cell c;
        const int p = tl.p0 + min(cn, tile_rows(tl) - 1);
        c.p = cell_thread && cn < tile_rows(tl) ? p : -1;
        c.rk = a.rootk[p];
        c.c0 = a.coff[p];
        c.c1 = a.coff[p + 1];
        return c;
    };
    auto fetch_kids = [&](const Cell& c) {
        Kids q;
        q.n = c.p >= 0 ? c.c1 - c.c0 : 0;
        q.c0 = c.c0;
        q.k[0] = q.n > 0 ? a.kids[c.c0] : 0;
        q.k[1] = q.n > 1 ? a.kids[c.c0 + 1] : 0;
        return q;
    };
    uint4 fx[JE];
    load_x(gr.t0, fx);
    Cell ce = fetch(gr.t0);
    mma_x(gr.t0, fx);
    Kids kd = fetch_kids(ce);
    __syncthreads();
    for (int t = gr.t0; t < gr.t1; ++t) {
        const Tile tl = win.at(t);
        const int rows = tile_rows(tl);
        const bool more = t + 1 < gr.t1;
        if (more) load_x(t + 1, fx);
        if (ce.p >= 0) {
            const int p = ce.p;
            const f32x4_t xw = sum4(redx + (t & 1) * kWaves * NT * 64);
            float ai = xw[0] + bias[0], ao = xw[1] + bias[1], au = xw[2] + bias[2], cs = 0.f;
            const float af = xw[3] + bias[3];
            each_kid(kd, a.kids, [&](int, int k) {
                f32x4_t gk;
                float ck;
                if (!PIECES || inside(gr, a.M0, k)) {
                    const int lo = local_of(gr, a.M0, k) * U + cu;
                    gk = gl[lo];
                    ck = cl[lo];
                } else {   // an earlier launch worked it
                    gk = *reinterpret_cast<const f32x4_t*>(a.Gx + int64_t(k) * a.ld4 + 4 * cj);
                    ck = a.C[int64_t(k) * a.ldh + cj];
                }
                ai += gk[0];
                ao += gk[1];
                au += gk[2];
                const float f = sigmoidf_(af + gk[3]);
                a.F[int64_t(k) * a.ldh + cj] = f;
                cs += f * ck;
            });
            const float gi = sigmoidf_(ai), go = sigmoidf_(ao), gu = tanhf_(au);
            const float c = gi * gu + cs;
            const float h = go * tanhf_(c);
            xcd::store_b32(rh, (uint32_t(p) * uint32_t(a.ldh) + uint32_t(cj)) * 4u, not_empty(__float_as_uint(h)));
            cl[local_of(gr, a.M0, p) * U + cu] = c;
            a.C[int64_t(p) * a.ldh + cj] = c;
            float* gt = a.Gt + int64_t(p) * a.ld3 + cj;
            gt[0] = gi;
            gt[H] = go;
            gt[2 * H] = gu;
            if (ce.rk >= 0) a.h_root[int64_t(ce.rk) * H + cj] = h;
        }
        // the last tile holds roots: nobody needs their G, unless they are pieces'
        if (!more && !(PIECES && gr.pieces)) break;
        const int pc = ce.p;
        const bool keep = PIECES && ce.rk == kPieceRoot;
        if (more) {
            ce = fetch(t + 1);
            mma_x(t + 1, fx);   // while h of this tile arrives
        }
        if (!local) xcd::remote_barrier(a.sync, g, phase, unsigned(a.nu));
        uint4 f[JH];
        xcd::load_operand<float>(f, rh, [&](int j) {
            return lr < rows && j < njh
                       ? (uint32_t(tl.p0 + lr) * uint32_t(a.ldh) + uint32_t(16 * (kh0 + j) + 4 * lq)) * 4u
                       : kOutOfRange;
        }, local, a.sync, dead);
        if (more) kd = fetch_kids(ce);
        f32x4_t acc[NT];
#pragma unroll
        for (int i = 0; i < NT; ++i) acc[i] = f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int j = 0; j < JH; ++j)
            if (j < njh) {
#pragma unroll
                for (int i = 0; i < NT; ++i) acc[i] = xcd::mma(wh[i][j], f[j], acc[i], static_cast<const float*>(nullptr));
            }
#pragma unroll
        for (int i = 0; i < NT; ++i) redg[(wave * NT + i) * 64 + lane] = acc[i];
        __syncthreads();
        if (pc >= 0) {
            const f32x4_t v = sum4(redg);
            gl[local_of(gr, a.M0, pc) * U + cu] = v;
            if (keep) *reinterpret_cast<f32x4_t*>(a.Gx + int64_t(pc) * a.ld4 + 4 * cj) = v;
        }
        __syncthreads();
    }
}

struct CsBwd {
    int H, M0;
    int groups, nu, xccs;
    const Group* group;
    const Tile* tile;
    const int32_t* coff;
    const int32_t* kids;
    const int32_t* rootk;
    const float* U;
    const float* Gt;
    int64_t ld3;
    const float* F;
    const float* C;
    int64_t ldh;
    const float* dh_root;
    float* dG;                 // [N x ld4] gradient of each node's G row (exchange); zero for roots
    int64_t ld4;
    uint32_t dG_bytes;
    float* dXW;                // [N x ld4]
    float* dcx;                // [N x ldh] dc of the roots of pieces, from the parents' launch
    TreeSync* sync;
};
// Set-up: empty rows of dG, zero for roots, counters zero.
static __global__ __launch_bounds__(256) void cs_bwd_init_kernel(int N, int H, const int32_t* rootk, float* dG,
                                                                 int64_t ld4, TreeSync* s) {
    const int64_t i0 = int64_t(blockIdx.x) * 256 + threadIdx.x, stride = int64_t(gridDim.x) * 256;
    zero_counters(s, i0, stride);
    const int q = int(ld4 / 4);
    uint4* d = reinterpret_cast<uint4*>(dG);
    for (int64_t i = i0; i < int64_t(N) * q; i += stride) {
        const int c = 4 * int(i % q);
        const uint32_t e = rootk[i / q] >= 0 ? 0u : kEmpty;
        d[i] = make_uint4(c < 4 * H ? e : 0u, c + 1 < 4 * H ? e : 0u, c + 2 < 4 * H ? e : 0u, c + 3 < 4 * H ? e : 0u);
    }
}

// One row tile of 16 units; K = 4H gate columns, at most J k-groups a wave.
struct CsBwdCfg {
    static constexpr int U = 16, J = 10;
    static constexpr int RED = kWaves * 256;
    static size_t lds(int nodes) { return sizeof(float) * (2 * size_t(RED) + size_t(nodes) * U); }
};
template <bool PIECES>
__global__ __launch_bounds__(kThreads) void childsum_bwd_xcd(CsBwd a) {
    using C = CsBwdCfg;
    constexpr int U = C::U, J = C::J;
    extern __shared__ __align__(16) float sm[];
    float* dcl = sm + 2 * C::RED;   // [nodes][U]
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int lr = lane & 15, lq = lane >> 4;
    const xcd::Place pl = xcd::take_place(a.sync, a.nu, a.groups, a.xccs);
    const int g = __builtin_amdgcn_readfirstlane(pl.g), m = __builtin_amdgcn_readfirstlane(pl.m);
    const bool local = __builtin_amdgcn_readfirstlane(pl.local) != 0;
    if (g < 0) return;
    const Group gr = a.group[g];
    if (gr.t0 >= gr.t1) return;   // a group without trees
    const int H = a.H, K = 4 * H, v0 = m * U, nk = (K + 15) / 16;
    const int kw0 = wave * nk / kWaves, nj = (wave + 1) * nk / kWaves - kw0;
    uint4 w[J];
#pragma unroll
    for (int j = 0; j < J; ++j) {
        const int u = v0 + lr, k = 16 * (kw0 + j) + 4 * lq;
        float tmp[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) tmp[e] = u < H && j < nj && k + e < K ? a.U[int64_t(k + e) * H + u] : 0.f;
        w[j] = make_uint4(__float_as_uint(tmp[0]), __float_as_uint(tmp[1]), __float_as_uint(tmp[2]), __float_as_uint(tmp[3]));
    }
    const int cu = tid >> 4, cn = tid & 15, cj = v0 + cu;
    const bool cell_thread = cu < U && cj < H;
    const auto rs = make_rsrc(a.dG, a.dG_bytes);
    TileWindow win;
    win.init(a.tile, gr.t1, max(gr.t1 - 64, gr.t0));
    bool dead = false;
    unsigned phase = 0;
    // a cell's inputs, a tile ahead: first what its position gives, then its
    // first children, then their values
    struct Cell {
        int p, rk, c0, c1;
        float gi, go, gu, c, dhr, dcr;
    };
    struct Kid2 {
        Kids q;
        float f[2], c[2];
    };
    auto fetch = [&](int t) {
        const Tile tl = win.at(t, true);
        Cell x;
        const int p = tl.p0 + min(cn, tile_rows(tl) - 1), j = cell_thread ? cj : 0;
        x.p = cell_thread && cn < tile_rows(tl) ? p : -1;
        x.rk = a.rootk[p];
        x.c0 = a.coff[p];
        x.c1 = a.coff[p + 1];
        const float* gt = a.Gt + int64_t(p) * a.ld3 + j;
        x.gi = gt[0];
        x.go = gt[H];
        x.gu = gt[2 * H];
        x.c = a.C[int64_t(p) * a.ldh + j];
        x.dhr = x.rk >= 0 ? a.dh_root[int64_t(x.rk) * H + j] : 0.f;
        x.dcr = PIECES && x.rk == kPieceRoot ? a.dcx[int64_t(p) * a.ldh + j] : 0.f;
        return x;
    };
    auto fetch_ids = [&](const Cell& x, Kid2& k) {
        k.q.n = x.p >= 0 ? x.c1 - x.c0 : 0;
        k.q.c0 = x.c0;
#pragma unroll
        for (int e = 0; e < 2; ++e) k.q.k[e] = e < k.q.n ? a.kids[x.c0 + e] : 0;
    };
    auto fetch_kids = [&](Kid2& k) {
#pragma unroll
        for (int e = 0; e < 2; ++e) {
            k.f[e] = e < k.q.n ? a.F[int64_t(k.q.k[e]) * a.ldh + cj] : 0.f;
            k.c[e] = e < k.q.n ? a.C[int64_t(k.q.k[e]) * a.ldh + cj] : 0.f;
        }
    };
    Cell x = fetch(gr.t1 - 1);
    Kid2 kd;
    fetch_ids(x, kd);
    fetch_kids(kd);
    for (int t = gr.t1 - 1; t >= gr.t0; --t) {
        const Tile tl = win.at(t, true);
        const int rows = tile_rows(tl);
        const bool more = t > gr.t0;
        Cell nx = x;
        if (more) nx = fetch(t - 1);
        if (!local && t < gr.t1 - 1) xcd::remote_barrier(a.sync, g, phase, unsigned(a.nu));
        uint4 f[J];
        xcd::load_operand<float>(f, rs, [&](int j) {
            return lr < rows && j < nj
                       ? (uint32_t(tl.p0 + lr) * uint32_t(a.ld4) + uint32_t(16 * (kw0 + j) + 4 * lq)) * 4u
                       : kOutOfRange;
        }, local, a.sync, dead);
        Kid2 nk2 = kd;
        if (more) fetch_ids(nx, nk2);
        f32x4_t acc = f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int j = 0; j < J; ++j)
            if (j < nj) acc = xcd::mma(w[j], f[j], acc, static_cast<const float*>(nullptr));
        float* red = sm + (t & 1) * C::RED;
        reinterpret_cast<f32x4_t*>(red)[wave * 64 + lane] = acc;
        __syncthreads();
        if (x.p >= 0) {
            const int p = x.p;
            const float dh = sum_waves<1>(red, cu, cn) + x.dhr;   // a root's dG row is 0
            const float tau = tanhf_(x.c);
            const float dc = x.rk != -1 ? x.dcr : dcl[local_of(gr, a.M0, p) * U + cu];
            const float dct = dc + dh * x.go * (1.f - tau * tau);
            const float dai = dct * x.gu * x.gi * (1.f - x.gi), dao = dh * tau * x.go * (1.f - x.go);
            const float dau = dct * x.gi * (1.f - x.gu * x.gu);
            float dafs = 0.f;
            each_kid(kd.q, a.kids, [&](int e, int k) {
                const float fk = e == 0 ? kd.f[0] : e == 1 ? kd.f[1] : a.F[int64_t(k) * a.ldh + cj];
                const float ck = e == 0 ? kd.c[0] : e == 1 ? kd.c[1] : a.C[int64_t(k) * a.ldh + cj];
                const float daf = dct * ck * fk * (1.f - fk);
                dafs += daf;
                const uint32_t o = (uint32_t(k) * uint32_t(a.ld4) + uint32_t(cj)) * 4u;
                xcd::store_b32(rs, o, not_empty(__float_as_uint(dai)));
                xcd::store_b32(rs, o + 4u * uint32_t(H), not_empty(__float_as_uint(dao)));
                xcd::store_b32(rs, o + 8u * uint32_t(H), not_empty(__float_as_uint(dau)));
                xcd::store_b32(rs, o + 12u * uint32_t(H), not_empty(__float_as_uint(daf)));
                if (!PIECES || inside(gr, a.M0, k)) dcl[local_of(gr, a.M0, k) * U + cu] = dct * fk;
                else a.dcx[int64_t(k) * a.ldh + cj] = dct * fk;
            });
            float* xw = a.dXW + int64_t(p) * a.ld4 + cj;
            xw[0] = dai;
            xw[H] = dao;
            xw[2 * H] = dau;
            xw[3 * H] = dafs;
        }
        if (more) fetch_kids(nk2);
        x = nx;
        kd = nk2;
    }
}

// ------------------------------------------------------------- host side
// Nodes a group may have: the most whose LDS (bytes(n)) a CU holds.
template <class F>
int node_capacity(size_t lds, F bytes) {
    int n = 0;
    for (int step = 1 << 16; step > 0; step >>= 1)
        if (bytes(n + step) + 1024 <= lds) n += step;
    return n;
}
// What the current device holds of groups of nu workgroups.
inline CutShape cut_shape(const tpersist::TreeDev& dev, int nu, int capacity, bool leaves = true) {
    CutShape s;
    s.leaves = leaves;
    s.nu = nu;
    s.xccs = dev.xccs > 0 && dev.xccs <= persist::kMaxXcds ? dev.xccs : 1;
    s.per_xcd = dev.cus / s.xccs;
    s.capacity = capacity;
    return s;
}

}  // namespace treex
}  // namespace janus
