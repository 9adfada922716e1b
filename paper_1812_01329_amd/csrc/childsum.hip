// Child-Sum TreeLSTM over a batch of trees of any arity, evaluated as
// level-wise frontiers.
//
// The cited TreeLSTM paper defines this variant next to the binary one: every
// node reads its word vector x, h~ is the sum of its children's h, and each
// child k has its own forget gate,
//     i, o = s(W x + U h~ + b),  u = tanh(W x + U h~ + b)   (blocks i, o, u)
//     f_k  = s(W_f x + U_f h_k + b_f)
//     c = i u + sum_k f_k c_k,   h = o tanh(c).
// Levels group nodes by height (a node after all of its children), the same
// frontiers as the binary TreeNNs (Section 6.3.1, "+PARL").
//
// By linearity U_iou h~ of a node is the sum of its children's rows
// G = h U^T (all four blocks), and child k's forget gate reads G_f of row k,
// so one contraction per level serves the level's parents.  A node's cell
// backward writes, for each child k, dG(k) = [da_iou(parent); da_f(parent, k)]
// and the child's dc, and for itself dXW = [da_iou; sum_k da_f]; a node's
// dh is its row of dG U (a root has dG = 0 and adds the head's gradient).
// Then dW = dXW^T X, dU = dG^T h, db = sum of dXW, and dX = dXW W for the
// embedding gradient.
//
// H below 320: one launch each way over groups of trees per XCD
// (tree_xcd.hpp), a few for large trees and batches.  Otherwise level by level, a cell kernel and a contraction
// per level, with XW = X W^T + b over all nodes first.
#include <algorithm>
#include <vector>

#include "device.hpp"
#include "ops.hpp"
#include "simt.hpp"
#include "tree_common.hpp"
#include "tree_tail.hpp"
#include "tree_xcd.hpp"

namespace janus {

namespace {

struct CsWs {
    int32_t* pword = nullptr;    // [N] word of the node at each position
    int32_t* pcoff = nullptr;    // [N + 1] children of position p: pkids[pcoff[p] .. pcoff[p + 1])
    int32_t* pkids = nullptr;    // [N] child positions
    int32_t* rootk = nullptr;    // [N] tree index of a root, -1 otherwise
    // level by level
    float* XW = nullptr;         // [N x 4H] X W^T + b
    float* G = nullptr;          // [N x 4H] h U^T (forward), dG (backward)
    float* Gt = nullptr;         // [N x 3H] gates i, o, u
    float* F = nullptr;          // [N x H]  forget gate of each node towards its parent
    float* C = nullptr;          // [N x H]
    float* Hn = nullptr;         // [N x H]
    float* dXW = nullptr;        // [N x 4H]
    float* dh = nullptr;         // [N x H]
    float* dc = nullptr;         // [N x H]
    float* dx = nullptr;         // [N x E]
    float* Wt = nullptr;         // [E x 4H]
    float* Ut = nullptr;         // [H x 4H]
    float* part = nullptr;
    int32_t* seg = nullptr;      // the nodes grouped by word, for the embedding gradient
    // groups of trees per XCD (tree_xcd.hpp): the groups, followed by their
    // tiles (carved after the schedule arrays, so that one copy uploads both),
    // the counters, and node rows padded to whole 128-byte lines
    treex::Group* xgroup = nullptr;  // the groups of every launch, then up to N tiles
    tpersist::TreeSync* tsync = nullptr;
    float* xl = nullptr;         // [N x ldx] inputs
    float* hx = nullptr;         // [N x ldh] h of every node
    float* dGp = nullptr;        // [N x ld4]
    float* dXWp = nullptr;       // [N x ld4]
    float* Gtp = nullptr;        // [N x ld3]
    float* Fp = nullptr;         // [N x ldh]
    float* Cp = nullptr;         // [N x ldh]
    float* dcx = nullptr;        // [N x ldh] dc of the roots of pieces of trees
    float* dxp = nullptr;        // [3][N x E] parts of the inputs' gradient
    float* tpart = nullptr;      // parts of dW and dU
    float* tsum = nullptr;       // parts of db
    int64_t ld4 = 0, ld3 = 0, ldh = 0, ldx = 0;
};

size_t carve_cs(const janus_treelstm_desc& d, int32_t N, void* base, CsWs& w) {
    Carver c(base);
    const int H = d.H, E = d.E;
    w.pword = c.take<int32_t>(N);
    w.pcoff = c.take<int32_t>(int64_t(N) + 1);
    w.pkids = c.take<int32_t>(N);
    w.rootk = c.take<int32_t>(N);
    w.xgroup = reinterpret_cast<treex::Group*>(c.take<char>(treex::kGroupBytes + size_t(N) * sizeof(treex::Tile)));
    w.tsync = c.take<tpersist::TreeSync>(1);
    w.seg = c.take<int32_t>(int64_t(embed_seg_ints(N)));   // the nodes grouped by word
    const size_t mark = c.off;
    // a call takes one of the two paths: their arrays share the space
    w.XW = c.take<float>(int64_t(N) * 4 * H);
    w.G = c.take<float>(int64_t(N) * 4 * H);
    w.Gt = c.take<float>(int64_t(N) * 3 * H);
    w.F = c.take<float>(int64_t(N) * H);
    w.C = c.take<float>(int64_t(N) * H);
    w.Hn = c.take<float>(int64_t(N) * H);
    w.dXW = c.take<float>(int64_t(N) * 4 * H);
    w.dh = c.take<float>(int64_t(N) * H);
    w.dc = c.take<float>(int64_t(N) * H);
    w.dx = c.take<float>(int64_t(N) * E);
    w.Wt = c.take<float>(int64_t(E) * 4 * H);
    w.Ut = c.take<float>(int64_t(H) * 4 * H);
    w.part = c.take<float>(colsum_partial_floats(4 * H));
    const size_t levels_end = c.off;
    c.off = mark;
    w.ld4 = round_up(int64_t(4) * H, 32);
    w.ld3 = round_up(int64_t(3) * H, 32);
    w.ldh = round_up(H, 32);
    w.ldx = round_up(E, 32);
    w.xl = c.take<float>(int64_t(N) * w.ldx);
    w.hx = c.take<float>(int64_t(N) * w.ldh);
    w.dGp = c.take<float>(int64_t(N) * w.ld4);
    w.dXWp = c.take<float>(int64_t(N) * w.ld4);
    w.Gtp = c.take<float>(int64_t(N) * w.ld3);
    w.Fp = c.take<float>(int64_t(N) * w.ldh);
    w.Cp = c.take<float>(int64_t(N) * w.ldh);
    w.dcx = c.take<float>(int64_t(N) * w.ldh);
    w.dxp = c.take<float>(int64_t(3) * N * E);
    w.tpart = c.take<float>(tail_part_floats(4 * H, E) + tail_part_floats(4 * H, H));
    w.tsum = c.take<float>(tail_sum_floats(N, 4 * H));
    c.off = std::max(c.off, levels_end);
    return c.off + 256;
}

__global__ void cs_fwd_cell_kernel(int p0, int rows, int H, const float* XW, const float* G, const int32_t* pcoff,
                                   const int32_t* pkids, const int32_t* rootk, float* Gt, float* F, float* C,
                                   float* Hn, float* h_root) {
    const int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
    if (i >= int64_t(rows) * H) return;
    const int p = p0 + int(i / H), j = int(i % H);
    const float* xw = XW + int64_t(p) * 4 * H;
    float ai = xw[j], ao = xw[H + j], au = xw[2 * H + j];
    const float af = xw[3 * H + j];
    float csum = 0.f;
    for (int e = pcoff[p]; e < pcoff[p + 1]; ++e) {
        const int k = pkids[e];
        const float* g = G + int64_t(k) * 4 * H;
        ai += g[j];
        ao += g[H + j];
        au += g[2 * H + j];
        const float f = sigmoidf_(af + g[3 * H + j]);
        F[int64_t(k) * H + j] = f;
        csum += f * C[int64_t(k) * H + j];
    }
    const float gi = sigmoidf_(ai), go = sigmoidf_(ao), gu = tanhf_(au);
    const float c = gi * gu + csum;
    const float h = go * tanhf_(c);
    C[int64_t(p) * H + j] = c;
    Hn[int64_t(p) * H + j] = h;
    float* gt = Gt + int64_t(p) * 3 * H;
    gt[j] = gi;
    gt[H + j] = go;
    gt[2 * H + j] = gu;
    if (rootk[p] >= 0) h_root[int64_t(rootk[p]) * H + j] = h;
}

__global__ void cs_bwd_cell_kernel(int p0, int rows, int H, const float* dh, const float* dh_root,
                                   const int32_t* rootk, const float* Gt, const float* F, const float* C,
                                   const int32_t* pcoff, const int32_t* pkids, float* dc, float* dG, float* dXW) {
    const int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
    if (i >= int64_t(rows) * H) return;
    const int p = p0 + int(i / H), j = int(i % H);
    const int rk = rootk[p];
    const float dhv = dh[int64_t(p) * H + j] + (rk >= 0 ? dh_root[int64_t(rk) * H + j] : 0.f);
    const float* gt = Gt + int64_t(p) * 3 * H;
    const float gi = gt[j], go = gt[H + j], gu = gt[2 * H + j];
    const float tau = tanhf_(C[int64_t(p) * H + j]);
    const float dct = dc[int64_t(p) * H + j] + dhv * go * (1.f - tau * tau);
    const float dai = dct * gu * gi * (1.f - gi);
    const float dao = dhv * tau * go * (1.f - go);
    const float dau = dct * gi * (1.f - gu * gu);
    float dafs = 0.f;
    for (int e = pcoff[p]; e < pcoff[p + 1]; ++e) {
        const int k = pkids[e];
        const float f = F[int64_t(k) * H + j];
        const float daf = dct * C[int64_t(k) * H + j] * f * (1.f - f);
        dafs += daf;
        float* g = dG + int64_t(k) * 4 * H;
        g[j] = dai;
        g[H + j] = dao;
        g[2 * H + j] = dau;
        g[3 * H + j] = daf;
        dc[int64_t(k) * H + j] = dct * f;
    }
    float* x = dXW + int64_t(p) * 4 * H;
    x[j] = dai;
    x[H + j] = dao;
    x[2 * H + j] = dau;
    x[3 * H + j] = dafs;
}

janus_status check_cs(const janus_treelstm_desc* d) {
    if (!d || d->E <= 0 || d->H <= 0 || d->V <= 0) return JANUS_ERR_INVALID_ARG;
    if (d->dtype != JANUS_F32) return JANUS_ERR_UNSUPPORTED;
    return JANUS_OK;
}

// Validates the call and carves the workspace.
janus_status prepare_cs(const janus_treelstm_desc* d, const janus_nary_tree_batch* t, void* ws, size_t ws_bytes,
                        NarySchedule& s, CsWs& w) {
    janus_status e = check_cs(d);
    if (e != JANUS_OK) return e;
    if ((e = build_nary_schedule(t, d->V, s)) != JANUS_OK) return e;
    if (!ws || ws_bytes < carve_cs(*d, s.N, nullptr, w) || reinterpret_cast<uintptr_t>(ws) % 256 != 0)
        return JANUS_ERR_WORKSPACE;
    carve_cs(*d, s.N, ws, w);
    return JANUS_OK;
}

// Copies the schedule arrays (carved one after another: one copy) for the
// level-by-level kernels.
janus_status upload_cs(const NarySchedule& s, const CsWs& w, hipStream_t st) {
    const size_t nb = sizeof(int32_t) * s.N;
    // the error flag is zeroed too, so the device report of a call on this
    // path reads no stale one
    const std::vector<char> zero_sync(tpersist::kTreeSyncCounters, 0);
    const UploadPiece pieces[] = {{w.pword, s.pword.data(), nb},
                                  {w.pcoff, s.pcoff.data(), nb + sizeof(int32_t)},
                                  {w.pkids, s.pkids.data(), sizeof(int32_t) * s.pkids.size()},
                                  {w.rootk, s.rootk.data(), nb},
                                  {w.tsync, zero_sync.data(), zero_sync.size()}};
    return upload_pieces(pieces, 5, st);
}

// ------------------------------------------------- groups of trees per XCD
// Four gates of 4 NT units per forward workgroup, 16 units of dh per backward
// workgroup.  H below 320 (the forward's G rows of a group's nodes then still
// leave room in the LDS for a few hundred nodes per group; larger trees run in
// pieces), E up to 512; off with JANUS_TREE_PERSIST=0.  Other sizes run level by level.
struct CsPlan {
    bool on = false;
    int NT = 0, fwd_nu = 0, bwd_nu = 0;
    treex::Cut cut;
    size_t fwd_lds = 0, bwd_lds = 0;
    // the schedule in the cut's order (in cut.more)
    int32_t *word = nullptr, *coff = nullptr, *kids = nullptr, *rootk = nullptr;
    size_t nkids = 0;
};
size_t cs_fwd_lds(int NT, int nodes) {
    return NT == 1 ? treex::CsFwdCfg<1>::lds(nodes) : NT == 2 ? treex::CsFwdCfg<2>::lds(nodes) : treex::CsFwdCfg<3>::lds(nodes);
}
CsPlan cs_plan(const janus_treelstm_desc& d, const janus_nary_tree_batch* t, const NarySchedule& s) {
    CsPlan p;
    const char* env = getenv("JANUS_TREE_PERSIST");
    if (env && env[0] == '0') return p;
    const tpersist::TreeDev dev = tpersist::tree_dev();
    if (dev.cus <= 0 || dev.lds == 0 || d.H >= 320 || d.E > tpersist::kMaxE) return p;
    const int32_t N = s.N;
    if (int64_t(N) * round_up(4 * d.H, 32) * 4 >= (int64_t(1) << 31) || int64_t(N) * round_up(d.E, 32) * 4 >= (int64_t(1) << 31))
        return p;   // 32-bit byte offsets
    p.NT = d.H <= 128 ? 1 : d.H <= 256 ? 2 : 3;
    p.fwd_nu = (d.H + 4 * p.NT - 1) / (4 * p.NT);
    p.bwd_nu = (d.H + treex::CsBwdCfg::U - 1) / treex::CsBwdCfg::U;
    const int capacity = treex::node_capacity(
        dev.lds, [&](int n) { return std::max(cs_fwd_lds(p.NT, n), treex::CsBwdCfg::lds(n)); });
    p.cut.take(N, size_t(4) * N + 1);
    std::fill(p.cut.parent, p.cut.parent + N, -1);
    for (int32_t q = 0; q < N; ++q)
        for (int32_t e = s.pcoff[q]; e < s.pcoff[q + 1]; ++e) p.cut.parent[s.pkids[e]] = q;
    p.cut.root.resize(t->num_trees);
    for (int32_t q = 0; q < N; ++q)
        if (s.rootk[q] >= 0) p.cut.root[s.rootk[q]] = q;
    if (!treex::cut_batch(N, s.level_offsets, int(s.level_offsets.size()) - 1,
                          treex::cut_shape(dev, std::max(p.fwd_nu, p.bwd_nu), capacity), p.cut))
        return p;
    p.fwd_lds = cs_fwd_lds(p.NT, p.cut.most_nodes);
    p.bwd_lds = treex::CsBwdCfg::lds(p.cut.most_nodes);
    p.word = p.cut.more;
    p.rootk = p.word + N;
    p.kids = p.rootk + N;
    p.coff = p.kids + N;
    p.coff[0] = 0;
    for (int32_t q = 0; q < N; ++q) {
        const int32_t o = p.cut.order[q];
        p.word[q] = s.pword[o];
        p.rootk[q] = p.cut.split && p.cut.piece[o] ? treex::kPieceRoot : s.rootk[o];
        for (int32_t e = s.pcoff[o]; e < s.pcoff[o + 1]; ++e) p.kids[p.nkids++] = p.cut.pos[s.pkids[e]];
        p.coff[q + 1] = int32_t(p.nkids);
    }
    p.on = true;
    return p;
}
treex::Tile* cs_tiles(const CsWs& w, const treex::Cut& c) {
    return reinterpret_cast<treex::Tile*>(w.xgroup + c.group.size());
}
unsigned cs_fill_blocks(int64_t n) { return unsigned(std::min<int64_t>((n + 1023) / 1024, 1024)); }
int cs_xccs(const treex::Cut& c) {
    const char* e = getenv("JANUS_XCD_REMOTE");
    return e && e[0] == '1' ? 0 : c.xccs;
}

template <int NT, bool PIECES>
janus_status launch_cs_fwd(int blocks, size_t lds, const treex::CsFwd& a, hipStream_t st) {
    static size_t attr = 0;
    return tpersist::tree_persistent_launch(treex::childsum_fwd_xcd<NT, PIECES>, blocks, lds, a, st, attr,
                                            treex::kThreads);
}
template <int NT>
janus_status launch_cs_fwd(const CsPlan& p, int blocks, const treex::CsFwd& a, hipStream_t st) {
    return p.cut.split ? launch_cs_fwd<NT, true>(blocks, p.fwd_lds, a, st)
                       : launch_cs_fwd<NT, false>(blocks, p.fwd_lds, a, st);
}
template <bool PIECES>
janus_status launch_cs_bwd(int blocks, size_t lds, const treex::CsBwd& a, hipStream_t st) {
    static size_t attr = 0;
    return tpersist::tree_persistent_launch(treex::childsum_bwd_xcd<PIECES>, blocks, lds, a, st, attr, treex::kThreads);
}

janus_status cs_fwd_xcd_call(const janus_treelstm_desc& d, const NarySchedule& s, const CsWs& w, const CsPlan& p,
                             const void* emb, const void* W, const void* U, const void* b, void* h_root,
                             hipStream_t st) {
    const int32_t N = s.N;
    const size_t nb = sizeof(int32_t) * N;
    const UploadPiece pieces[] = {{w.pword, p.word, nb},
                                  {w.pcoff, p.coff, nb + sizeof(int32_t)},
                                  {w.pkids, p.kids, sizeof(int32_t) * p.nkids},
                                  {w.rootk, p.rootk, nb},
                                  {w.xgroup, p.cut.group.data(), sizeof(treex::Group) * p.cut.group.size()},
                                  {cs_tiles(w, p.cut), p.cut.tile.data(), sizeof(treex::Tile) * p.cut.tile.size()}};
    janus_status e = upload_pieces(pieces, 6, st);
    if (e != JANUS_OK) return e;
    treex::CsFwd a = {};
    a.E = d.E;
    a.H = d.H;
    a.M0 = s.level_offsets[1];
    a.nu = p.fwd_nu;
    a.xccs = cs_xccs(p.cut);
    a.tile = cs_tiles(w, p.cut);
    a.coff = w.pcoff;
    a.kids = w.pkids;
    a.rootk = w.rootk;
    a.W = static_cast<const float*>(W);
    a.U = static_cast<const float*>(U);
    a.b = static_cast<const float*>(b);
    a.x = w.xl;
    a.ldx = w.ldx;
    a.x_bytes = uint32_t(int64_t(N) * w.ldx * 4);
    a.hx = w.hx;
    a.ldh = w.ldh;
    a.hx_bytes = uint32_t(int64_t(N) * w.ldh * 4);
    a.Gt = w.Gtp;
    a.ld3 = w.ld3;
    a.F = w.Fp;
    a.C = w.Cp;
    a.Gx = w.dGp;   // free until the backward
    a.ld4 = w.ld4;
    a.h_root = static_cast<float*>(h_root);
    a.sync = w.tsync;
    const int parts = int(p.cut.launch.size());
    for (int part = 0; part < parts; ++part) {
        if (part == 0) {
            TraceScope trace("tree_fwd_init", 0.0, 4.0 * double(N) * (w.ldh + 2.0 * w.ldx), st);
            hipLaunchKernelGGL(treex::fwd_init_kernel, dim3(cs_fill_blocks(int64_t(N) * (w.ldh + w.ldx))), dim3(256), 0,
                               st, N, N, d.E, w.pword, static_cast<const float*>(emb), w.xl, w.ldx, w.hx, w.ldh, d.H,
                               w.tsync);
        } else {   // the counters of the next launch
            hipLaunchKernelGGL(treex::fill_kernel, dim3(4), dim3(256), 0, st, w.hx, w.ldh, int64_t(0), int64_t(0), d.H,
                               w.tsync);
        }
        JANUS_LAUNCH_CHECK();
        const treex::CutLaunch& l = p.cut.launch[part];
        a.group = w.xgroup + l.first;
        a.groups = l.groups;
        const int blocks = p.cut.blocks(l, p.fwd_nu);
        TraceScope trace("childsum_fwd_persistent", 2.0 * N * 4.0 * d.H * (double(d.E) + double(d.H)) / parts, 0.0, st);
        e = p.NT == 1   ? launch_cs_fwd<1>(p, blocks, a, st)
            : p.NT == 2 ? launch_cs_fwd<2>(p, blocks, a, st)
                        : launch_cs_fwd<3>(p, blocks, a, st);
        if (e != JANUS_OK) return e;
    }
    return JANUS_OK;
}

// The schedule is the forward's (the workspace is unchanged between the calls).
janus_status cs_bwd_xcd_call(const janus_treelstm_desc& d, const NarySchedule& s, const CsWs& w, const CsPlan& p,
                             const void* W, const void* U, const void* dh_root, float* demb, float* dW, float* dU,
                             float* db, hipStream_t st) {
    const int32_t N = s.N;
    const int H = d.H, E = d.E;
    std::vector<int32_t> seg;
    const int nseg = embed_segments(p.word, N, d.V, seg);
    janus_status e = upload(w.seg, seg.data(), seg.size() * sizeof(int32_t), st);
    if (e != JANUS_OK) return e;
    treex::CsBwd a = {};
    a.H = H;
    a.M0 = s.level_offsets[1];
    a.nu = p.bwd_nu;
    a.xccs = cs_xccs(p.cut);
    a.tile = cs_tiles(w, p.cut);
    a.coff = w.pcoff;
    a.kids = w.pkids;
    a.rootk = w.rootk;
    a.U = static_cast<const float*>(U);
    a.Gt = w.Gtp;
    a.ld3 = w.ld3;
    a.F = w.Fp;
    a.C = w.Cp;
    a.ldh = w.ldh;
    a.dh_root = static_cast<const float*>(dh_root);
    a.dG = w.dGp;
    a.ld4 = w.ld4;
    a.dG_bytes = uint32_t(int64_t(N) * w.ld4 * 4);
    a.dXW = w.dXWp;
    a.dcx = w.dcx;
    a.sync = w.tsync;
    const int parts = int(p.cut.launch.size());
    for (int part = parts; part-- > 0;) {   // parents before the pieces below them
        if (part == parts - 1) {
            TraceScope trace("tree_bwd_init", 0.0, 4.0 * double(N) * w.ld4, st);
            hipLaunchKernelGGL(treex::cs_bwd_init_kernel, dim3(cs_fill_blocks(int64_t(N) * w.ld4)), dim3(256), 0, st, N, H,
                               w.rootk, w.dGp, w.ld4, w.tsync);
        } else {
            hipLaunchKernelGGL(treex::fill_kernel, dim3(4), dim3(256), 0, st, w.hx, w.ldh, int64_t(0), int64_t(0), H,
                               w.tsync);
        }
        JANUS_LAUNCH_CHECK();
        const treex::CutLaunch& l = p.cut.launch[part];
        a.group = w.xgroup + l.first;
        a.groups = l.groups;
        const int blocks = p.cut.blocks(l, p.bwd_nu);
        TraceScope trace("childsum_bwd_persistent", 2.0 * N * 4.0 * H * double(H) / parts, 0.0, st);
        e = p.cut.split ? launch_cs_bwd<true>(blocks, p.bwd_lds, a, st) : launch_cs_bwd<false>(blocks, p.bwd_lds, a, st);
        if (e != JANUS_OK) return e;
    }
    TailArgs q;
    GemmDesc g;
    g.dtype = JANUS_F32;
    // dW = dXW^T X, dU = dG^T h (roots' rows of dG are 0)
    g.M = 4 * H;
    g.N = E;
    g.K = N;
    g.a_t = g.b_t = true;
    g.A = w.dXWp;
    g.lda = w.ld4;
    g.B = w.xl;
    g.ldb = w.ldx;
    g.C = dW;
    g.ldc = E;
    tail_add(q, g, w.tpart);
    g.N = H;
    g.A = w.dGp;
    g.B = w.hx;
    g.ldb = w.ldh;
    g.C = dU;
    g.ldc = H;
    tail_add(q, g, w.tpart + tail_part_floats(4 * H, E));
    // dX = dXW W, in up to three parts that the embedding rows add up
    g.M = N;
    g.N = E;
    g.K = 4 * H;
    g.a_t = false;
    g.A = w.dXWp;
    g.B = W;
    g.ldb = E;
    g.C = nullptr;
    tail_add(q, g, w.dxp, 3);
    TailProblem& dx = q.p[q.n - 1];
    if (dx.splits == 1) {
        dx.g.C = w.dxp;
        dx.g.ldc = E;
    }
    q.dx = w.dxp;
    q.ldx = E;
    q.dx_parts = dx.splits;
    q.dx_stride = int64_t(N) * E;
    q.src = w.dXWp;
    q.ld = w.ld4;
    q.rows = N;
    q.cols = 4 * H;
    q.sum_part = w.tsum;
    q.sum_out = db;
    q.demb = demb;
    q.demb_n = int64_t(d.V) * E;
    q.E = E;
    q.leaves = N;
    q.nseg = nseg;
    q.seg = w.seg;
    return tail_run(q, "childsum_bwd_tail", st);
}

}  // namespace

}  // namespace janus

using namespace janus;

extern "C" size_t janus_childsum_workspace_bytes(const janus_childsum_desc* d, int32_t max_nodes) {
    if (check_cs(d) != JANUS_OK || max_nodes <= 0) return 0;
    CsWs w;
    return carve_cs(*d, max_nodes, nullptr, w);
}

extern "C" janus_status janus_childsum_fwd(const janus_childsum_desc* d, const janus_nary_tree_batch* t,
                                           const void* emb, const void* W, const void* U, const void* b, void* h_root,
                                           void* ws, size_t ws_bytes, void* stream) {
    if (!emb || !W || !U || !b || !h_root) return JANUS_ERR_INVALID_ARG;
    hipStream_t st = static_cast<hipStream_t>(stream);
    NarySchedule s;
    CsWs w;
    janus_status e = prepare_cs(d, t, ws, ws_bytes, s, w);
    if (e != JANUS_OK) return e;
    const CsPlan plan = cs_plan(*d, t, s);
    if (plan.on) return cs_fwd_xcd_call(*d, s, w, plan, emb, W, U, b, h_root, st);
    if ((e = upload_cs(s, w, st)) != JANUS_OK) return e;
    const int H = d->H, E = d->E, N = s.N;
    const int L = int(s.level_offsets.size()) - 1;
    if ((e = transpose_f32(static_cast<const float*>(W), 4 * H, E, w.Wt, st)) != JANUS_OK) return e;
    if ((e = transpose_f32(static_cast<const float*>(U), 4 * H, H, w.Ut, st)) != JANUS_OK) return e;
    // the input part of every node's gates at once
    e = simt_gemm<false, kSimtStore>("childsum_x_gemm", N, 4 * H, E, static_cast<const float*>(emb), E, w.pword, w.Wt,
                                     4 * H, nullptr, static_cast<const float*>(b), w.XW, 4 * H, st);
    if (e != JANUS_OK) return e;
    for (int k = 0; k < L; ++k) {
        const int p0 = s.level_offsets[k], rows = s.level_offsets[k + 1] - p0;
        const int64_t n = int64_t(rows) * H;
        {
            TraceScope trace("childsum_fwd_cell", 0.0, 4.0 * n * 16.0, st);
            hipLaunchKernelGGL(cs_fwd_cell_kernel, dim3(unsigned((n + 255) / 256)), dim3(256), 0, st, p0, rows, H,
                               w.XW, w.G, w.pcoff, w.pkids, w.rootk, w.Gt, w.F, w.C, w.Hn,
                               static_cast<float*>(h_root));
            JANUS_LAUNCH_CHECK();
        }
        if (k + 1 < L) {   // the top level has no parents
            e = simt_gemm<false, kSimtStore>("childsum_level_gemm", rows, 4 * H, H, w.Hn + int64_t(p0) * H, H, nullptr,
                                             w.Ut, 4 * H, nullptr, nullptr, w.G + int64_t(p0) * 4 * H, 4 * H, st);
            if (e != JANUS_OK) return e;
        }
    }
    return JANUS_OK;
}

extern "C" janus_status janus_childsum_bwd(const janus_childsum_desc* d, const janus_nary_tree_batch* t,
                                           const void* emb, const void* W, const void* U, void* ws, size_t ws_bytes,
                                           const void* dh_root, float* demb, float* dW, float* dU, float* db,
                                           void* stream) {
    if (!emb || !W || !U || !dh_root || !demb || !dW || !dU || !db) return JANUS_ERR_INVALID_ARG;
    hipStream_t st = static_cast<hipStream_t>(stream);
    NarySchedule s;
    CsWs w;
    janus_status e = prepare_cs(d, t, ws, ws_bytes, s, w);
    if (e != JANUS_OK) return e;
    const CsPlan plan = cs_plan(*d, t, s);
    if (plan.on) return cs_bwd_xcd_call(*d, s, w, plan, W, U, dh_root, demb, dW, dU, db, st);
    if ((e = upload_cs(s, w, st)) != JANUS_OK) return e;
    const int H = d->H, E = d->E, N = s.N;
    const int L = int(s.level_offsets.size()) - 1;
    // roots have no parent: their dG rows and dc stay 0
    if ((e = zero_fill(w.G, sizeof(float) * size_t(N) * 4 * H, st)) != JANUS_OK) return e;
    if ((e = zero_fill(w.dc, sizeof(float) * size_t(N) * H, st)) != JANUS_OK) return e;
    for (int k = L - 1; k >= 0; --k) {
        const int p0 = s.level_offsets[k], rows = s.level_offsets[k + 1] - p0;
        // dh of the level from the dG rows its parents wrote
        e = simt_gemm<false, kSimtStore>("childsum_dh_gemm", rows, H, 4 * H, w.G + int64_t(p0) * 4 * H, 4 * H, nullptr,
                                         static_cast<const float*>(U), H, nullptr, nullptr, w.dh + int64_t(p0) * H, H,
                                         st);
        if (e != JANUS_OK) return e;
        const int64_t n = int64_t(rows) * H;
        TraceScope trace("childsum_bwd_cell", 0.0, 4.0 * n * 20.0, st);
        hipLaunchKernelGGL(cs_bwd_cell_kernel, dim3(unsigned((n + 255) / 256)), dim3(256), 0, st, p0, rows, H, w.dh,
                           static_cast<const float*>(dh_root), w.rootk, w.Gt, w.F, w.C, w.pcoff, w.pkids, w.dc, w.G,
                           w.dXW);
        JANUS_LAUNCH_CHECK();
    }
    // dW = dXW^T X (rows of emb gathered by word), dU = dG^T H, db = sum dXW
    e = simt_gemm<true, kSimtStore>("childsum_dW_gemm", 4 * H, E, N, w.dXW, 4 * H, nullptr,
                                    static_cast<const float*>(emb), E, w.pword, nullptr, dW, E, st);
    if (e != JANUS_OK) return e;
    e = simt_gemm<true, kSimtStore>("childsum_dU_gemm", 4 * H, H, N, w.G, 4 * H, nullptr, w.Hn, H, nullptr, nullptr,
                                    dU, H, st);
    if (e != JANUS_OK) return e;
    if ((e = colsum(JANUS_F32, w.dXW, N, 4 * H, 4 * H, db, w.part, st)) != JANUS_OK) return e;
    // dX = dXW W, then the embedding gradient
    e = simt_gemm<false, kSimtStore>("childsum_dx_gemm", N, E, 4 * H, w.dXW, 4 * H, nullptr,
                                     static_cast<const float*>(W), E, nullptr, nullptr, w.dx, E, st);
    if (e != JANUS_OK) return e;
    return embed_backward(JANUS_F32, w.dx, s.pword.data(), N, E, demb, d->V, w.seg, st);
}

extern "C" janus_status janus_childsum_device_report(const janus_childsum_desc* d, const janus_nary_tree_batch* t,
                                                     const void* ws, size_t ws_bytes, int32_t* timed_out,
                                                     void* stream) {
    if (!timed_out) return JANUS_ERR_INVALID_ARG;
    hipStream_t st = static_cast<hipStream_t>(stream);
    NarySchedule s;
    CsWs w;
    janus_status e = prepare_cs(d, t, const_cast<void*>(ws), ws_bytes, s, w);
    if (e != JANUS_OK) return e;
    unsigned flag = 0;
    JANUS_HIP(hipStreamSynchronize(st));
    JANUS_HIP(hipMemcpy(&flag, &w.tsync->error, sizeof(flag), hipMemcpyDeviceToHost));
    *timed_out = flag != 0u ? 1 : 0;
    return flag != 0u ? JANUS_ERR_DEVICE : JANUS_OK;
}
