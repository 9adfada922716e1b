// What follows the levels of a tree step's backward: the contractions over
// nodes (weight gradients, gradients of the leaf inputs), the bias gradient
// and the embedding gradient, in two launches.
//
// Each contraction alone has too few 64 x 64 tiles for the chip (60 for the
// weights at H 150) and walks hundreds of nodes, so the first launch takes
// all of them together, each with its K split so that the whole is about a
// thousand equal pieces; a piece writes its part (fixed order, summed by the
// second launch).  The launch also sums columns for the bias and zeroes the
// embedding gradient, which are memory traffic beside its MFMA work.  The
// second launch adds the parts, and one workgroup per word of the batch adds
// the gradients of that word's leaves.
//
// Binary TreeLSTM, 25 trees, E 300, H 150: 21 + 9 us against 77 as phases of
// one resident launch; 100 trees, H 300: 135 + 24 against 384.
#pragma once

#include <algorithm>

#include "gemm_f32.hpp"
#include "runtime.hpp"

namespace janus {
namespace {

constexpr int kTailProblems = 3;
constexpr int kTailPieces = 1024;       // pieces of all contractions together, about
constexpr int kTailSplits = 8;          // K parts of one contraction at most
constexpr int kTailRows = 256;          // rows of a column-sum piece
constexpr int kTailZero = 1 << 14;      // 16-byte words of a zeroing piece

struct TailProblem {
    GemmDesc g;              // float32; C / ldc: the result (rows of ldc)
    int tiles_m = 0, tiles_n = 0, splits = 1, per = 0;
    int first = 0;           // its first piece
    float* part = nullptr;   // [splits][M][N] where splits > 1
};
struct TailArgs {
    TailProblem p[kTailProblems];
    int n = 0;
    // column sums of src [rows x ld] over `cols` columns: parts [chunks][cols]
    const float* src = nullptr;
    int64_t ld = 0;
    int rows = 0, cols = 0, chunks = 0, sum_first = 0;
    float* sum_part = nullptr;
    float* sum_out = nullptr;
    // embedding gradient: zeroed whole, then the rows of the words in the batch
    float* demb = nullptr;
    int64_t demb_n = 0;      // floats
    int zero_first = 0;
    // second launch
    const float* dx = nullptr;   // gradient of leaf r: row r (pitch ldx), dx_parts of them dx_stride apart
    int64_t ldx = 0, dx_stride = 0;
    int dx_parts = 1, E = 0, leaves = 0, nseg = 0;
    const int32_t* seg = nullptr;
    int64_t reduce_n = 0;    // elements the second launch adds up
};

__global__ __launch_bounds__(F32Cfg::NT) void tree_tail_kernel(TailArgs a) {
    __shared__ __align__(16) float smem[F32Cfg::SMEM / 4];
    const int it = int(blockIdx.x), tid = threadIdx.x;
    if (it >= a.zero_first) {
        const int64_t n4 = a.demb_n / 4, z0 = int64_t(it - a.zero_first) * kTailZero;
        const bool vec = (reinterpret_cast<uintptr_t>(a.demb) & 15) == 0;
        if (vec) {
            float4* d = reinterpret_cast<float4*>(a.demb);
            for (int64_t i = z0 + tid; i < min(z0 + kTailZero, n4); i += F32Cfg::NT) d[i] = make_float4(0.f, 0.f, 0.f, 0.f);
            if (it == a.zero_first && 4 * n4 + tid < a.demb_n) a.demb[4 * n4 + tid] = 0.f;
        } else {
            for (int64_t i = 4 * z0 + tid; i < min(4 * (z0 + kTailZero), a.demb_n); i += F32Cfg::NT) a.demb[i] = 0.f;
        }
        return;
    }
    if (it >= a.sum_first) {
        // 64 columns of kTailRows rows: wave w takes every 4th row, eight loads in flight
        const int ncol = (a.cols + 63) / 64, i = it - a.sum_first, chunk = i / ncol;
        const int lane = tid & 63, wave = tid >> 6, c = 64 * (i % ncol) + lane;
        const int r1 = min(a.rows, (chunk + 1) * kTailRows);
        float s = 0.f;
        if (c < a.cols) {
            int r = chunk * kTailRows + wave;
            for (; r + 28 < r1; r += 32) {
                float v[8];
#pragma unroll
                for (int e = 0; e < 8; ++e) v[e] = a.src[int64_t(r + 4 * e) * a.ld + c];
#pragma unroll
                for (int e = 0; e < 8; ++e) s += v[e];
            }
            for (; r < r1; r += 4) s += a.src[int64_t(r) * a.ld + c];
        }
        smem[wave * 64 + lane] = s;
        __syncthreads();
        if (wave == 0 && c < a.cols)
            a.sum_part[int64_t(chunk) * a.cols + c] = (smem[lane] + smem[64 + lane]) + (smem[128 + lane] + smem[192 + lane]);
        return;
    }
    int q = 0;
#pragma unroll
    for (int i = 1; i < kTailProblems; ++i)
        if (i < a.n && it >= a.p[i].first) q = i;
    const TailProblem& p = a.p[q];
    const int r = it - p.first, tiles = p.tiles_m * p.tiles_n, split = r / tiles, t = r % tiles;
    const int m0 = (t / p.tiles_n) * F32Cfg::BM, n0 = (t % p.tiles_n) * F32Cfg::BN;
    const int k0 = split * p.per, k1 = min(p.g.K, k0 + p.per);
    f32x16_t acc;
    if (p.g.a_t) f32_tile<true, true>(p.g, m0, n0, k0, k1, smem, acc);
    else f32_tile<false, true>(p.g, m0, n0, k0, k1, smem, acc);
    const int lane = tid & 63, wave = tid >> 6;
    const int col = n0 + 32 * (wave & 1) + acc_col(lane);
    if (col >= p.g.N) return;
    float* out = p.splits > 1 ? p.part + int64_t(split) * p.g.M * p.g.N : static_cast<float*>(p.g.C);
    const int64_t ldo = p.splits > 1 ? p.g.N : p.g.ldc;
#pragma unroll
    for (int v = 0; v < 16; ++v) {
        const int row = m0 + 32 * (wave >> 1) + acc_row(v, lane);
        if (row < p.g.M) out[int64_t(row) * ldo + col] = acc[v];
    }
}

constexpr int kFinishThreads = 512;
__global__ __launch_bounds__(kFinishThreads) void tree_tail_finish_kernel(TailArgs a) {
    __shared__ float red[kFinishThreads / 64][5][64];
    const int tid = threadIdx.x;
    if (int(blockIdx.x) >= a.nseg) {
        // element i of the split results, then of the column sums
        int64_t i = int64_t(int(blockIdx.x) - a.nseg) * kFinishThreads + tid;
        if (i >= a.reduce_n) return;
#pragma unroll
        for (int q = 0; q < kTailProblems; ++q) {
            const TailProblem& p = a.p[q];
            if (q >= a.n || p.splits == 1 || !p.g.C) continue;
            const int64_t n = int64_t(p.g.M) * p.g.N;
            if (i < n) {
                float s = 0.f;
                for (int k = 0; k < p.splits; ++k) s += p.part[int64_t(k) * n + i];
                const int row = int(i / p.g.N);
                static_cast<float*>(p.g.C)[int64_t(row) * p.g.ldc + (i - int64_t(row) * p.g.N)] = s;
                return;
            }
            i -= n;
        }
        float s = 0.f;
        for (int k = 0; k < a.chunks; ++k) s += a.sum_part[int64_t(k) * a.cols + i];
        a.sum_out[i] = s;
        return;
    }
    // one word: its leaves are dealt to the waves, each lane adds up to five
    // columns (320 at a time), and the waves' sums are added in order
    const int32_t* order = a.seg;
    const int32_t* off = order + a.leaves;
    const int32_t* sid = off + a.nseg + 1;
    const int g = int(blockIdx.x), lane = tid & 63, wave = tid >> 6;
    constexpr int W = kFinishThreads / 64;
    const int k0 = off[g], k1 = off[g + 1];
    float* dst = a.demb + int64_t(sid[g]) * a.E;
    for (int e0 = 0; e0 < a.E; e0 += 320) {
        float s[5] = {0.f, 0.f, 0.f, 0.f, 0.f};
        for (int k = k0 + wave; k < k1; k += 4 * W) {
            float v[4][5];
#pragma unroll
            for (int j = 0; j < 4; ++j)
#pragma unroll
                for (int c = 0; c < 5; ++c) v[j][c] = 0.f;
            for (int part = 0; part < a.dx_parts; ++part) {
                float x[4][5];
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const bool ok = k + j * W < k1;
                    const float* row = a.dx + part * a.dx_stride + int64_t(order[ok ? k + j * W : k0]) * a.ldx;
#pragma unroll
                    for (int c = 0; c < 5; ++c) {
                        const int e = e0 + 64 * c + lane;
                        x[j][c] = ok && e < a.E ? row[e] : 0.f;
                    }
                }
#pragma unroll
                for (int j = 0; j < 4; ++j)
#pragma unroll
                    for (int c = 0; c < 5; ++c) v[j][c] += x[j][c];
            }
#pragma unroll
            for (int j = 0; j < 4; ++j)
#pragma unroll
                for (int c = 0; c < 5; ++c) s[c] += v[j][c];
        }
#pragma unroll
        for (int c = 0; c < 5; ++c) red[wave][c][lane] = s[c];
        __syncthreads();
        for (int i = tid; i < 320; i += kFinishThreads) {
            const int c = i >> 6, l = i & 63;
            if (e0 + i < a.E) {
                float t = 0.f;
#pragma unroll
                for (int w = 0; w < W; ++w) t += red[w][c][l];
                dst[e0 + i] = t;
            }
        }
        __syncthreads();
    }
}

// ------------------------------------------------------------- host side
// floats of the parts of an M x N result at most
inline size_t tail_part_floats(int64_t M, int64_t N) {
    const int64_t tiles = ((M + 63) / 64) * ((N + 63) / 64);
    return size_t(std::min<int64_t>(kTailSplits, 1 + kTailPieces / tiles)) * size_t(M) * size_t(N);
}
inline size_t tail_sum_floats(int64_t rows, int64_t cols) { return size_t((rows + kTailRows - 1) / kTailRows + 1) * size_t(cols); }

// Adds a contraction; empty ones (K = 0) give zeros.  `part` holds
// tail_part_floats(M, N) floats; `most` limits the splits.
inline void tail_add(TailArgs& a, const GemmDesc& g, float* part, int most = kTailSplits) {
    if (g.M <= 0 || g.N <= 0) return;
    TailProblem& p = a.p[a.n++];
    p.g = g;
    p.tiles_m = (g.M + F32Cfg::BM - 1) / F32Cfg::BM;
    p.tiles_n = (g.N + F32Cfg::BN - 1) / F32Cfg::BN;
    p.part = part;
    const int chunks = std::max(1, (g.K + F32Cfg::BK - 1) / F32Cfg::BK), tiles = p.tiles_m * p.tiles_n;
    // pieces in proportion to the work of a batch of three equal problems
    const int want = std::min({most, kTailSplits, 1 + kTailPieces / tiles, std::max(1, chunks / 2)});
    const int pieces = std::max(1, (kTailPieces / kTailProblems + tiles - 1) / tiles);
    const int n = std::max(1, std::min(want, pieces));
    p.per = (chunks + n - 1) / n * F32Cfg::BK;
    p.splits = std::max(1, (g.K + p.per - 1) / p.per);
}

// The two launches.
inline janus_status tail_run(TailArgs& a, const char* label, hipStream_t st) {
    double flops = 0.0;
    int items = 0;
    a.reduce_n = 0;
    for (int q = 0; q < a.n; ++q) {
        TailProblem& p = a.p[q];
        p.first = items;
        items += p.tiles_m * p.tiles_n * p.splits;
        if (p.splits > 1 && p.g.C) a.reduce_n += int64_t(p.g.M) * p.g.N;
        flops += 2.0 * p.g.M * p.g.N * double(p.g.K);
    }
    a.chunks = (a.rows + kTailRows - 1) / kTailRows;
    a.sum_first = items;
    items += a.chunks * ((a.cols + 63) / 64);
    a.reduce_n += a.cols;
    a.zero_first = items;
    items += int((a.demb_n + 4 * kTailZero - 1) / (4 * kTailZero));
    {
        TraceScope trace(label, flops, 0.0, st);
        hipLaunchKernelGGL(tree_tail_kernel, dim3(unsigned(items)), dim3(F32Cfg::NT), 0, st, a);
        JANUS_LAUNCH_CHECK();
    }
    const int64_t blocks = a.nseg + (a.reduce_n + kFinishThreads - 1) / kFinishThreads;
    TraceScope trace("tree_tail_finish", 0.0, 0.0, st);
    hipLaunchKernelGGL(tree_tail_finish_kernel, dim3(unsigned(blocks)), dim3(kFinishThreads), 0, st, a);
    JANUS_LAUNCH_CHECK();
    return JANUS_OK;
}

}  // namespace
}  // namespace janus
