// The float32 contraction's tile: operands, LDS layouts and main loop, shared
// by the plain contraction and the MSE head.
#pragma once

#include "device.hpp"
#include "ops.hpp"

namespace janus {
namespace {

// --------------------------------------------------------- float32 path
// C = A . B^T for float32 operands in any of the three layouts, 64 x 64 tiles
// of four waves (one 32 x 32 quadrant each, 32x32x2 products), K in chunks
// of 64.  Such a contraction is bound by the latency of its loads, not by
// their bytes: a chunk's MFMA work (0.85 us per wave) is about a load round
// trip, so the next chunk is loaded while one is contracted, four workgroups
// share a CU, and a K that is long for the number of tiles is split over the
// chip (partials summed in order by splitk_reduce_kernel).
//
// An operand whose k is contiguous goes to LDS as [row][k]: a lane reads the
// eight consecutive k of its row.  One whose rows are contiguous (stored
// k-major) goes there as it is, [k][row], and a lane reads its eight k one by
// one (consecutive lanes take consecutive words), so nothing is transposed.
// Product step jj of k-step ks takes k = 16 ks + 8 (l / 32) + jj of both.
//
// Loads are 16 bytes at any 4-byte alignment.  Rows past the operand are
// clamped to its last row (their products land in rows and columns that are
// not stored); a row-contiguous piece that crosses the last row, and the
// chunk that crosses K, are read element by element with zeros past the end.
struct F32Cfg {
    static constexpr int BM = 64, BN = 64, BK = 64, NT = 256;
    static constexpr int LD = BK + 4;                       // pitch of both LDS layouts
    static constexpr int SMEM = 2 * 64 * LD * 4;
};

struct float4_u {   // four floats at 4-byte alignment
    float x, y, z, w;
} __attribute__((packed, aligned(4)));

template <bool T>   // T: stored k-major (rows contiguous)
struct F32Operand {
    const float* p[4];       // !T: this thread's four rows
    const float* base;       // T
    int64_t ld;
    const int32_t* kidx;     // T: k -> stored row, or NULL
    int koff[4];             // T: k rows of the coming chunk (with kidx)
    int c4;                  // !T: first k of the piece in the chunk; T: first row of the piece
    int nv;                  // T: rows of the piece inside the operand (0 .. 4)
    float4_u v[4];

    // rows r0 .. of an operand with `rows` rows, this thread's pieces: !T:
    // rows tid / 16 + 16 i, k 4 (tid % 16); T: k tid / 16 + 16 i, rows 4 (tid % 16)
    __device__ __forceinline__ void init(const float* b, int64_t l, const int32_t* idx, int r0, int rows, int tid) {
        base = b;
        ld = l;
        kidx = idx;
        c4 = 4 * (tid & 15);
        if constexpr (!T) {
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int r = min(r0 + (tid >> 4) + 16 * i, rows - 1);
                p[i] = b + (idx ? int64_t(idx[r]) : int64_t(r)) * l;
            }
        } else {
            nv = min(max(rows - (r0 + c4), 0), 4);
            base = b + (nv > 0 ? r0 + c4 : 0);
        }
    }
    // stored rows of chunk k0 (a chunk ahead of load())
    __device__ __forceinline__ void index(int k0, int k1, int tid) {
        if constexpr (T) {
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int k = min(k0 + (tid >> 4) + 16 * i, k1 - 1);
                koff[i] = kidx ? kidx[k] : k;
            }
        }
    }
    __device__ __forceinline__ void load(int k0, int k1, int tid) {
        if constexpr (!T) {
            const int n = k1 - (k0 + c4);   // k of this thread's pieces inside
            if (n >= 4) {
#pragma unroll
                for (int i = 0; i < 4; ++i) v[i] = *reinterpret_cast<const float4_u*>(p[i] + k0 + c4);
            } else {
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const float* q = p[i] + k0 + c4;
                    v[i] = float4_u{n > 0 ? q[0] : 0.f, n > 1 ? q[1] : 0.f, n > 2 ? q[2] : 0.f, 0.f};
                }
            }
        } else {
            const bool part = nv > 0 && nv < 4;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const float* q = base + int64_t(koff[i]) * ld;
                if (!part) v[i] = nv ? *reinterpret_cast<const float4_u*>(q) : float4_u{0.f, 0.f, 0.f, 0.f};
                else v[i] = float4_u{q[0], nv > 1 ? q[1] : 0.f, nv > 2 ? q[2] : 0.f, 0.f};
            }
            if (k0 + F32Cfg::BK > k1) {   // the chunk that crosses the end: the clamped k rows count as zero
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    if (k0 + (tid >> 4) + 16 * i >= k1) v[i] = float4_u{0.f, 0.f, 0.f, 0.f};
            }
        }
    }
    __device__ __forceinline__ void store(float* s, int tid) const {
#pragma unroll
        for (int i = 0; i < 4; ++i)
            *reinterpret_cast<float4*>(s + ((tid >> 4) + 16 * i) * F32Cfg::LD + c4) =
                make_float4(v[i].x, v[i].y, v[i].z, v[i].w);
    }
    // the eight k of k-step ks for this lane's row `r` (tile relative)
    __device__ static __forceinline__ void frag(const float* s, int r, int ks, int lane, float (&f)[8]) {
        const int k = 16 * ks + 8 * (lane >> 5);
        if constexpr (!T) {
            const float4 a = *reinterpret_cast<const float4*>(s + r * F32Cfg::LD + k);
            const float4 b = *reinterpret_cast<const float4*>(s + r * F32Cfg::LD + k + 4);
            f[0] = a.x; f[1] = a.y; f[2] = a.z; f[3] = a.w;
            f[4] = b.x; f[5] = b.y; f[6] = b.z; f[7] = b.w;
        } else {
#pragma unroll
            for (int j = 0; j < 8; ++j) f[j] = s[(k + j) * F32Cfg::LD + r];
        }
    }
};

// One workgroup's tile at (m0, n0) over k in [k0, k1): acc is this wave's
// quadrant, rows 32 (wave / 2), columns 32 (wave % 2).
template <bool AT, bool BT>
__device__ __forceinline__ void f32_tile(const GemmDesc& g, int m0, int n0, int k0, int k1, float* smem, f32x16_t& acc) {
    using C = F32Cfg;
    float* sA = smem;
    float* sB = smem + 64 * C::LD;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    F32Operand<AT> a;
    F32Operand<BT> b;
    a.init(static_cast<const float*>(g.A), g.lda, g.a_idx, m0, g.M, tid);
    b.init(static_cast<const float*>(g.B), g.ldb, g.b_idx, n0, g.N, tid);
#pragma unroll
    for (int v = 0; v < 16; ++v) acc[v] = 0.f;
    if (k0 >= k1) return;
    const int ar = 32 * (wave >> 1) + (lane & 31), br = 32 * (wave & 1) + (lane & 31);
    a.index(k0, k1, tid);
    b.index(k0, k1, tid);
    a.load(k0, k1, tid);
    b.load(k0, k1, tid);
    a.index(k0 + C::BK, k1, tid);
    b.index(k0 + C::BK, k1, tid);
    for (int k = k0; k < k1; k += C::BK) {
        __syncthreads();   // the previous chunk has been read
        a.store(sA, tid);
        b.store(sB, tid);
        __syncthreads();
        if (k + C::BK < k1) {
            a.load(k + C::BK, k1, tid);
            b.load(k + C::BK, k1, tid);
            a.index(k + 2 * C::BK, k1, tid);
            b.index(k + 2 * C::BK, k1, tid);
        }
        // a chunk's products start from zero and are added to the total at its
        // end: the sum over a long K then rounds like one of K / 64 terms
        const int steps = (min(C::BK, k1 - k) + 15) / 16;
        f32x16_t part;
#pragma unroll
        for (int v = 0; v < 16; ++v) part[v] = 0.f;
#pragma unroll
        for (int ks = 0; ks < C::BK / 16; ++ks) {
            if (ks >= steps) break;
            float fa[8], fb[8];
            F32Operand<AT>::frag(sA, ar, ks, lane, fa);
            F32Operand<BT>::frag(sB, br, ks, lane, fb);
#pragma unroll
            for (int j = 0; j < 8; ++j) part = __builtin_amdgcn_mfma_f32_32x32x2f32(fa[j], fb[j], part, 0, 0, 0);
        }
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[v] += part[v];
    }
}

}  // namespace
}  // namespace janus
