// Plans of the contractions: how operands reach the kernels, which tiles, how
// many K splits, and the scratch these take.  Host code without device parts.
#pragma once

#include <algorithm>
#include <cstddef>
#include <cstdint>

#include "ops.hpp"

namespace janus {

struct TileDims {
    int BM, BN, BK;
};
constexpr TileDims kNtTile{256, 256, 64};    // bf16
constexpr TileDims kMidTile{128, 128, 64};   // bf16, grids of few tiles
constexpr TileDims kF32Tile{64, 64, 64};

// How an operand reaches the kernel: read in place, or first written to
// scratch as a K-contiguous copy (transposed when stored K-major, padded with
// zeros to a 16-byte multiple of K when its rows cannot be read in 16-byte
// chunks).
enum OperandMode { kInPlace = 0, kCopyRows = 1, kCopyTransposed = 2 };

struct NtPlan {
    bool fast = false;
    int64_t ldt = 0;                 // leading dimension of copies (K rounded to 64)
    int amode = kInPlace, bmode = kInPlace;
    int splits = 1, ktiles_per_split = 0;
    bool mid = false;                // 128 x 128 tiles
    size_t a_off = 0, b_off = 0, p_off = 0, bytes = 0;
};

inline bool rows16(const void* p, int64_t ld) { return reinterpret_cast<uintptr_t>(p) % 16 == 0 && ld % 8 == 0; }

// K splits of a contraction of `tiles` tiles and `ktiles` K blocks: the count
// with the least expected time, a K block taking about 1.5 us and the
// partials going to memory and back at 4 TB/s plus the launch that sums them.
// A grid of 160 tiles and more fills the chip without.
// (700 x 650 outputs over K = 10000: 35 us in 8 splits, 29 in 16.)
constexpr int kMaxSplits = 32;
inline int nt_tiles(int M, int N) {
    const int64_t t = int64_t((M + kNtTile.BM - 1) / kNtTile.BM) * ((N + kNtTile.BN - 1) / kNtTile.BN);
    return int(std::min<int64_t>(t, INT32_MAX));
}
inline int nt_splits(int tiles, int ktiles, int M, int N) {
    if (tiles >= 160) return 1;
    int best = 1;
    double least = 1.5 * ktiles;
    for (int n = 2; n <= std::min({kMaxSplits, 256 / tiles, ktiles / 4}); ++n) {
        const double us = 1.5 * ktiles / n + 5.0 + 2e-6 * n * double(M) * N;
        if (us < least) {
            least = us;
            best = n;
        }
    }
    return best;
}

// Whether 128 x 128 tiles are expected to be faster, with how many splits (at
// most those of the 256 x 256 tiles, whose scratch the caller has).  A K block
// takes about 0.65 us while the grid is one round of the chip, and a further
// round costs another 2.5 us to start.  (2624 x 656 outputs over K = 700: 24 us
// in 33 tiles of 256, 14 in 126 of 128; over 700 rows and K = 656 27 and 16.5;
// 700 x 10000 over K = 650, two rounds: 26 and 28; 4096 x 512 over K = 13000: 88
// with splits, 127 in 128 tiles without.)
inline bool nt_mid(int tiles, int ktiles, int M, int N, int& splits) {
    if (tiles >= 160) return false;
    auto sum = [&](int n) { return n > 1 ? 5.0 + 2e-6 * n * double(M) * N : 0.0; };
    double least = 1.5 * ((ktiles + splits - 1) / splits) + sum(splits);
    const int64_t small = int64_t((M + kMidTile.BM - 1) / kMidTile.BM) * ((N + kMidTile.BN - 1) / kMidTile.BN);
    int best = 0;
    for (int n = 1; n <= splits; ++n) {
        const double rounds = double((small * n + 255) / 256);
        const double us = 0.65 * ((ktiles + n - 1) / n) * rounds + 2.5 * (rounds - 1) + sum(n);
        if (us < least) {
            least = us;
            best = n;
        }
    }
    if (best == 0) return false;
    splits = best;
    return true;
}

// The fast path takes bf16 contractions with at least 16 rows and columns and
// K of 64 and more.  Below 128 rows or columns most of a 256-wide
// tile is padding, but such a contraction has few tiles and its K, when long,
// is then split over the chip, which the general kernel's serial walk of K
// cannot do (96 x 300 outputs over K = 15000: 3430 us there).  Where B
// alone is k-major, the rows are aligned and K is below 128, the general kernel's
// one launch is faster than the copies of B, and of A where K is no multiple of
// 8, if both are needed or both sides are short (softmax head of 60 rows, H 64:
// dh over 65 classes 12 us there and 22 here, 17 rows over 80 classes 2 us less
// there; over 128, 12 and 13; weight gradients of 256 x 16 over K = 64 1.2 us more
// there; with unaligned rows, or A k-major too, 18 to 20 us more).
inline NtPlan plan_nt(const GemmDesc& g) {
    NtPlan p;
    if (g.dtype != JANUS_BF16 || g.M < 16 || g.N < 16 || g.K < 64) return p;
    constexpr int64_t kMaxOff = int64_t(1) << 31;
    // an operand read in place: 16-byte chunks along K (K a multiple of 8, or
    // rows zero-padded past K), byte offsets in 31 bits
    auto in_place_ok = [&](const void* ptr, int64_t ld, const int32_t* idx, int64_t src_rows, bool zero_pad) {
        if (!rows16(ptr, ld) || (g.K % 8 != 0 && !zero_pad)) return false;
        if (idx) return src_rows > 0 && src_rows * ld * 2 < kMaxOff;
        return int64_t(kNtTile.BM) * ld * 2 < kMaxOff;
    };
    p.amode = g.a_t ? kCopyTransposed
                    : in_place_ok(g.A, g.lda, g.a_idx, g.a_src_rows, g.a_zero_pad) ? kInPlace : kCopyRows;
    p.bmode = g.b_t ? kCopyTransposed
                    : in_place_ok(g.B, g.ldb, g.b_idx, g.b_src_rows, g.b_zero_pad) ? kInPlace : kCopyRows;
    const int narrow = (g.M < 128) + (g.N < 128), copies = (p.amode != kInPlace) + (p.bmode != kInPlace);
    if (g.K < 128 && !g.a_t && g.b_t && narrow + copies >= 3 && narrow > 0 && rows16(g.A, g.lda) && rows16(g.B, g.ldb))
        return p;
    p.ldt = round_up(int64_t(g.K), 64);
    if (int64_t(kNtTile.BM) * p.ldt * 2 >= kMaxOff) return p;
    const int tiles = nt_tiles(g.M, g.N);
    const int ktiles = (g.K + kNtTile.BK - 1) / kNtTile.BK;
    int splits = nt_splits(tiles, ktiles, g.M, g.N);
    p.mid = nt_mid(tiles, ktiles, g.M, g.N, splits);
    p.ktiles_per_split = (ktiles + splits - 1) / splits;
    p.splits = (ktiles + p.ktiles_per_split - 1) / p.ktiles_per_split;
    size_t off = 0;
    auto take = [&](size_t bytes) { const size_t o = off; off += (bytes + 255) / 256 * 256; return o; };
    if (p.amode != kInPlace) p.a_off = take(size_t(g.M) * p.ldt * 2);
    if (p.bmode != kInPlace) p.b_off = take(size_t(g.N) * p.ldt * 2);
    if (p.splits > 1) p.p_off = take(size_t(p.splits) * g.M * g.N * 4);
    p.bytes = off;
    p.fast = true;
    return p;
}

// K splits of a float32 contraction: the count with the least expected time.
// Up to four workgroups share a CU (1024 on the chip); a chunk of 64 k takes
// a workgroup about 1.6 us with one per CU and 3.4 us with four (the MFMA
// rate), a split's partials go out and back at 4 TB/s, and the sum is a
// launch.  (1024 x 300 outputs over K = 800: 88 us in one piece.)
constexpr size_t kF32Scratch = size_t(16) << 20;   // partials of a contraction at most: 1024 tiles
inline int f32_splits(const GemmDesc& g) {
    const int64_t tiles = int64_t((g.M + kF32Tile.BM - 1) / kF32Tile.BM) * ((g.N + kF32Tile.BN - 1) / kF32Tile.BN);
    const int chunks = (g.K + kF32Tile.BK - 1) / kF32Tile.BK;
    auto us = [&](int n) {
        const int64_t wgs = tiles * n;
        const double waves = double((wgs + 1023) / 1024), per_cu = std::min(4.0, double(wgs) / 256.0);
        const double t = waves * chunks / n * std::max(1.6, 0.85 * per_cu);
        return n == 1 ? t : t + 5.0 + 2e-6 * n * double(g.M) * g.N;
    };
    int best = 1;
    for (int n = 2; n <= std::min(kMaxSplits, chunks) && size_t(n) * g.M * g.N * 4 <= kF32Scratch; ++n)
        if (us(n) < us(best)) best = n;
    return best;
}

// Scratch enough for a contraction whose size is known up to one side
// (GemmSize).  The split counts follow expected times and whole K blocks, so
// they do not grow evenly with K or M: a plan of a smaller K can have more
// splits (320 x 240 outputs: 8 over K = 2048, 7 over 2160).  Where a side may
// be smaller, the bound is what the rules allow at most, whatever they choose.
inline size_t gemm_scratch_bound(const GemmDesc& g, GemmSize size) {
    auto round = [](size_t b) { return (b + 255) / 256 * 256; };
    const size_t out = size_t(g.M) * g.N * 4;
    if (g.dtype == JANUS_F32) {
        const int chunks = (g.K + kF32Tile.BK - 1) / kF32Tile.BK;
        size_t n = size_t(std::min(kMaxSplits, chunks));
        if (size == GemmSize::kExact) n = size_t(f32_splits(g));
        if (size == GemmSize::kUpToK && out > 0) n = std::min(n, kF32Scratch / out);
        return n > 1 ? std::min(kF32Scratch, n * out) : 0;
    }
    GemmDesc q = g;
    q.A = q.B = nullptr;            // 16-byte aligned stand-ins (unaligned caller tensors may need more;
                                    // gemm() then takes the slower path that needs none)
    q.a_src_rows = q.a_idx ? int64_t(1) : 0;
    q.b_src_rows = q.b_idx ? int64_t(1) : 0;
    const NtPlan p = plan_nt(q);
    if (!p.fast) return 0;
    size_t b = 0;
    if (p.amode != kInPlace) b += round(size_t(g.M) * p.ldt * 2);
    if (p.bmode != kInPlace) b += round(size_t(g.N) * p.ldt * 2);
    constexpr size_t kTileBytes = size_t(kNtTile.BM) * kNtTile.BN * 4;
    int n = p.splits;
    if (size != GemmSize::kExact) {
        n = std::min(kMaxSplits, (g.K + kNtTile.BK - 1) / kNtTile.BK / 4);
        if (size == GemmSize::kUpToK) n = std::min(n, 256 / nt_tiles(g.M, g.N));
    }
    if (n > 1) b += round(size == GemmSize::kUpToM ? std::min(256 * kTileBytes, size_t(n) * out) : size_t(n) * out);
    return b;
}

}  // namespace janus
