// Recurrence kernels whose row groups each live on one XCD.
//
// The rows of a batch are independent sequences, so a step's exchange of h
// (forward) or dG (backward) is needed only among the workgroups that share
// rows.  Here the batch is cut in groups of 16 RT sorted rows and each group
// is worked by NU workgroups (at most the CUs of one XCD) that run on the
// same XCD: workgroup m of a group owns units [U m, U m + U), U = 8 Q, keeps
// their weights in VGPRs for the whole launch, and the group exchanges its
// step through that XCD's L2 alone.  Different groups never wait for each
// other.
//
// What bounds a step is the chain "load operand -> MFMA -> sum over the
// waves -> cell -> store", all latency, so the exchange has no barrier and no
// flag: the operand slots are prefilled with a bit pattern no result takes
// (0xffffffff, a NaN; results that equal it are stored as another NaN), and a
// consumer loads its operand until no word holds the pattern.  That makes a
// step one L2 store and one L2 load deep, where the device-wide barrier costs
// an acknowledged write-through, an atomic and a poll in memory (about 3 us).
// Four slots are used in turn, so the exchange stays in the L2; see the slot
// argument below.
//
// Memory operations complete in issue order for a wave that waits for its
// loads, so nothing a poll need not wait for stands between a publication and
// the next poll: the loads of the next step's own operands, and the forward's
// results for later kernels (gates, c, h), are issued once the operand of the
// exchange has arrived, and complete while it is multiplied.  (The backward's
// only results, dG, follow their publication: 3% better in float32 than after
// the poll, the same in bf16.)  (Forward per step,
// stores and loads issued right after the publication: H 1024 2.9 us, H 656
// 2.5, H 512 1.9; issued after the poll: 2.2, 1.6, 1.5.)
//
// Measured per time step against the kernels with a device-wide barrier:
// H 1024, B 128: forward 2.2 against 5.9 us, backward 3.2 against 7.7; H 656,
// B 20: 1.6 against 4.5 and 2.2 against 6.5; H 512, B 33: forward 1.5 against
// 4.1.  float32, H 256, B 32, against one launch per step: 1.6 against 9.7 us
// and 2.3 against 53.  A launch adds 5-22 us before its first step (mostly its
// weights).  The backward's step is longer by its operand, four times the
// forward's: every workgroup reads all gate columns of its rows from the L2.
//
// Inside a workgroup the eight waves split the contraction's k range (each
// loads only its share of the operand, once), add their partial tiles through
// LDS, and each cell belongs to one thread.
//
// Slots.  Forward step t reads h_{t-1} from slot t % 4 and stores h_t to slot
// (t + 1) % 4; the backward reads dG_{t+1} from slot (t + 1) % 4 and stores
// dG_t to slot t % 4.  When a workgroup has all operands of a step, every
// member has finished the previous step and so has read the slot before this
// one: its owner refills its own pieces of that slot with the pattern, after
// storing its result.  The slot is written again two steps later and read the
// step after.  Each thread waits for its earlier stores (the refill among
// them) between its poll and its next result, so whoever has read a thread's
// result of one step finds the pattern or the new value in the pieces that
// thread refilled before, never the old value.
#pragma once

#include <type_traits>

#include "device.hpp"
#include "lstm_persist.hpp"

namespace janus {
namespace xcd {

using persist::act_at;
using persist::kOutOfRange;
using persist::make_rsrc;
using persist::off_at;
using persist::Sync;

typedef float f32x4_t __attribute__((ext_vector_type(4)));

constexpr int kThreads = 512;
constexpr int kWaves = kThreads / 64;
constexpr int kSlots = 4;
constexpr int kMaxGroups = 16;            // row groups of one launch (256 rows of 16)
constexpr int kSpinLimit = 1 << 20;       // bounded wait for an operand
constexpr uint32_t kEmpty = 0xffffffffu;  // "not stored yet"

// Operand layout: k-groups of KG = 4 EPL columns (EPL elements are 16 bytes);
// element (row r of a 16-row tile, column k) is element k % EPL of lane
// ((k % KG) / EPL) * 16 + r of its k-group, which is the lane and order in
// which a 16x16 MFMA takes it as the B operand.
template <typename T>
struct Lay {
    static constexpr int EPL = 16 / int(sizeof(T));
    static constexpr int KG = 4 * EPL;
    __host__ __device__ static int64_t index(int64_t tile, int nkg, int r, int k) {
        return ((tile * nkg + k / KG) * 64 + ((k % KG) / EPL) * 16 + r) * EPL + k % EPL;
    }
};

__device__ __forceinline__ f32x4_t mma(uint4 a, uint4 b, f32x4_t acc, const bf16_t*) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, a), __builtin_bit_cast(bf16x8_t, b),
                                                   acc, 0, 0, 0);
}
// float32: the four k of a lane one after another (the same k of both operands)
__device__ __forceinline__ f32x4_t mma(uint4 a, uint4 b, f32x4_t acc, const float*) {
    acc = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(a.x), __uint_as_float(b.x), acc, 0, 0, 0);
    acc = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(a.y), __uint_as_float(b.y), acc, 0, 0, 0);
    acc = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(a.z), __uint_as_float(b.z), acc, 0, 0, 0);
    acc = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(a.w), __uint_as_float(b.w), acc, 0, 0, 0);
    return acc;
}

// An operand piece still holds the pattern.  bf16 results are stored 8 bytes
// at a time (one aligned access, which a reader sees whole), float32 results
// 4 bytes at a time.
__device__ __forceinline__ bool empty_piece(uint4 v, const bf16_t*) { return max(v.y, v.w) == kEmpty; }
__device__ __forceinline__ bool empty_piece(uint4 v, const float*) {
    return max(max(v.x, v.y), max(v.z, v.w)) == kEmpty;
}
__device__ __forceinline__ uint32_t not_empty(uint32_t w) { return w == kEmpty ? 0xfffffffeu : w; }

// loads that skip the L1 (device scope): they return what the L2 holds
__device__ __forceinline__ uint4 load_l2(__amdgpu_buffer_rsrc_t rs, uint32_t off) { return persist::load16_l2(rs, off); }
__device__ __forceinline__ void store_b64(__amdgpu_buffer_rsrc_t rs, uint32_t off, uint32_t x, uint32_t y) {
    persist::store8<persist::kStoreBack>(rs, off, make_uint2(x, y));
}
__device__ __forceinline__ void store_b32(__amdgpu_buffer_rsrc_t rs, uint32_t off, uint32_t x) {
    __builtin_amdgcn_raw_buffer_store_b32(x, rs, int(off), 0, persist::kStoreBack);
}
__device__ __forceinline__ void store_b128(__amdgpu_buffer_rsrc_t rs, uint32_t off, uint4 v) {
    persist::store16<persist::kStoreBack>(rs, off, v);
}
// every earlier memory operation of this wave has completed
__device__ __forceinline__ void wait_own_stores() {
    __atomic_signal_fence(__ATOMIC_SEQ_CST);
    __builtin_amdgcn_s_waitcnt(0x0f70);   // vmcnt(0)
    __atomic_signal_fence(__ATOMIC_SEQ_CST);
}

// Place of a workgroup: member m of row group g, or g = -1 for a workgroup
// that has nothing to do.  A launch has the same number of workgroups for
// every XCD, a multiple of nu, and they count themselves on their XCD.  The
// i-th of XCD x belongs to its turn i / nu, group (i / nu) xccs + x; once the
// turn's nu workgroups have arrived (all on one XCD, `local`) it starts,
// without waiting for the rest of the device.  Where the placement was
// uneven, a turn stays incomplete: when every workgroup of the launch has been
// counted, those of incomplete turns and those past their XCD's last turn are
// ranked over all XCDs and serve the groups left in consecutive nu; the steps
// of such a group are separated by a barrier of its own with device-scope
// fences (with xccs 0, all groups).  All of them derive the same ranks from
// the final counts.
// (Waiting for the whole launch on one counter took 12 us of a launch of 256;
// a turn is complete after 1.4.)
struct Place {
    int g, m, local;
};
template <class S>
__device__ __forceinline__ unsigned census_at(S* s, int q) {
    return __hip_atomic_load(&s->census[q][0], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
template <class S>
__device__ __forceinline__ Place take_place(S* s, int nu, int groups, int xccs) {
    __shared__ int place[3];
    if (threadIdx.x == 0) {
        const int x = int(persist::xcc_id());
        const int i =
            int(__hip_atomic_fetch_add(&s->census[x][0], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
        // turns of XCD q: the groups q, q + xccs, .. below `groups`
        auto turns = [&](int q) { return q < xccs ? (groups - q + xccs - 1) / xccs : 0; };
        const int turn = i / nu;
        int g = -1, m = i % nu, local = 0;
        unsigned c[persist::kMaxXcds];
        for (int spins = 0;; ++spins) {
            if (turn < turns(x) && int(census_at(s, x)) >= (turn + 1) * nu) {
                g = turn * xccs + x;
                local = 1;
                break;
            }
            unsigned all = 0;
            if (turn >= turns(x) || (spins & 15) == 15) {
#pragma unroll
                for (int q = 0; q < persist::kMaxXcds; ++q) c[q] = census_at(s, q);
#pragma unroll
                for (int q = 0; q < persist::kMaxXcds; ++q) all += c[q];
            }
            if (all == gridDim.x) {
                const int full = min(turns(x), int(c[x]) / nu);
                if (turn < full) continue;   // the turn was completed meanwhile
                // rank among the workgroups outside complete turns, and the
                // group of that rank among those no complete turn works
                int rank = i - full * nu;
                for (int q = 0; q < x; ++q) rank += int(c[q]) - min(turns(q), int(c[q]) / nu) * nu;
                int left = rank / nu;
                m = rank % nu;
                for (int k = 0; k < groups && g < 0; ++k) {
                    bool worked = false;
                    if (xccs > 0) worked = k / xccs < int(census_at(s, k % xccs)) / nu;
                    if (!worked && left-- == 0) g = k;
                }
                break;
            }
            if (turn >= turns(x)) __builtin_amdgcn_s_sleep(16);
            if ((spins & 63) == 63 && __hip_atomic_load(&s->error, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0u)
                break;
            if (spins > persist::kSpinLimit) {
                __hip_atomic_store(&s->error, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                break;
            }
        }
        place[0] = g;
        place[1] = m;
        place[2] = local;
    }
    __syncthreads();
    return Place{place[0], place[1], place[2]};
}

// Barrier of a group that does not share an L2: release, arrive, wait, acquire.
template <class S>
__device__ __forceinline__ void remote_barrier(S* s, int g, unsigned& phase, unsigned members) {
    ++phase;
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
    __syncthreads();
    if (threadIdx.x == 0) {
        __hip_atomic_fetch_add(&s->group[g][0], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        persist::spin_until(s, &s->group[g][0], phase * members);
    }
    __syncthreads();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
}

// N operand pieces of 16 bytes per lane, loaded until none holds the pattern
// (`poll`; only the k-groups that still do are loaded again).  Offsets out
// of range read zeros, which pass.  A wait that runs out sets the error flag;
// from then on (`dead`) nothing waits.
template <typename T, int N, class Off, class S>
__device__ __forceinline__ void load_operand(uint4 (&f)[N], __amdgpu_buffer_rsrc_t rs, Off off, bool poll, S* s,
                                             bool& dead) {
#pragma unroll
    for (int i = 0; i < N; ++i) f[i] = load_l2(rs, off(i));
    if (!poll || dead) return;
    uint32_t need = 0;
#pragma unroll
    for (int i = 0; i < N; ++i)
        if (__any(empty_piece(f[i], static_cast<const T*>(nullptr)))) need |= 1u << i;
    int spins = 0;
    while (need != 0u) {
#pragma unroll
        for (int i = 0; i < N; ++i)
            if (need >> i & 1u) f[i] = load_l2(rs, off(i));
#pragma unroll
        for (int i = 0; i < N; ++i)
            if ((need >> i & 1u) && !__any(empty_piece(f[i], static_cast<const T*>(nullptr)))) need &= ~(1u << i);
        if ((++spins & 255) == 0) {
            if (__hip_atomic_load(&s->error, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0u) dead = true;
            if (spins > kSpinLimit) {
                __hip_atomic_store(&s->error, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                dead = true;
            }
            if (dead) return;
        }
    }
}

// --------------------------------------------------------------- cell values
// the four gates of a cell (interleaved columns 4u .. 4u + 3): 8 or 16 bytes
template <typename T> struct Gates;
template <> struct Gates<bf16_t> {
    uint2 w;
    __device__ __forceinline__ void load(__amdgpu_buffer_rsrc_t rs, uint32_t off) {
        typedef uint32_t u32x2_t __attribute__((ext_vector_type(2)));
        const u32x2_t v = __builtin_amdgcn_raw_buffer_load_b64(rs, int(off), 0, 0);
        w = make_uint2(v.x, v.y);
    }
    __device__ __forceinline__ void get(float (&g)[4]) const {
        g[0] = __uint_as_float(w.x << 16);
        g[1] = __uint_as_float(w.x & 0xffff0000u);
        g[2] = __uint_as_float(w.y << 16);
        g[3] = __uint_as_float(w.y & 0xffff0000u);
    }
    __device__ __forceinline__ void set(const float (&g)[4]) {
        w.x = uint32_t(f2bf(g[0])) | (uint32_t(f2bf(g[1])) << 16);
        w.y = uint32_t(f2bf(g[2])) | (uint32_t(f2bf(g[3])) << 16);
    }
    __device__ __forceinline__ void store(__amdgpu_buffer_rsrc_t rs, uint32_t off) const { store_b64(rs, off, w.x, w.y); }
    __device__ __forceinline__ void publish(__amdgpu_buffer_rsrc_t rs, uint32_t off) const {
        store_b64(rs, off, w.x, not_empty(w.y));
    }
    __device__ static __forceinline__ void clear(__amdgpu_buffer_rsrc_t rs, uint32_t off) { store_b64(rs, off, kEmpty, kEmpty); }
};
template <> struct Gates<float> {
    uint4 w;
    __device__ __forceinline__ void load(__amdgpu_buffer_rsrc_t rs, uint32_t off) { w = persist::load16(rs, off); }
    __device__ __forceinline__ void get(float (&g)[4]) const {
        g[0] = __uint_as_float(w.x);
        g[1] = __uint_as_float(w.y);
        g[2] = __uint_as_float(w.z);
        g[3] = __uint_as_float(w.w);
    }
    __device__ __forceinline__ void set(const float (&g)[4]) {
        w = make_uint4(__float_as_uint(g[0]), __float_as_uint(g[1]), __float_as_uint(g[2]), __float_as_uint(g[3]));
    }
    __device__ __forceinline__ void store(__amdgpu_buffer_rsrc_t rs, uint32_t off) const { store_b128(rs, off, w); }
    __device__ __forceinline__ void publish(__amdgpu_buffer_rsrc_t rs, uint32_t off) const {
        store_b128(rs, off, make_uint4(not_empty(w.x), not_empty(w.y), not_empty(w.z), not_empty(w.w)));
    }
    __device__ static __forceinline__ void clear(__amdgpu_buffer_rsrc_t rs, uint32_t off) {
        store_b128(rs, off, make_uint4(kEmpty, kEmpty, kEmpty, kEmpty));
    }
};

// ------------------------------------------------------------------ set-up
// Gate-interleaved copies of a layer's Wx and b: row n of the copy is row
// (n % 4) H + n / 4, in 16-byte pieces where the rows are whole pieces, one a
// thread (H 656, with the set-up of the forward: 5 us; four pieces a thread on a
// quarter of the workgroups: 17).
template <typename T>
struct Interleave {
    const T* W;
    T* Wi;
    const T* b;
    T* bi;
    int H, cols;
};
template <typename T>
__device__ __forceinline__ void interleave(const Interleave<T>& a, int64_t i0, int64_t stride) {
    const int H = a.H;
    auto copy = [&](auto* d, const auto* s, int per_row) {
        const int64_t n = int64_t(4) * H * per_row;
        for (int64_t i = i0; i < n; i += stride) {
            const int r = int(n <= 0xffffffffll ? int64_t(unsigned(i) / unsigned(per_row)) : i / per_row);
            d[i] = s[(int64_t(r & 3) * H + (r >> 2)) * per_row + (i - int64_t(r) * per_row)];
        }
    };
    constexpr int P = 16 / int(sizeof(T));
    if (a.cols % P == 0 && ((reinterpret_cast<uintptr_t>(a.W) | reinterpret_cast<uintptr_t>(a.Wi)) & 15) == 0)
        copy(reinterpret_cast<uint4*>(a.Wi), reinterpret_cast<const uint4*>(a.W), a.cols / P);
    else
        copy(a.Wi, a.W, a.cols);
    copy(a.bi, a.b, 1);
}
template <typename T>
__global__ __launch_bounds__(256) void interleave_kernel(Interleave<T> a) {
    interleave(a, int64_t(blockIdx.x) * 256 + threadIdx.x, int64_t(gridDim.x) * 256);
}

// Forward: slot 0 = h0 of rows rbase + [0, 16 tiles) (zero past the batch and
// past H), the other slots empty, the barrier counters zero, and the initial
// state in the activation store (Hs, Cs rows [0, B), columns [0, B) of HT);
// a length-0 sequence ends in its initial state.  The first wblocks workgroups
// interleave the layer's weights instead.
template <typename T>
__global__ __launch_bounds__(256) void fwd_init_kernel(int B, int H, int64_t ldh, int rbase, int tiles, int nkg,
                                                       const int32_t* perm, const float* h0, const float* c0, T* Hs,
                                                       float* Cs, int active0, float* hT, float* cT, T* HT, int64_t ldht,
                                                       T* ring, Sync* sync, Interleave<T> weights, int wblocks) {
    using L = Lay<T>;
    if (int(blockIdx.x) < wblocks) {
        interleave(weights, int64_t(blockIdx.x) * 256 + threadIdx.x, int64_t(wblocks) * 256);
        return;
    }
    const int64_t n = int64_t(tiles) * nkg * 64 * L::EPL;   // elements of a slot
    const int64_t stride = int64_t(gridDim.x - wblocks) * 256,
                  i0 = int64_t(blockIdx.x - wblocks) * 256 + threadIdx.x;
    uint4* rest = reinterpret_cast<uint4*>(ring + n);
    for (int64_t i = i0; i < (kSlots - 1) * n / L::EPL; i += stride)
        rest[i] = make_uint4(kEmpty, kEmpty, kEmpty, kEmpty);
    uint32_t* cnt = reinterpret_cast<uint32_t*>(sync);
    for (int64_t i = i0; i < int64_t(persist::kSyncCounterBytes / 4); i += stride) cnt[i] = 0u;
    // (row, unit) pairs, units padded to whole k-groups
    const int Kp = nkg * L::KG;
    for (int64_t i = i0; i < int64_t(tiles) * 16 * Kp; i += stride) {
        const int u = int(i % Kp), rr = int(i / Kp), r = rbase + rr;
        const bool ok = r < B && u < H;
        float hv = 0.f;
        if (ok) {
            const int b = perm ? perm[r] : r;
            hv = h0 ? h0[int64_t(b) * H + u] : 0.f;
            const float cv = c0 ? c0[int64_t(b) * H + u] : 0.f;
            Hs[int64_t(r) * ldh + u] = from_f<T>(hv);
            Cs[int64_t(r) * ldh + u] = cv;
            if (HT) HT[int64_t(u) * ldht + r] = from_f<T>(hv);
            if (r >= active0) {
                if (hT) hT[int64_t(b) * H + u] = hv;
                if (cT) cT[int64_t(b) * H + u] = cv;
            }
        }
        // a NaN in h0 must not read as an empty piece
        T q = from_f<T>(hv);
        if (hv != hv) q = from_f<T>(__uint_as_float(0x7fc00000u));
        ring[L::index(rr >> 4, nkg, rr & 15, u)] = q;
    }
}

// Backward: every slot empty, the barrier counters zero, and the map of the
// interleaved gate rows to gate-major rows (perm4, may be NULL).
static __global__ __launch_bounds__(256) void bwd_init_kernel(uint4* ring, int64_t n16, Sync* sync, int H,
                                                              int32_t* perm4) {
    const int64_t stride = int64_t(gridDim.x) * 256, i0 = int64_t(blockIdx.x) * 256 + threadIdx.x;
    for (int64_t i = i0; i < n16; i += stride) ring[i] = make_uint4(kEmpty, kEmpty, kEmpty, kEmpty);
    uint32_t* cnt = reinterpret_cast<uint32_t*>(sync);
    for (int64_t i = i0; i < int64_t(persist::kSyncCounterBytes / 4); i += stride) cnt[i] = 0u;
    if (perm4)
        for (int64_t i = i0; i < 4 * H; i += stride) perm4[i] = int(i & 3) * H + int(i >> 2);
}

// db[g * H + u] = sum over the row groups of their sums, in group order
static __global__ __launch_bounds__(256) void db_reduce_kernel(const float* part, int groups, int H, float* db) {
    const int n = blockIdx.x * 256 + threadIdx.x;
    if (n >= 4 * H) return;
    float s = 0.f;
    for (int q = 0; q < groups; ++q) s += part[int64_t(q) * 4 * H + n];
    db[(n & 3) * H + (n >> 2)] = s;
}

// ----------------------------------------------------------------- forward
template <typename T>
struct FwdArgs {
    int H, B, t_eff, fixed;
    int rbase;                 // first sorted row of this launch
    int groups, nu, nkg;       // row groups, workgroups of a group, k-groups of the operand
    int xccs;                  // XCDs the groups are dealt to (0: no group shares an L2)
    int steps[kMaxGroups];     // steps each group runs (length of its first row)
    const int32_t* active;
    const int32_t* perm;
    const T* Wh;
    T* Hs;                     // may be NULL
    float* Cs;
    const T* XG;
    T* Gs;
    T* y;                      // may be NULL
    float* hT;
    float* cT;
    int64_t ldh, ldg;
    T* HT;                     // bf16 only, may be NULL
    int64_t ldht;
    T* ring;
    Sync* sync;
};

template <int Q, int RT>
struct FwdCfg {
    static constexpr int U = 8 * Q;                  // units of a workgroup
    static constexpr int NT = 2 * Q;                 // 16-row tiles: four units x four gates
    static constexpr int NP = NT * RT;               // (gate tile, row tile) pairs
    static constexpr int CPW = (NP + kWaves - 1) / kWaves;
    static constexpr int TILE = 64 * 4;              // floats of a 16 x 16 tile
    static constexpr bool DB = 2 * kWaves * NP * TILE * 4 <= 128 * 1024;   // two buffers for the partial tiles
    static constexpr int SMEM = (DB ? 2 : 1) * kWaves * NP * TILE * 4;
};

template <typename T, int Q, int RT>
__global__ __launch_bounds__(kThreads) void lstm_fwd_xcd(FwdArgs<T> a) {
    using L = Lay<T>;
    using C = FwdCfg<Q, RT>;
    constexpr int J = 32 * Q / L::KG;     // k-groups of a wave
    constexpr int NT = C::NT, NP = C::NP, CPW = C::CPW;
    extern __shared__ __align__(16) unsigned char smem_raw[];
    f32x4_t* red = reinterpret_cast<f32x4_t*>(smem_raw);   // [buffer][wave][pair][64]
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const Place pl = take_place(a.sync, a.nu, a.groups, a.xccs);
    const int g = __builtin_amdgcn_readfirstlane(pl.g), m = __builtin_amdgcn_readfirstlane(pl.m);
    const bool local = __builtin_amdgcn_readfirstlane(pl.local) != 0;
    if (g < 0) return;
    const int H = a.H, v0 = m * C::U, row0 = a.rbase + 16 * RT * g;
    const int kv = L::EPL == 4 ? (H + 3) & ~3 : H;   // columns that hold values (padding ones zero)
    const int lr = lane & 15, lq = lane >> 4;

    // weights: tile i holds units v0 + 4 i + [0, 4), gates interleaved
    uint4 w[NT][J];
#pragma unroll
    for (int i = 0; i < NT; ++i)
#pragma unroll
        for (int j = 0; j < J; ++j) {
            const int u = v0 + 4 * i + (lr >> 2), k = (wave * J + j) * L::KG + L::EPL * lq;
            w[i][j] = make_uint4(0, 0, 0, 0);
            if (u < H && k < H) {
                const T* src = a.Wh + (int64_t(lr & 3) * H + u) * H + k;
                if ((H * int(sizeof(T))) % 16 == 0) {
                    w[i][j] = *reinterpret_cast<const uint4*>(src);
                } else {
                    T tmp[L::EPL];
#pragma unroll
                    for (int e = 0; e < L::EPL; ++e) tmp[e] = k + e < H ? src[e] : T(0);
                    __builtin_memcpy(&w[i][j], tmp, 16);
                }
            }
        }

    // cells: pair p = wave + 8 c, its lane's unit and row
    int cu[CPW], cr[CPW], cb[CPW];
    bool own[CPW], pad[CPW];   // own: a cell; pad: a zero column of the operand's last 16 bytes
    float creg[CPW];
    Gates<T> xg[CPW];
#pragma unroll
    for (int c = 0; c < CPW; ++c) {
        const int p = wave + 8 * c;
        cu[c] = v0 + 4 * (p % NT) + lq;
        cr[c] = row0 + 16 * (p / NT) + lr;
        own[c] = p < NP && cu[c] < H && cr[c] < a.B;
        pad[c] = p < NP && cu[c] >= H && cu[c] < kv && cr[c] < a.B;
        cb[c] = own[c] && a.perm ? a.perm[cr[c]] : cr[c];
        creg[c] = own[c] ? a.Cs[int64_t(cr[c]) * a.ldh + cu[c]] : 0.f;
    }
    // Gate rows of a step are addressed from the group's first row on, so that
    // their 32-bit offsets hold for any batch; only cells are loaded and stored.
    // (Sizes cut off at the step's last row cost 0.1 us a step.)
    const uint32_t gate_bytes = uint32_t(16 * RT) * uint32_t(a.ldg) * uint32_t(sizeof(T));
    const T* const xg_rows = a.XG + int64_t(row0) * a.ldg;
    T* const gs_rows = a.Gs + int64_t(row0) * a.ldg;
    auto gate_off = [&](int c) {
        return (uint32_t(cr[c] - row0) * uint32_t(a.ldg) + 4u * uint32_t(cu[c])) * uint32_t(sizeof(T));
    };
    auto prefetch = [&](int act, int64_t off) {
        const auto rs = make_rsrc(xg_rows + off * a.ldg, gate_bytes);
#pragma unroll
        for (int c = 0; c < CPW; ++c) xg[c].load(rs, own[c] && cr[c] < act ? gate_off(c) : kOutOfRange);
    };
    const int steps = a.steps[g];
    const int ntiles = a.groups * RT;
    const int64_t slot = int64_t(ntiles) * a.nkg * 64 * L::EPL;   // elements
    const uint32_t slot_bytes = uint32_t(slot * int64_t(sizeof(T)));
    // byte offsets in a slot: this lane's piece of k-group j, and its cells' results
    const uint32_t fo = uint32_t(((g * RT) * a.nkg + wave * J) * 64 + lane) * 16u;
    const uint32_t fstep = uint32_t(a.nkg) * 1024u;   // next row tile
    uint32_t so[CPW];
#pragma unroll
    for (int c = 0; c < CPW; ++c)
        so[c] = uint32_t(L::index(g * RT + (wave + 8 * c) / NT, a.nkg, lr, cu[c])) * uint32_t(sizeof(T));
    unsigned phase = 0;
    bool dead = false;
    // the schedule, carried: rows of steps t - 1, t and t + 1, packed offset of
    // step t; the row count of step t + 2 is loaded a step before it is needed
    int act_prev = 0, act = act_at(a.active, a.fixed, a.B, 0, a.t_eff);
    int act_next = act_at(a.active, a.fixed, a.B, 1, a.t_eff), act_raw = 0;
    int64_t off_t = 0;
    prefetch(act, 0);

    // a step's results, stored for later kernels while the next step's products
    // run: between a result's publication and the poll for the others' no store
    // and no load from memory is issued that the poll would have to wait for
    float hn[CPW];
    Gates<T> gs[CPW];
    uint32_t hw[CPW][2];   // bf16: h of the four units of lanes lr, lr + 16, ..
    auto store_results = [&](int t, int64_t off, int rows, int rows_next) {
        const int64_t nrow = int64_t(a.B) + off;
        const auto rgs = make_rsrc(gs_rows + off * a.ldg, gate_bytes);
#pragma unroll
        for (int c = 0; c < CPW; ++c) {
            if (!(own[c] && cr[c] < rows)) continue;
            const int u = cu[c], r = cr[c];
            a.Cs[(nrow + r) * a.ldh + u] = creg[c];
            gs[c].store(rgs, gate_off(c));
            T* ydst = a.y ? a.y + (int64_t(t) * a.B + cb[c]) * H + u : nullptr;
            if constexpr (L::EPL == 8) {
                if (lq == 0) {   // H is a multiple of 8, so the four units are cells
                    const uint2 v = make_uint2(hw[c][0], hw[c][1]);
                    if (a.Hs) *reinterpret_cast<uint2*>(a.Hs + (nrow + r) * a.ldh + u) = v;
                    if (ydst) *reinterpret_cast<uint2*>(ydst) = v;
                }
                if (a.HT) a.HT[int64_t(u) * a.ldht + nrow + r] = f2bf(hn[c]);
            } else {
                if (a.Hs) a.Hs[(nrow + r) * a.ldh + u] = hn[c];
                if (ydst) *ydst = hn[c];
            }
            if (r >= rows_next) {   // last step of this sequence
                if (a.hT) a.hT[int64_t(cb[c]) * H + u] = hn[c];
                if (a.cT) a.cT[int64_t(cb[c]) * H + u] = creg[c];
            }
        }
    };

    for (int t = 0; t < steps; ++t) {
        const bool more = t + 1 < steps;
        if (!local && t > 0) remote_barrier(a.sync, g, phase, unsigned(a.nu));
        f32x4_t acc[NP];
#pragma unroll
        for (int p = 0; p < NP; ++p) acc[p] = f32x4_t{0.f, 0.f, 0.f, 0.f};
        uint4 f[RT * J];
        {
            const auto rs = make_rsrc(a.ring + (t & 3) * slot, slot_bytes);
            load_operand<T>(f, rs, [&](int i) {
                const int rt = i / J, j = i % J;
                const bool ok = row0 + 16 * rt + lr < act && (wave * J + j) * L::KG + L::EPL * lq < kv;
                return ok ? fo + uint32_t(rt) * fstep + uint32_t(j) * 1024u : kOutOfRange;
            }, local, a.sync, dead);
        }
        // whatever this wave stored in the step before, the refill of its slot
        // pieces among it, is complete
        wait_own_stores();
        Gates<T> x4[CPW];
#pragma unroll
        for (int c = 0; c < CPW; ++c) x4[c] = xg[c];
        if (t > 0) act_next = __builtin_amdgcn_readfirstlane(act_raw);
#pragma unroll
        for (int j = 0; j < J; ++j)
#pragma unroll
            for (int rt = 0; rt < RT; ++rt)
#pragma unroll
                for (int i = 0; i < NT; ++i)
                    acc[rt * NT + i] = mma(w[i][j], f[rt * J + j], acc[rt * NT + i], static_cast<const T*>(nullptr));
        if (t > 0) store_results(t - 1, off_t - act_prev, act_prev, act);
        act_raw = t + 2 < a.t_eff ? a.B : 0;
        if (more) {
            prefetch(act_next, off_t + act);
            if (!a.fixed) act_raw = a.active[min(t + 2, a.t_eff)];
        }
        // sum over the waves, in wave order
        f32x4_t* buf = red + (C::DB ? (t & 1) * kWaves * NP * 64 : 0);
        if (!C::DB && t > 0) __syncthreads();   // the previous step's partial tiles have been read
#pragma unroll
        for (int p = 0; p < NP; ++p) buf[(wave * NP + p) * 64 + lane] = acc[p];
        __syncthreads();
        f32x4_t sum[CPW];
#pragma unroll
        for (int c = 0; c < CPW; ++c) {
            sum[c] = f32x4_t{0.f, 0.f, 0.f, 0.f};
            if (NP % kWaves == 0 || wave + 8 * c < NP) {
#pragma unroll
                for (int q = 0; q < kWaves; ++q) sum[c] += buf[(q * NP + wave + 8 * c) * 64 + lane];
            }
        }
#pragma unroll
        for (int c = 0; c < CPW; ++c) {
            float x[4], ga[4];
            x4[c].get(x);
            ga[0] = sigmoidf_(sum[c][0] + x[0]);
            ga[1] = sigmoidf_(sum[c][1] + x[1]);
            ga[2] = tanhf_(sum[c][2] + x[2]);
            ga[3] = sigmoidf_(sum[c][3] + x[3]);
            const bool cell = own[c] && cr[c] < act;
            const float cn = ga[1] * creg[c] + ga[0] * ga[2];
            creg[c] = cell ? cn : creg[c];
            hn[c] = cell ? ga[3] * tanhf_(cn) : 0.f;
            gs[c].set(ga);
        }
        // h_t for the next step: the only values the other members read
        {
            const auto rn = make_rsrc(a.ring + ((t + 1) & 3) * slot, slot_bytes);
            const auto rp = make_rsrc(a.ring + ((t + 3) & 3) * slot, slot_bytes);
#pragma unroll
            for (int c = 0; c < CPW; ++c) {
                if constexpr (L::EPL == 8) {
                    const uint32_t h1 = f2bf(hn[c]);
                    const uint32_t pr = h1 | (uint32_t(__shfl_xor(h1, 16)) << 16);
                    hw[c][0] = pr;
                    hw[c][1] = uint32_t(__shfl_xor(pr, 32));
                    const bool st = own[c] && lq == 0;
                    if (more && st && cr[c] < act_next) store_b64(rn, so[c], hw[c][0], not_empty(hw[c][1]));
                    if (local && t > 0 && st) store_b64(rp, so[c], kEmpty, kEmpty);
                } else {
                    const bool st = own[c] || pad[c];
                    if (more && st && cr[c] < act_next) store_b32(rn, so[c], not_empty(__float_as_uint(hn[c])));
                    if (local && t > 0 && st) store_b32(rp, so[c], kEmpty);
                }
            }
        }
        off_t += act;
        act_prev = act;
        act = act_next;
    }
    if (steps > 0) store_results(steps - 1, off_t - act_prev, act_prev, act);
}

// ---------------------------------------------------------------- backward
template <typename T>
struct BwdArgs {
    int H, B, t_eff, fixed;
    int rbase;
    int groups, nu, nkg;       // nkg: k-groups of the 4H interleaved gate columns
    int xccs;                  // XCDs the groups are dealt to (0: no group shares an L2)
    int gbase;                 // row groups of the earlier launches (rows of db_part)
    int steps[kMaxGroups];
    const int32_t* active;
    const int32_t* offsets;
    const int32_t* perm;
    const T* Wh;
    T* G;                      // dG row-major, interleaved, or NULL
    const T* Gs;
    const float* Cs;
    const T* dy;
    int64_t dy_ld;
    int dy_time;               // 1: dy row of (t, r) is t B + perm[r]; 0: the packed row
    const float* dhT;
    const float* dcT;
    float* dh0;
    float* dc0;
    float* db_part;            // [row group][4H] interleaved
    T* GT;                     // bf16 only: dG transposed, or NULL
    int64_t ldk;
    int64_t ldh, ldg;
    T* ring;
    Sync* sync;
};

template <int Q, int RT>
struct BwdCfg {
    static constexpr int U = 8 * Q;
    static constexpr int MT = (U + 15) / 16;         // 16-unit tiles
    static constexpr int NP = MT * RT;
    static constexpr int CPT = (NP * 256 + kThreads - 1) / kThreads;   // cells of a thread
    static constexpr int SMEM = 2 * kWaves * NP * 256 * 4;
};

template <typename T, int Q, int RT>
__global__ __launch_bounds__(kThreads) void lstm_bwd_xcd(BwdArgs<T> a) {
    using L = Lay<T>;
    using C = BwdCfg<Q, RT>;
    constexpr int J = 128 * Q / L::KG;    // k-groups of a wave
    constexpr int MT = C::MT, NP = C::NP, CPT = C::CPT;
    extern __shared__ __align__(16) unsigned char smem_raw[];
    f32x4_t* red = reinterpret_cast<f32x4_t*>(smem_raw);   // [buffer][wave][pair][64]
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const Place pl = take_place(a.sync, a.nu, a.groups, a.xccs);
    const int g = __builtin_amdgcn_readfirstlane(pl.g), m = __builtin_amdgcn_readfirstlane(pl.m);
    const bool local = __builtin_amdgcn_readfirstlane(pl.local) != 0;
    if (g < 0) return;
    const int H = a.H, v0 = m * C::U, row0 = a.rbase + 16 * RT * g;
    const int vend = min(H, v0 + C::U);
    const int lr = lane & 15, lq = lane >> 4;
    if (tid == 0 && m == 0) {
        __hip_atomic_fetch_add(&a.sync->groups, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (local) __hip_atomic_fetch_add(&a.sync->local_groups, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }

    // weights: Wh^T, rows = units v0 + 16 i + lr, k = interleaved gate columns
    uint4 w[MT][J];
    if constexpr (L::EPL == 8) {
        // Rows of Wh (one k each) hold the workgroup's U units in 2 U bytes: a
        // wave loads each k-group's 32 rows in 16-byte pieces, then turns them
        // through its part of the LDS.  Against 2-byte loads of each element
        // (8 times as many instructions): H 1024, time before the first step
        // 33 us less; H 656, 12 us less.
        constexpr int PR = C::U / 8, PIECES = 32 * PR, PPL = (PIECES + 63) / 64;   // pieces of a row, a k-group, a lane
        constexpr int LD = 16 * MT + 2;                                            // row pitch (elements)
        static_assert(32 * LD * 2 * kWaves <= C::SMEM, "a k-group per wave in LDS");
        uint32_t* sw = reinterpret_cast<uint32_t*>(smem_raw) + wave * 16 * LD;
        uint4 raw[J][PPL];
#pragma unroll
        for (int j = 0; j < J; ++j)
#pragma unroll
            for (int q = 0; q < PPL; ++q) {
                const int e = lane + 64 * q, k = (wave * J + j) * 32 + e / PR, u = v0 + 8 * (e % PR);
                const int uu = k >> 2, ga = k & 3;
                raw[j][q] = e < PIECES && u < vend && uu < H
                                ? *reinterpret_cast<const uint4*>(a.Wh + (int64_t(ga) * H + uu) * H + u)
                                : make_uint4(0, 0, 0, 0);
            }
#pragma unroll
        for (int j = 0; j < J; ++j) {
            __builtin_amdgcn_wave_barrier();
#pragma unroll
            for (int q = 0; q < PPL; ++q) {
                const int e = lane + 64 * q;
                if (e < PIECES) {
                    uint32_t* d = sw + ((e / PR) * LD + 8 * (e % PR)) / 2;
                    d[0] = raw[j][q].x;
                    d[1] = raw[j][q].y;
                    d[2] = raw[j][q].z;
                    d[3] = raw[j][q].w;
                }
            }
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            __builtin_amdgcn_wave_barrier();
            const bf16_t* sr = reinterpret_cast<const bf16_t*>(sw);
#pragma unroll
            for (int i = 0; i < MT; ++i) {
                bf16_t tmp[8];
#pragma unroll
                for (int e = 0; e < 8; ++e) tmp[e] = 16 * i + lr < C::U ? sr[(8 * lq + e) * LD + 16 * i + lr] : bf16_t(0);
                __builtin_memcpy(&w[i][j], tmp, 16);
            }
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        }
        __syncthreads();   // the sums over the waves use this LDS
    } else {
#pragma unroll
        for (int i = 0; i < MT; ++i)
#pragma unroll
            for (int j = 0; j < J; ++j) {
                const int u = v0 + 16 * i + lr, k = (wave * J + j) * L::KG + L::EPL * lq;
                T tmp[L::EPL];
#pragma unroll
                for (int e = 0; e < L::EPL; ++e) {
                    const int uu = (k + e) >> 2, ga = e & 3;
                    tmp[e] = (u < vend && uu < H) ? a.Wh[(int64_t(ga) * H + uu) * H + u] : T(0);
                }
                __builtin_memcpy(&w[i][j], tmp, 16);
            }
    }

    // cells: entry q = tid + 512 c of the pairs' 16 x 16 tiles
    int cu[CPT], cr[CPT], cb[CPT];
    bool own[CPT];
    float dhp[CPT], dcr[CPT], cnx[CPT], dbs[CPT][4];
    uint32_t so[CPT];
#pragma unroll
    for (int c = 0; c < CPT; ++c) {
        const int q = tid + kThreads * c, p = q >> 8, ln = (q & 255) >> 2;
        cu[c] = v0 + 16 * (p % MT) + 4 * (ln >> 4) + (q & 3);
        cr[c] = row0 + 16 * (p / MT) + (ln & 15);
        own[c] = p < NP && cu[c] < vend && cr[c] < a.B;
        cb[c] = own[c] && a.perm ? a.perm[cr[c]] : cr[c];
        dhp[c] = own[c] && a.dhT ? a.dhT[int64_t(cb[c]) * H + cu[c]] : 0.f;
        dcr[c] = own[c] && a.dcT ? a.dcT[int64_t(cb[c]) * H + cu[c]] : 0.f;
        cnx[c] = 0.f;
#pragma unroll
        for (int e = 0; e < 4; ++e) dbs[c][e] = 0.f;
        so[c] = uint32_t(L::index(g * RT + p / MT, a.nkg, ln & 15, 4 * cu[c])) * uint32_t(sizeof(T));
    }
    // gate rows from the group's first row on, as in the forward
    const uint32_t gate_bytes = uint32_t(16 * RT) * uint32_t(a.ldg) * uint32_t(sizeof(T));
    const T* const gs_rows = a.Gs + int64_t(row0) * a.ldg;
    T* const g_rows = a.G ? a.G + int64_t(row0) * a.ldg : nullptr;
    auto gate_off = [&](int c) {
        return (uint32_t(cr[c] - row0) * uint32_t(a.ldg) + 4u * uint32_t(cu[c])) * uint32_t(sizeof(T));
    };
    // operands of the cells that do not depend on dh, one step ahead
    Gates<T> gt_[CPT];
    float cpv[CPT], cnv[CPT], dyv[CPT];
    auto prefetch = [&](int t, int act, int act_next, int act_prev, int64_t off_t) {
        const int64_t prev_base = t == 0 ? 0 : int64_t(a.B) + off_t - act_prev;
        const auto rgs = make_rsrc(gs_rows + off_t * a.ldg, gate_bytes);
#pragma unroll
        for (int c = 0; c < CPT; ++c) {
            const bool cell = own[c] && cr[c] < act;
            gt_[c].load(rgs, cell ? gate_off(c) : kOutOfRange);
            cpv[c] = cell ? a.Cs[(prev_base + cr[c]) * a.ldh + cu[c]] : 0.f;
            // c_t is carried from the later step where the row ran there
            cnv[c] = cell && cr[c] >= act_next ? a.Cs[(a.B + off_t + cr[c]) * a.ldh + cu[c]] : 0.f;
            dyv[c] = 0.f;
            if (cell && a.dy) {
                const int64_t row = a.dy_time ? int64_t(t) * a.B + cb[c] : off_t + cr[c];
                dyv[c] = to_f(a.dy[row * a.dy_ld + cu[c]]);
            }
        }
    };
    const int steps = a.steps[g];
    const int64_t slot = int64_t(a.groups * RT) * a.nkg * 64 * L::EPL;
    const uint32_t slot_bytes = uint32_t(slot * int64_t(sizeof(T)));
    const uint32_t fo = uint32_t(((g * RT) * a.nkg + wave * J) * 64 + lane) * 16u;
    const uint32_t fstep = uint32_t(a.nkg) * 1024u;
    unsigned phase = 0;
    bool dead = false;
    // the schedule, carried: rows of steps t + 1, t, t - 1 (raw: loaded a step
    // before it is needed) and t - 2, packed offset of step t
    auto rows_at = [&](int t) { return act_at(a.active, a.fixed, a.B, t, a.t_eff); };
    int act_next = 0, act = steps > 0 ? rows_at(steps - 1) : a.B;
    int act_m1 = rows_at(steps - 2), act_m2 = rows_at(steps - 3);
    int64_t off_t = steps > 0 ? off_at(a.offsets, a.fixed, a.B, steps - 1) : 0;
    if (steps > 0) {
        act_next = rows_at(steps);
        prefetch(steps - 1, act, act_next, act_m1, off_t);
    } else {
        act_next = rows_at(0);
    }

    for (int t = steps - 1; t >= -1; --t) {
        const bool first = t == steps - 1;   // no later step: nothing to contract
        float dh[CPT];
#pragma unroll
        for (int c = 0; c < CPT; ++c) dh[c] = dhp[c];
        f32x4_t acc[NP];
        if (!first) {
            if (!local) remote_barrier(a.sync, g, phase, unsigned(a.nu));
#pragma unroll
            for (int p = 0; p < NP; ++p) acc[p] = f32x4_t{0.f, 0.f, 0.f, 0.f};
            const auto rs = make_rsrc(a.ring + ((t + 1) & 3) * slot, slot_bytes);
#pragma unroll
            for (int rt = 0; rt < RT; ++rt) {
                uint4 f[J];
                load_operand<T>(f, rs, [&](int j) {
                    const bool ok = row0 + 16 * rt + lr < act_next && (wave * J + j) * L::KG + L::EPL * lq < 4 * H;
                    return ok ? fo + uint32_t(rt) * fstep + uint32_t(j) * 1024u : kOutOfRange;
                }, local, a.sync, dead);
#pragma unroll
                for (int j = 0; j < J; ++j)
#pragma unroll
                    for (int i = 0; i < MT; ++i)
                        acc[rt * MT + i] = mma(w[i][j], f[j], acc[rt * MT + i], static_cast<const T*>(nullptr));
            }
        }
        // whatever this wave stored in the step before, the refill of its slot
        // pieces among it, is complete, and this step's operands are here
        wait_own_stores();
        Gates<T> g4[CPT];
        float cp[CPT], cl[CPT], dyc[CPT];
#pragma unroll
        for (int c = 0; c < CPT; ++c) {
            g4[c] = gt_[c];
            cp[c] = cpv[c];
            cl[c] = cnv[c];
            dyc[c] = dyv[c];
        }
        const int m2 = __builtin_amdgcn_readfirstlane(act_m2);
        if (t > 0) prefetch(t - 1, act_m1, act, m2, off_t - act_m1);
        act_m2 = t < 3 ? 0 : a.fixed ? a.B : a.active[t - 3];
        if (!first) {
            f32x4_t* buf = red + (t & 1) * kWaves * NP * 64;
#pragma unroll
            for (int p = 0; p < NP; ++p) buf[(wave * NP + p) * 64 + lane] = acc[p];
            __syncthreads();
            const float* bf = reinterpret_cast<const float*>(buf);
#pragma unroll
            for (int c = 0; c < CPT; ++c) {
                const int q = tid + kThreads * c;
                if ((NP * 256) % kThreads != 0 && q >= NP * 256) continue;
                float s = 0.f;
#pragma unroll
                for (int v = 0; v < kWaves; ++v) s += bf[v * NP * 256 + q];
                if (cr[c] < act_next) dh[c] = s;
            }
        }
        if (t < 0) {   // gradient of the initial state
#pragma unroll
            for (int c = 0; c < CPT; ++c)
                if (own[c]) {
                    if (a.dh0) a.dh0[int64_t(cb[c]) * H + cu[c]] = dh[c];
                    if (a.dc0) a.dc0[int64_t(cb[c]) * H + cu[c]] = dcr[c];
                }
            break;
        }
        Gates<T> dg[CPT];
#pragma unroll
        for (int c = 0; c < CPT; ++c) {
            const bool cell = own[c] && cr[c] < act;
            float ga[4];
            g4[c].get(ga);
            if (cell && cr[c] >= act_next) cnx[c] = cl[c];
            const float dhv = dh[c] + dyc[c];
            const float gi = ga[0], gf = ga[1], gg = ga[2], go = ga[3];
            const float tau = tanhf_(cnx[c]);
            const float d_o = dhv * tau;
            const float dct = dcr[c] + dhv * go * (1.f - tau * tau);
            const float d4[4] = {dct * gg * gi * (1.f - gi), dct * cp[c] * gf * (1.f - gf), dct * gi * (1.f - gg * gg),
                                 d_o * go * (1.f - go)};
            dg[c].set(d4);
            if (cell) {
                dcr[c] = dct * gf;
                cnx[c] = cp[c];
#pragma unroll
                for (int e = 0; e < 4; ++e) dbs[c][e] += d4[e];
            }
        }
        // dG_t for the next (earlier) step: the only values the other members read
        {
            const auto rn = make_rsrc(a.ring + (t & 3) * slot, slot_bytes);
            const auto rp = make_rsrc(a.ring + ((t + 2) & 3) * slot, slot_bytes);
#pragma unroll
            for (int c = 0; c < CPT; ++c) {
                if (own[c] && cr[c] < act) dg[c].publish(rn, so[c]);
                if (local && !first && own[c]) Gates<T>::clear(rp, so[c]);
            }
        }
#pragma unroll
        for (int c = 0; c < CPT; ++c) {
            if (!(own[c] && cr[c] < act)) continue;
            const int u = cu[c], r = cr[c];
            if (g_rows) {
                const auto rg = make_rsrc(g_rows + off_t * a.ldg, gate_bytes);
                dg[c].store(rg, gate_off(c));
            }
            if constexpr (L::EPL == 8) {
                if (a.GT) {
                    bf16_t* gt = a.GT + int64_t(4) * u * a.ldk + off_t + r;
                    gt[0] = bf16_t(dg[c].w.x & 0xffffu);
                    gt[a.ldk] = bf16_t(dg[c].w.x >> 16);
                    gt[2 * a.ldk] = bf16_t(dg[c].w.y & 0xffffu);
                    gt[3 * a.ldk] = bf16_t(dg[c].w.y >> 16);
                }
            }
        }
        act_next = act;
        act = t > 0 ? act_m1 : a.B;
        off_t -= act_m1;
        act_m1 = m2;
    }

    // bias gradient of this group's rows: per unit and gate, rows in order
    __syncthreads();
#pragma unroll
    for (int c = 0; c < CPT; ++c) {
        const int q = tid + kThreads * c;
        if (q < NP * 256) red[q] = f32x4_t{dbs[c][0], dbs[c][1], dbs[c][2], dbs[c][3]};
    }
    __syncthreads();
    if (tid < 4 * C::U && v0 + (tid >> 2) < vend) {
        const int ul = tid >> 2, ga = tid & 3;
        float s = 0.f;
        for (int rr = 0; rr < 16 * RT; ++rr) {
            const int p = (rr >> 4) * MT + (ul >> 4);
            const int ln = ((ul & 15) >> 2) * 16 + (rr & 15);
            s += red[p * 256 + ln * 4 + (ul & 3)][ga];
        }
        a.db_part[int64_t(a.gbase + g) * 4 * H + 4 * (v0 + ul) + ga] = s;
    }
}

}  // namespace xcd
}  // namespace janus
