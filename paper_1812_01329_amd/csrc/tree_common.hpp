// Shared pieces of the persistent tree programs (binary TreeLSTM, TreeRNN,
// Child-Sum TreeLSTM): the counter block of a launch and the host-side launch
// of a grid whose workgroups must all be resident.
#pragma once

#include <mutex>

#include "device.hpp"
#include "lstm_persist.hpp"
#include "runtime.hpp"

namespace janus {
namespace tpersist {

constexpr int kMaxE = 512;    // widest input row of the persistent Child-Sum

// Counter block of a launch.  `error` comes first: the backward zeroes the
// counters that follow it and leaves a flag the forward set.
struct TreeSync {
    unsigned error;
    unsigned pad_e[63];
    unsigned census[16][64];    // workgroups that have arrived on each XCD
    unsigned group[64][64];     // arrivals of each tree group's workgroups (groups that share no L2)
};
constexpr size_t kTreeSyncCounters = offsetof(TreeSync, census);   // byte offset of the counters

// ------------------------------------------------------------ host side
struct TreeDev {
    int cus = 0;
    size_t lds = 0;
    int xccs = 0;
};
// Properties of the current device, queried once per device under a lock.
inline TreeDev tree_dev() {
    static std::mutex m;
    static TreeDev cache[64];
    static bool have[64] = {};
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return TreeDev{};
    std::lock_guard<std::mutex> lock(m);
    if (!have[dev]) {
        TreeDev t;
        int v = 0;
        if (hipDeviceGetAttribute(&v, hipDeviceAttributeMultiprocessorCount, dev) == hipSuccess) t.cus = v;
        if (hipDeviceGetAttribute(&v, hipDeviceAttributeMaxSharedMemoryPerBlock, dev) == hipSuccess) t.lds = size_t(v);
        if (hipDeviceGetAttribute(&v, hipDeviceAttributeNumberOfXccs, dev) == hipSuccess) t.xccs = v;
        (void)hipGetLastError();
        cache[dev] = t;
        have[dev] = true;
    }
    return cache[dev];
}

// An ordinary launch of a grid whose workgroups must all be resident (the
// plan allows one per CU and no more than the CUs; the occupancy query
// confirms one fits a CU).  The barrier's waits are bounded.
template <class K, class A>
inline janus_status tree_persistent_launch(K kernel, int blocks, size_t smem, const A& args, hipStream_t st,
                                           size_t& attr_smem, int threads) {
    static std::mutex m;
    {
        std::lock_guard<std::mutex> lock(m);
        if (smem > attr_smem) {
            JANUS_HIP(hipFuncSetAttribute(reinterpret_cast<const void*>(kernel),
                                          hipFuncAttributeMaxDynamicSharedMemorySize, int(smem)));
            attr_smem = smem;
        }
    }
    int per_cu = 0;
    JANUS_HIP(hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, reinterpret_cast<const void*>(kernel),
                                                           threads, smem));
    if (per_cu < 1 || int64_t(per_cu) * tree_dev().cus < blocks) return JANUS_ERR_UNSUPPORTED;
    void* argv[] = {const_cast<A*>(&args)};
    return resident_launch(reinterpret_cast<const void*>(kernel), blocks, threads, smem, argv, st, tree_dev().cus);
}

}  // namespace tpersist
}  // namespace janus
