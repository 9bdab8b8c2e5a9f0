// launch.cpp -- grid sizing shared by every launcher.
#include "launch.hpp"

#include <hip/hip_runtime.h>

#include <mutex>
#include <unordered_map>

namespace sdp4 {

namespace {
struct Device {
    int cus = 0, lds_per_cu = 0, lds_per_block = 0;
};
std::mutex g_mu;
Device g_dev[64];
std::unordered_map<const void *, int> g_static_lds; // kernel -> its own LDS bytes

hipError_t current_device(Device &d)
{
    int dev = 0;
    hipError_t err = hipGetDevice(&dev);
    if (err != hipSuccess)
        return err;
    std::lock_guard<std::mutex> lk(g_mu);
    if (dev < 64 && g_dev[dev].cus) {
        d = g_dev[dev];
        return hipSuccess;
    }
    const struct { hipDeviceAttribute_t attr; int *value; } want[] = {
        {hipDeviceAttributeMultiprocessorCount, &d.cus},
        {hipDeviceAttributeMaxSharedMemoryPerMultiprocessor, &d.lds_per_cu},
        {hipDeviceAttributeMaxSharedMemoryPerBlock, &d.lds_per_block},
    };
    for (const auto &w : want) {
        err = hipDeviceGetAttribute(w.value, w.attr, dev);
        if (err != hipSuccess)
            return err;
    }
    if (dev < 64)
        g_dev[dev] = d;
    return hipSuccess;
}

// LDS to reserve so that k blocks of `kernel` fit a compute unit and one more does not.
size_t reserve_lds(const void *kernel, int k, const Device &d, hipError_t &err)
{
    std::lock_guard<std::mutex> lk(g_mu);
    auto it = g_static_lds.find(kernel);
    if (it == g_static_lds.end()) {
        hipFuncAttributes a;
        err = hipFuncGetAttributes(&a, kernel);
        if (err != hipSuccess)
            return 0;
        it = g_static_lds.emplace(kernel, (int)a.sharedSizeBytes).first;
    }
    // each takes lds / k less a margin of one allocation granule or so
    int64_t each = d.lds_per_cu / k - 1024;
    if (each > d.lds_per_block) // a block cannot hold more: residency is then bounded by the block limit
        each = d.lds_per_block;
    const int64_t dyn = each - it->second;
    return dyn > 0 ? (size_t)dyn : 0;
}
} // namespace

LaunchShape shape_for(const void *kernel, int64_t nwork_blocks, int cap, hipError_t &err)
{
    err = hipSuccess;
    if (nwork_blocks < 1)
        nwork_blocks = 1;
    size_t dyn = 0;
    if (cap != kUncapped) {
        Device d;
        err = current_device(d);
        if (err != hipSuccess)
            return {};
        if (cap == kPersistent)
            nwork_blocks = nwork_blocks < d.cus ? nwork_blocks : d.cus;
        else if (nwork_blocks > (int64_t)kPacedBlocks * d.cus)
            dyn = reserve_lds(kernel, cap, d, err);
    }
    if (nwork_blocks <= kGridX)
        return {(unsigned)nwork_blocks, 1, dyn};
    return {(unsigned)kGridX, (unsigned)((nwork_blocks + kGridX - 1) / kGridX), dyn};
}

} // namespace sdp4
