// What every .hip translation unit needs: the HIP error macro, small constants, dynamic LDS of a kernel.
// Everything has internal linkage.
#pragma once

#include <hip/hip_runtime.h>

#include <mutex>
#include <utility>
#include <vector>

#include "ivfpq_internal.hpp"

#define HIP_TRY(expr)                                                                               \
    do {                                                                                            \
        hipError_t e_ = (expr);                                                                     \
        if (e_ != hipSuccess)                                                                       \
            return ivfpq::fail(IVFPQ_EHIP, "%s failed: %s (%s:%d)", #expr, hipGetErrorString(e_), __FILE__, __LINE__); \
    } while (0)

namespace {

using ivfpq::fail;

constexpr int kWave = 64;
constexpr size_t kLdsBytes = 160 * 1024;       // LDS of one gfx950 compute unit
constexpr size_t kAlign = 256;

inline size_t align_up(size_t x, size_t a = kAlign) { return (x + a - 1) / a * a; }

// Lets `kernel` use dynamic LDS up to the whole compute unit's; done once per kernel and device, so
// that later launches make no call besides the launch itself (a caller may be capturing a HIP graph).
inline int allow_full_lds_ptr(const void* kernel) {
    static std::mutex mu;
    static std::vector<std::pair<const void*, int>> done;
    int dev = 0;
    HIP_TRY(hipGetDevice(&dev));
    std::lock_guard<std::mutex> lock(mu);
    for (const auto& e : done)
        if (e.first == kernel && e.second == dev) return IVFPQ_OK;
    HIP_TRY(hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)kLdsBytes));
    done.emplace_back(kernel, dev);
    return IVFPQ_OK;
}
template <class Kernel>
int allow_full_lds(Kernel kernel) { return allow_full_lds_ptr(reinterpret_cast<const void*>(kernel)); }

// The scan kernels address their tables by LDS offsets counted from 0: their dynamic LDS must be the first
// thing in the workgroup's LDS, which holds when the compiled kernel has no static LDS.  Checked once per
// kernel (hipFuncGetAttributes is not a stream operation; later launches make no call besides the launch).
inline int require_no_static_lds(const void* kernel) {
    static std::mutex mu;
    static std::vector<const void*> ok;
    std::lock_guard<std::mutex> lock(mu);
    for (const void* k : ok)
        if (k == kernel) return IVFPQ_OK;
    hipFuncAttributes attr;
    HIP_TRY(hipFuncGetAttributes(&attr, kernel));
    if (attr.sharedSizeBytes != 0)
        return fail(IVFPQ_EUNSUPPORTED, "internal: a scan kernel was built with %zu bytes of static LDS", (size_t)attr.sharedSizeBytes);
    ok.push_back(kernel);
    return IVFPQ_OK;
}

}  // namespace
