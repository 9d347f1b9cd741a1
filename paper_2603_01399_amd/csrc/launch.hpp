// Launch helpers shared by the translation units of the library.
#pragma once

#include "../../include/quasar.h"

#include <hip/hip_runtime.h>

#include <mutex>
#include <utility>
#include <vector>

#include "stream_gemm.hpp"

namespace quasar {

constexpr int kMaxLds = 160 * 1024;          // gfx950 LDS per compute unit

// Kernels that use more than the default dynamic LDS limit need a one-time opt-in per
// function (and per device); remember which ones have had it.
inline bool allow_large_lds(const void *fn) {
    static std::mutex mu;
    static std::vector<std::pair<const void *, int>> done;
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess) return false;
    std::lock_guard<std::mutex> lock(mu);
    for (const auto &e : done)
        if (e.first == fn && e.second == dev) return true;
    if (hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, kMaxLds) != hipSuccess) return false;
    done.emplace_back(fn, dev);
    return true;
}

template <typename KernelT>
int launch(KernelT kernel, int grid, int block, int lds_bytes, hipStream_t stream, const GemmParams &p) {
    if (lds_bytes > kMaxLds) return QUASAR_ERR_SHAPE;
    if (!allow_large_lds(reinterpret_cast<const void *>(kernel))) return QUASAR_ERR_HIP;
    hipLaunchKernelGGL(kernel, dim3(grid), dim3(block), lds_bytes, stream, p);
    return hipGetLastError() == hipSuccess ? QUASAR_OK : QUASAR_ERR_HIP;
}

// ---- the kernel that holds the activations in registers (stream_direct.hpp) ----

// Waves of a workgroup by form (XS slots of 64 k per wave): where the activations take more than about half of a wave's
// 128 registers, eight waves of 256 - the ring, the accumulators and the addresses are then paid for half as often.
constexpr int direct_waves(int MP, int XS) { return MP == 32 || (MP == 16 && XS > 8) ? 8 : 16; }

// Slots of activations that pass through a wave's LDS region at a time (0: straight into registers).  Up to 64 KB of x a
// workgroup the gather of 16-byte pieces is as fast; beyond that the direct-to-LDS path, whose instructions read whole
// cache lines, is: 6.0 -> 5.5 us for 4096 x 3072 at M = 16, 7.6 -> 7.1 for 4096 x 6144 at M = 8.  128 KB a workgroup at most.
constexpr int direct_pass(int MP, int XS) {
    if (MP == 8 && XS <= 4) return 0;
    const int fit = 1024 / (direct_waves(MP, XS) * MP);
    return XS < fit ? XS : fit;
}
// LDS of the waves' regions (C chunks of partial tiles, two tiles' worth)
constexpr int direct_region_bytes(int MP, int XS, int C) {
    const int x = direct_pass(MP, XS) * MP * 128, tiles = 2 * C * (MP == 32 ? 2 : 1) * 1024;
    return direct_waves(MP, XS) * (x > tiles ? x : tiles);
}

struct DirectPlan {
    int XS, SC, C, ksplit, slice_steps, groups, sc_bytes, lds_bytes;
};

// p: as for the other kernels (its step counts are replaced by slots of 64 k).  epi, pre, resid: EPI_*, PRE_* and whether a
// residual is added.
int launch_direct_int8(int epi, int pre, bool resid, const GemmParams &p, int MP, const DirectPlan &d, hipStream_t stream);
int launch_direct_bf16(int epi, const GemmParams &p, int MP, const DirectPlan &d, hipStream_t stream);

int launch_direct_w8a8(int epi, const GemmParams &p, int MP, const DirectPlan &d, hipStream_t stream);

inline int launch_direct(bool w16, int epi, int pre, bool resid, const GemmParams &p, int MP, const DirectPlan &d, hipStream_t stream) {
    return w16 ? launch_direct_bf16(epi, p, MP, d, stream) : launch_direct_int8(epi, pre, resid, p, MP, d, stream);
}

}  // namespace quasar
