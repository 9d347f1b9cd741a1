// RMSNorm as a launch of its own (gfx950): in front of the linears whose fused form would spill or scan too much.
#pragma once

#include "stream_gemm.hpp"

namespace quasar {

// y[m, k] = bf16( gamma[k] * bf16( x[m, k] * rsqrt(mean_k x[m, :]^2 + eps) ) ), the roundings of the fused forms; y [M, K] dense.
// One workgroup a token: launch-sized (2.6 us), bounded by one trip to x, the meeting for the row sum and the stores.  Pieces
// beyond the 32768 k that the registers hold are read again.
[[maybe_unused]] static __global__ __launch_bounds__(1024) void rmsnorm_rows_kernel(const uint16_t *x, long long ldx, int K, const uint16_t *gamma,
                                                                                    float eps, uint16_t *y) {
    constexpr int HOLD = 4;
    __shared__ float red[16];
    const int m = blockIdx.x, tid = threadIdx.x, pieces = K / 8;
    const uint16_t *row = x + (long long)m * ldx;
    u32x4 raw[HOLD], gm[HOLD];
    auto load = [&](int j, int p8) {
        raw[j] = u32x4{0u, 0u, 0u, 0u};
        if (p8 < pieces) {
            raw[j] = *reinterpret_cast<const u32x4 *>(row + 8ll * p8);
            gm[j] = *reinterpret_cast<const u32x4 *>(gamma + 8ll * p8);
        }
    };
    float ss = 0.f;
    for (int base = ((pieces - 1) / (1024 * HOLD)) * 1024 * HOLD; base >= 0; base -= 1024 * HOLD) {      // (the first ones last: they stay)
#pragma unroll
        for (int j = 0; j < HOLD; ++j) load(j, base + 1024 * j + tid);
#pragma unroll
        for (int j = 0; j < HOLD; ++j) ss += piece_sumsq(raw[j]);
    }
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) ss += __shfl_xor(ss, off, 64);
    if ((tid & 63) == 0) red[tid >> 6] = ss;
    __syncthreads();
    float tot = 0.f;
#pragma unroll
    for (int i = 0; i < 16; ++i) tot += red[i];
    const float r = __fdiv_rn(1.0f, __fsqrt_rn(__fdiv_rn(tot, (float)K) + eps));
    for (int base = 0; base < pieces; base += 1024 * HOLD) {
        if (base > 0)
#pragma unroll
            for (int j = 0; j < HOLD; ++j) load(j, base + 1024 * j + tid);
#pragma unroll
        for (int j = 0; j < HOLD; ++j) {
            const int p8 = base + 1024 * j + tid;
            if (p8 < pieces) *reinterpret_cast<u32x4 *>(y + (long long)m * K + 8ll * p8) = pre_rmsnorm_piece(raw[j], gm[j], r);
        }
    }
}

}  // namespace quasar
