// W8A8 forms of the streaming kernel with K outermost, and the quantiser that makes their activation operands.
#include "stream_outer.hpp"
#include "stream_direct_a8.hpp"

namespace quasar {

// x[M, K] bf16 -> int8 codes as the matrix instruction's B operands, [step of 64 k][16 tokens][g 4][token][16 k] (at most 8
// tokens: [step][g][8 tokens][16 k]), and the step sizes dx[M].  The arithmetic is that of the kernels that quantise for
// themselves, so the codes are the same bits.  One workgroup a token: what bounds it is the chain of a launch, one trip to x,
// the meeting for the maximum and the stores; pieces beyond the 32768 k that the registers hold are read again.
template <bool SMOOTH>
static __global__ __launch_bounds__(1024) void quantize_operand_kernel(const uint16_t *x, long long ldx, int K, const float *smooth,
                                                                       int MP, unsigned char *codes, float *dx) {
    constexpr int HOLD = 4;
    __shared__ float red[16];
    const int m = blockIdx.x, tid = threadIdx.x, pieces = K / 8;
    const uint16_t *row = x + (long long)m * ldx;
    u32x4 raw[HOLD];
    f32x4 sm[HOLD][2];
    auto load = [&](int j, int p8) {
        raw[j] = u32x4{0u, 0u, 0u, 0u};
        if (p8 < pieces) {
            raw[j] = *reinterpret_cast<const u32x4 *>(row + 8ll * p8);
            if constexpr (SMOOTH) {
                sm[j][0] = *reinterpret_cast<const f32x4 *>(smooth + 8ll * p8);
                sm[j][1] = *reinterpret_cast<const f32x4 *>(smooth + 8ll * p8 + 4);
            }
        }
    };
    auto smoothed = [&](int j, float (&xt)[8]) {
        smooth_piece(raw[j], nullptr, 0, xt);
        if constexpr (SMOOTH) {
            xt[0] = xt[0] * sm[j][0].x; xt[1] = xt[1] * sm[j][0].y; xt[2] = xt[2] * sm[j][0].z; xt[3] = xt[3] * sm[j][0].w;
            xt[4] = xt[4] * sm[j][1].x; xt[5] = xt[5] * sm[j][1].y; xt[6] = xt[6] * sm[j][1].z; xt[7] = xt[7] * sm[j][1].w;
        }
    };
    float amax = 0.f;
    for (int base = ((pieces - 1) / (1024 * HOLD)) * 1024 * HOLD; base >= 0; base -= 1024 * HOLD) {      // (the first ones last: they stay)
#pragma unroll
        for (int j = 0; j < HOLD; ++j) load(j, base + 1024 * j + tid);
#pragma unroll
        for (int j = 0; j < HOLD; ++j)
            if (base + 1024 * j + tid < pieces) {
                float xt[8];
                smoothed(j, xt);
                amax = fmaxf(amax, piece_amax(xt));
            }
    }
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) amax = fmaxf(amax, __shfl_xor(amax, off, 64));
    if ((tid & 63) == 0) red[tid >> 6] = amax;
    __syncthreads();
#pragma unroll
    for (int i = 0; i < 16; ++i) amax = fmaxf(amax, red[i]);
    const float inv = inverse_step_of(amax);
    if (tid == 0) dx[m] = step_of(amax);
    for (int base = 0; base < pieces; base += 1024 * HOLD) {
        if (base > 0)
#pragma unroll
            for (int j = 0; j < HOLD; ++j) load(j, base + 1024 * j + tid);
#pragma unroll
        for (int j = 0; j < HOLD; ++j) {
            const int p8 = base + 1024 * j + tid;
            if (p8 < pieces) {
                float xt[8];
                smoothed(j, xt);
                const int step = p8 >> 3, g = (p8 & 7) >> 1;
                const long long at = MP == 8 ? ((long long)step * 4 + g) * 8 + m
                                             : (((long long)step * (MP / 16) + (m >> 4)) * 4 + g) * 16 + (m & 15);
                *reinterpret_cast<u32x2 *>(codes + 16 * at + 8 * (p8 & 1)) =
                    u32x2{quantize_quad(xt[0], xt[1], xt[2], xt[3], inv), quantize_quad(xt[4], xt[5], xt[6], xt[7], inv)};
            }
        }
    }
}

// codes: at least K / 64 * (MP == 8 ? 512 : 64 * MP) bytes; dx: M floats
int launch_quantize_operand(const GemmParams &p, int MP, unsigned char *codes, float *dx, hipStream_t stream) {
    if (p.smooth)
        hipLaunchKernelGGL(quantize_operand_kernel<true>, dim3(p.M), dim3(1024), 0, stream, p.x, p.ldx, p.K, p.smooth, MP, codes, dx);
    else
        hipLaunchKernelGGL(quantize_operand_kernel<false>, dim3(p.M), dim3(1024), 0, stream, p.x, p.ldx, p.K, p.smooth, MP, codes, dx);
    return hipGetLastError() == hipSuccess ? QUASAR_OK : QUASAR_ERR_HIP;
}

int launch_outer_w8a8(const GemmParams &p, int MP, const DirectPlan &d, hipStream_t stream) { return launch_outer_as<FMT_A8>(p, MP, d, stream); }

}  // namespace quasar
