// W8A8 streaming with the activation codes held in registers (gfx950): the decomposition of stream_direct.hpp with the
// arithmetic of stream_w8a8.hpp.
//
// A wave quantises only the K slice it multiplies: it loads its slice of x, takes the per-token maxima of the smoothed
// values, meets the other waves once (a maximum does not depend on the order, so the step sizes are those of the
// stand-alone quantiser bit for bit), and turns its values into the int8 operand registers it keeps: four a slot and 16
// tokens.  The staged kernel (stream_w8a8.hpp) made every thread scan and quantise for all waves, through LDS and two more
// barriers, and remains for slices that do not fit.
//
// What bounds it: the quantiser's vector instructions (about eight per element and workgroup, 1.3 us at M = 8, K = 4096)
// while the first weights are on their way; then the weight stream.  Back to back, HBM-cold, us a launch, staged -> this:
//     M = 8:  4096 x 4096 11.8 -> 6.4, 12288 x 4096 17.2 -> 10.4, 4096 x 12288 28.4 -> 17.9 (12 slots: every workgroup
//             quantises 98304 values; 20.7 with x gathered);  M = 16: 17.8 -> 8.4, 23.1 -> 11.9, 45.2 -> 29.3;  M = 32: 31.6 -> 21.5,
//             36.0 -> 27.6.  Linears of large M x K with a workspace: stream_outer.hpp (4096 x 4096, M = 32 10.1)
#pragma once

#include "launch.hpp"
#include "stream_w8a8.hpp"

namespace quasar {

// Four codes from four smoothed values: clamp(rint(x~ * inv)), the rounding made by an addition that leaves the integer in
// the low bits (products are within +-127 after the clamp).  The median of three takes the least operand that is a number if
// one is not: NaN becomes -127 as in quantize_piece.
__device__ __forceinline__ unsigned int quantize_quad(float x0, float x1, float x2, float x3, float inv) {
    constexpr float kRound = 12582912.0f;       // 1.5 x 2^23
    const unsigned int u0 = __float_as_uint(__builtin_amdgcn_fmed3f(x0 * inv, -127.f, 127.f) + kRound);
    const unsigned int u1 = __float_as_uint(__builtin_amdgcn_fmed3f(x1 * inv, -127.f, 127.f) + kRound);
    const unsigned int u2 = __float_as_uint(__builtin_amdgcn_fmed3f(x2 * inv, -127.f, 127.f) + kRound);
    const unsigned int u3 = __float_as_uint(__builtin_amdgcn_fmed3f(x3 * inv, -127.f, 127.f) + kRound);
    const unsigned int lo = __builtin_amdgcn_perm(u1, u0, 0x0c0c0400u), hi = __builtin_amdgcn_perm(u3, u2, 0x0c0c0400u);
    return lo | (hi << 16);
}

// A slot is 64 k of one tile: one 1 KB load, one v_mfma_i32_16x16x64_i8 per 16 tokens.
// LDS: [a region per wave: activations on their way in, then 2 x NB partial tiles of 1 KB][row scales][16 x MP maxima]
//      [smoothing factors: 16 waves x XS x 256 B]
// PREQ: p.x is the operand codes that quantize_operand_kernel made (at 32 tokens), p.dx their step sizes; nothing is quantised here.
template <int MP, int EPI, int XS, bool SMOOTH, bool PREQ = false>
__global__ __launch_bounds__(1024) void stream_direct_a8_kernel(const GemmParams p) {
    extern __shared__ __align__(16) unsigned char lds[];
    constexpr int NW = 16;
    constexpr int NB = (MP == 32) ? 2 : 1;
    constexpr int XP = (MP == 8) ? 1 : 2;           // 8-value pieces per lane, slot and token block
    constexpr int U = XS >= 4 ? 1 : 4 / XS;
    constexpr int RD = XS * U <= 6 ? XS * U : (XS == 10 ? 5 : (XS == 8 && MP == 8 ? 8 : 4));
    static_assert((XS * U) % RD == 0, "a round is whole turns of the ring");
    constexpr bool HOLD = a8_hold(MP, XS);
    static_assert(!PREQ || (MP == 32 && !SMOOTH && !HOLD), "operand codes are read where nothing else of x is");

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int g = lane >> 4, mcol = lane & 15;
    const int b = blockIdx.x;
    using Share = TileShare<1, deal_tiles(FMT_A8, MP, NW, XS, EPI == EPI_ARGMAX), EPI == EPI_ARGMAX>;
    loaded_together<Share>(p, p.x, p.ldx, p.w, p.scales, p.M, p.S, p.smooth, p.dx, p.sc_bytes);
    const Share share(p, b);
    const int ntiles = share.units;

    constexpr int kPass = a8_pass(MP, XS);
    constexpr int region = a8_region_bytes(MP, XS) / NW;
    unsigned char *own = lds + w * region;
    uint16_t *sc_lds = reinterpret_cast<uint16_t *>(lds + NW * region);              // [tiles][16]
    float *maxima = reinterpret_cast<float *>(lds + NW * region + p.sc_bytes);       // [NW][MP]
    const unsigned int sm_ofs = (unsigned int)(NW * region + p.sc_bytes + NW * MP * 4 + w * (XS * 256));

    const int first = (p.S * w) / NW;
    const int n = (p.S * (w + 1)) / NW - first;
    const int last = n > 0 ? first + n - 1 : first;     // (slots beyond the share repeat its last step)
    int step[XS];
#pragma unroll
    for (int i = 0; i < XS; ++i) step[i] = min(first + i, last);

    // ---- requests: smoothing factors (each wave's own, into LDS), activations, row scales, weight ring
    if constexpr (SMOOTH) {
        const unsigned int base = lds_address_of(lds) + sm_ofs;
#pragma unroll
        for (int j = 0; j < (XS + 3) / 4; ++j) {
            const int i = 4 * j + (lane >> 4);
            const int st = min(first + i, last);
            if (4 * j + 3 < XS || i < XS)
                load_to_lds_16(reinterpret_cast<unsigned long long>(p.smooth), (unsigned int)st * 256u + 16u * (lane & 15), base + 1024 * j);
        }
    }
    const int tok = (MP == 8) ? (mcol & 7) : mcol;
    const int half8 = (MP == 8) ? (mcol >> 3) : 0;
    const uint16_t *xrow[NB];
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) xrow[nb] = p.x + (long long)min(tok + 16 * nb, p.M - 1) * p.ldx + 16 * g + 8 * half8;
    auto load_x = [&](int i, int j) { return *reinterpret_cast<const u32x4 *>(xrow[j / XP] + 64 * step[i] + 8 * (j % XP)); };
    u32x4 raw[HOLD ? XS : 1][NB * XP];
    static_assert(HOLD || kPass == 0, "activations that are read twice come straight from memory");
    // through LDS in whole cache lines, as in stream_direct.hpp
    [[maybe_unused]] auto fetch_x = [&](int at) {
        fetch_rows<MP, 128>(p.x, p.ldx, p.M, first + at, last, min(kPass, XS - at), lds_address_of(lds) + (unsigned int)(w * region), lane);
    };
    [[maybe_unused]] auto read_x = [&](int at) {
#pragma unroll
        for (int i = 0; i < kPass; ++i)
            if (at + i < XS)
#pragma unroll
                for (int j = 0; j < NB * XP; ++j) {
                    const int t = tok + 16 * (j / XP), c = 2 * g + half8 + j % XP;
                    raw[HOLD ? at + i : 0][j] = *reinterpret_cast<const u32x4 *>(own + row_piece<MP, 128>(t, i, c, min(kPass, XS - at)));
                }
    };
    if constexpr (kPass > 0) fetch_x(0);
    else if constexpr (HOLD)
#pragma unroll
        for (int i = 0; i < XS; ++i)
#pragma unroll
            for (int j = 0; j < NB * XP; ++j) raw[i][j] = load_x(i, j);
    i32x4 bq[XS][NB];
    if constexpr (PREQ)
#pragma unroll
        for (int i = 0; i < XS; ++i)
#pragma unroll
            for (int nb = 0; nb < NB; ++nb)
                bq[i][nb] = *(reinterpret_cast<const i32x4 *>(p.x) + ((long long)step[i] * NB + nb) * 64 + lane);
    unsigned int sc_first = 0;
    if (2 * tid < ntiles * kTileRows)
        sc_first = *reinterpret_cast<const unsigned int *>(p.scales + (long long)share.tile(tid >> 3) * kTileRows + 2 * (tid & 7));

    const unsigned long long wbase = reinterpret_cast<unsigned long long>(p.w);
    const unsigned int tile_bytes = (unsigned int)p.S * (unsigned int)kStepBytes;
    u32x4 ring[RD];
    auto refill = [&](int d, int tl, int i) {
        const bool real = tl < ntiles;
        const unsigned long long a = real ? wbase + (unsigned long long)(unsigned int)share.tile(tl) * tile_bytes + (unsigned int)step[i] * (unsigned int)kStepBytes
                                          : reinterpret_cast<unsigned long long>(p.x);
        unsigned int off = real ? 16u * lane : 0u;
        ring[d] = ring_refill_at(a, off, ring[d]);
    };
#pragma unroll
    for (int d = 0; d < RD; ++d) {
        ring[d] = u32x4{0u, 0u, 0u, 0u};
        refill(d, d / XS, d % XS);
    }
    if (2 * tid < ntiles * kTileRows) reinterpret_cast<unsigned int *>(sc_lds)[tid] = sc_first;
    for (int i = 2 * (tid + NW * 64); i < ntiles * kTileRows; i += 2 * NW * 64)
        reinterpret_cast<unsigned int *>(sc_lds)[i >> 1] =
            *reinterpret_cast<const unsigned int *>(p.scales + (long long)share.tile(i >> 4) * kTileRows + (i & 15));
    // (the loads into LDS are older than the ring's and loads return in order)
    if constexpr (SMOOTH || kPass > 0) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(RD) : "memory");
    if constexpr (kPass > 0) {
        read_x(0);
#pragma unroll
        for (int at = kPass; at < XS; at += kPass) {
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
            fetch_x(at);
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
            read_x(at);
        }
    }

    // the eight smoothed values of piece j of slot i
    auto smoothed = [&](const u32x4 &v, int i, int j, float (&xt)[8]) {
        smooth_piece(v, nullptr, 0, xt);
        if constexpr (SMOOTH) {
            const f32x4 *s = reinterpret_cast<const f32x4 *>(lds + sm_ofs + i * 256 + g * 64 + (half8 + j % XP) * 32);
            const f32x4 s0 = s[0], s1 = s[1];
            xt[0] = xt[0] * s0.x; xt[1] = xt[1] * s0.y; xt[2] = xt[2] * s0.z; xt[3] = xt[3] * s0.w;
            xt[4] = xt[4] * s1.x; xt[5] = xt[5] * s1.y; xt[6] = xt[6] * s1.z; xt[7] = xt[7] * s1.w;
        }
    };

    float dx[NB];
    if constexpr (PREQ) {
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) dx[nb] = p.dx[tok + 16 * nb];
    } else {
    // ---- per-token maxima over the whole K, step sizes
    // KEEP: the smoothed values stay in registers between the maximum and the codes where there are at most 32 a lane, instead of being
    // unpacked and smoothed again (16 of 70 vector instructions of eight values; us, again, kept: 12288 x 4096 M = 8 10.60, 10.44,
    // 4096 x 2048 M = 16 5.77, 5.57, 1024 x 1024 M = 16 4.27, 4.14)
    constexpr bool KEEP = SMOOTH && HOLD && XS * XP <= 4;
    [[maybe_unused]] float kept[KEEP ? XS : 1][NB * XP][8];
    float amax[NB];
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) amax[nb] = 0.f;
#pragma unroll
    for (int i = 0; i < XS; ++i)
#pragma unroll
        for (int j = 0; j < NB * XP; ++j) {
            float xt[8];
            u32x4 v;
            if constexpr (HOLD) v = raw[i][j];
            else v = load_x(i, j);
            smoothed(v, i, j, xt);
            if constexpr (KEEP)
#pragma unroll
                for (int e = 0; e < 8; ++e) kept[i][j][e] = xt[e];
            const float a = piece_amax(xt);
            amax[j / XP] = fmaxf(amax[j / XP], a);      // (slots beyond the share repeat its last step)
            if (!HOLD && (i * NB * XP + j) % 8 == 7) __builtin_amdgcn_sched_barrier(0);     // (bounds the registers of the pass)
        }
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) {
        float a = n > 0 ? amax[nb] : 0.f;
        a = fmaxf(a, __shfl_xor(a, 16, 64));
        a = fmaxf(a, __shfl_xor(a, 32, 64));
        if constexpr (MP == 8) a = fmaxf(a, __shfl_xor(a, 8, 64));
        if (lane < (MP == 8 ? 8 : 16)) maxima[w * MP + lane + 16 * nb] = a;
    }
    lds_barrier();
    float inv[NB];
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) {
        float a = 0.f;
#pragma unroll
        for (int ww = 0; ww < NW; ++ww) a = fmaxf(a, maxima[ww * MP + tok + 16 * nb]);
        dx[nb] = step_of(a);
        inv[nb] = inverse_step_of(a);
    }
#pragma unroll
    for (int i = 0; i < XS; ++i)
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) {
            unsigned int o[4];
#pragma unroll
            for (int q = 0; q < XP; ++q) {
                float xt[8];
                if constexpr (KEEP) {
#pragma unroll
                    for (int e = 0; e < 8; ++e) xt[e] = kept[i][nb * XP + q][e];
                } else {
                    u32x4 v;
                    if constexpr (HOLD) v = raw[i][nb * XP + q];
                    else v = load_x(i, nb * XP + q);
                    smoothed(v, i, nb * XP + q, xt);
                }
                o[2 * q] = quantize_quad(xt[0], xt[1], xt[2], xt[3], inv[nb]);
                o[2 * q + 1] = quantize_quad(xt[4], xt[5], xt[6], xt[7], inv[nb]);
            }
            if constexpr (MP == 8) {
                // the other eight k of the token are in the lane eight columns on
                o[2] = (unsigned int)__builtin_amdgcn_update_dpp(0, (int)o[0], 0x128, 0xf, 0xf, true);
                o[3] = (unsigned int)__builtin_amdgcn_update_dpp(0, (int)o[1], 0x128, 0xf, 0xf, true);
            }
            bq[i][nb] = i32x4{(int)o[0], (int)o[1], (int)o[2], (int)o[3]};
            if (HOLD ? XS >= 6 : (i * NB + nb) % 2 == 1) __builtin_amdgcn_sched_barrier(0);
        }
    }

    i32x4 acc[NB];
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) acc[nb] = i32x4{0, 0, 0, 0};
    float bestv[NB];
    unsigned int besti[NB];
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) { bestv[nb] = -__builtin_inff(); besti[nb] = 0x7FFFFFFFu; }
    int parity = 0;

    // tile end: exact integer sum over the waves, Eq. 10 as fp32(acc) * (dx * dw), each one fp32 operation
    auto tile_end = [&](int tl) {
        const int at = (parity * NB * 64 + lane) * 16;
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) {
            *reinterpret_cast<i32x4 *>(own + at + nb * 1024) = acc[nb];
            acc[nb] = i32x4{0, 0, 0, 0};
        }
        lds_barrier();
        if (w == (tl % NW)) {
            const int n0 = share.tile(tl) * kTileRows + 4 * g;
            const u32x2 sb = *reinterpret_cast<const u32x2 *>(sc_lds + tl * kTileRows + 4 * g);
            const float dw0 = bf16_bits_to_float(sb.x & 0xFFFFu), dw1 = bf16_bits_to_float(sb.x >> 16);
            const float dw2 = bf16_bits_to_float(sb.y & 0xFFFFu), dw3 = bf16_bits_to_float(sb.y >> 16);
#pragma unroll
            for (int nb = 0; nb < NB; ++nb) {
                i32x4 r = {0, 0, 0, 0};
#pragma unroll 1
                for (int w0 = 0; w0 < NW; w0 += 8)             // (a loop: bounds the registers of the reads in flight)
#pragma unroll
                    for (int ww = w0; ww < w0 + 8; ++ww) r += *reinterpret_cast<const i32x4 *>(lds + ww * region + at + nb * 1024);
                const int m = mcol + 16 * nb;
                const float dxm = dx[nb];
                const float v0 = (float)r.x * (dxm * dw0), v1 = (float)r.y * (dxm * dw1);
                const float v2 = (float)r.z * (dxm * dw2), v3 = (float)r.w * (dxm * dw3);
                if constexpr (EPI == EPI_LINEAR) {
                    if (m < p.M) {
                        u32x2 o;
                        o.x = float_to_bf16_bits(v0) | (float_to_bf16_bits(v1) << 16);
                        o.y = float_to_bf16_bits(v2) | (float_to_bf16_bits(v3) << 16);
                        *reinterpret_cast<u32x2 *>(p.y + m * p.ldy + n0) = o;
                    }
                } else {
                    // strictly greater keeps the lowest index inside a lane
                    if (v0 > bestv[nb]) { bestv[nb] = v0; besti[nb] = n0; }
                    if (v1 > bestv[nb]) { bestv[nb] = v1; besti[nb] = n0 + 1; }
                    if (v2 > bestv[nb]) { bestv[nb] = v2; besti[nb] = n0 + 2; }
                    if (v3 > bestv[nb]) { bestv[nb] = v3; besti[nb] = n0 + 3; }
                }
            }
        }
        parity ^= 1;
    };
    auto round = [&](int tl0, auto last) {
        constexpr bool kLast = decltype(last)::value;
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int tl = tl0 + u;
#pragma unroll
            for (int i = 0; i < XS; ++i) {
                const int j = u * XS + i, jn = j + RD;
                if (i < n && (U == 1 || tl < ntiles)) {
#pragma unroll
                    for (int nb = 0; nb < NB; ++nb)
                        acc[nb] = __builtin_amdgcn_mfma_i32_16x16x64_i8(__builtin_bit_cast(i32x4, ring[j % RD]), bq[i][nb], acc[nb], 0, 0, 0);
                }
                if (!kLast || jn < U * XS) refill(j % RD, tl0 + (jn / (U * XS)) * U + (jn % (U * XS)) / XS, jn % XS);
            }
            if (U == 1 || tl < ntiles) tile_end(tl);
        }
    };
    int tl0 = 0;
    for (; tl0 + U < ntiles; tl0 += U) round(tl0, std::false_type{});
    round(tl0, std::true_type{});

    if constexpr (EPI == EPI_ARGMAX) publish_argmax<MP, NB, NW>(bestv, besti, lds, p.partial + (long long)b * MP);
}

// ---- dispatch over the built forms ----

template <int MP, int EPI, bool SMOOTH, int... XS>
int launch_a8_forms(int xs, int grid, int lds_bytes, hipStream_t stream, const GemmParams &p) {
    int rc = QUASAR_ERR_SHAPE;
    ((xs == XS ? (void)(rc = launch(stream_direct_a8_kernel<MP, EPI, XS, SMOOTH>, grid, 1024, lds_bytes, stream, p)) : (void)0), ...);
    return rc;
}
template <int... XS>
int launch_a8_codes(int xs, int grid, int lds_bytes, hipStream_t stream, const GemmParams &p) {
    int rc = QUASAR_ERR_SHAPE;
    ((xs == XS ? (void)(rc = launch(stream_direct_a8_kernel<32, EPI_ARGMAX, XS, false, true>, grid, 1024, lds_bytes, stream, p)) : (void)0), ...);
    return rc;
}
template <int EPI, bool SMOOTH>
int launch_a8_as(const GemmParams &p, int MP, const DirectPlan &d, hipStream_t stream) {
    if (MP == 8) return launch_a8_forms<8, EPI, SMOOTH, 1, 2, 3, 4, 5, 6, 8, 10, 12>(d.XS, d.groups, d.lds_bytes, stream, p);
    if (MP == 16) return launch_a8_forms<16, EPI, SMOOTH, 1, 2, 3, 4, 5, 6, 8, 10, 12>(d.XS, d.groups, d.lds_bytes, stream, p);
    if constexpr (SMOOTH) return launch_a8_forms<32, EPI, SMOOTH, 1, 2, 3, 4, 5>(d.XS, d.groups, d.lds_bytes, stream, p);
    else return launch_a8_forms<32, EPI, SMOOTH, 1, 2, 3, 4, 5, 6, 8>(d.XS, d.groups, d.lds_bytes, stream, p);
}

}  // namespace quasar
