// 4-bit streaming with the activations held in registers (gfx950): the decomposition of stream_direct.hpp with the format and
// arithmetic of stream_w4.hpp.
//
// A slot is one packed step: 16 rows x one group of 128 k, 1024 bytes of codes and the rows' 16 step sizes.  A wave holds
// its K slice of all tokens as matrix operands (four per slot and 16 tokens; at M <= 8 two full loads, see
// stream_direct.hpp) and, per slot and token block, the group's offset -136 * (sum of the group's activations) that takes the
// codes' bias out of the accumulator.  The offset is itself a matrix product - with an A operand of -136 everywhere it lands in
// every row of the accumulator, exactly where the group's sum starts from.
//
// What bounds it: per byte of weights twice the activations and conversions of the 8-bit kernel, so the activations' fetch
// and, over many tiles, instruction issue.  Back to back, HBM-cold, us a launch, staged -> this:
//     M = 8:  4096 x 4096 8.1 -> 5.1, 12288 x 4096 11.3 -> 9.0, 4096 x 12288 15.4 -> 9.9, 151936 x 4096 59.5 -> 55
//     M = 16: 10.5 -> 5.8, 13.4 -> 10.0, 24.1 -> 18.4, 88.2 -> 57;  M = 32: 19.5 -> 7.1, 26.7 -> 11.2, 151936 x 4096 232 -> 66
// Longer shares of K: linears in stream_outer.hpp (plan_w4_outer), argmax and other launch shapes in the staged kernel.
#pragma once

#include "launch.hpp"
#include "stream_w4.hpp"

namespace quasar {

// LDS: [a region per wave: activations on their way in, then 2 x NB partial tiles of 1 KB]
template <int MP, int EPI, int XS>
__global__ __launch_bounds__(w4_waves(MP, XS) * 64) void stream_direct_w4_kernel(const GemmParams p) {
    extern __shared__ __align__(16) unsigned char lds[];
    constexpr int NW = w4_waves(MP, XS);
    constexpr int NB = (MP == 32) ? 2 : 1;
    constexpr int XP = (MP == 8) ? 2 : 4;           // operand registers (of 8 k a lane) per slot and token block
    constexpr int U = XS >= 3 ? 1 : 4 / XS;         // tiles per round
    constexpr int RD = XS * U <= 4 ? XS * U : (XS % 4 == 0 ? 4 : (XS % 3 == 0 ? 3 : XS));
    static_assert((XS * U) % RD == 0, "a round is whole turns of the ring");

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int g = lane >> 4, mcol = lane & 15;
    const int b = blockIdx.x;
    using Share = TileShare<1, deal_tiles(FMT_W4, MP, NW, XS, EPI == EPI_ARGMAX), EPI == EPI_ARGMAX>;
    loaded_together<Share>(p, p.x, p.ldx, p.w, p.M, p.S);
    const Share share(p, b);
    const int ntiles = share.units;

    const int first = (p.S * w) / NW;
    const int n = (p.S * (w + 1)) / NW - first;
    int step[XS];
#pragma unroll
    for (int i = 0; i < XS; ++i) step[i] = i < n ? first + i : min(first, p.S - 1);

    // ---- activations: slot i, operand j holds k = 128 step + 32 j + 8 g .. of the lane's token; at M <= 8 register j holds
    // operands 2 j (columns 0 .. 7) and 2 j + 1 (columns 8 .. 15)
    constexpr int kPass = w4_pass(MP, XS);
    constexpr int region = w4_region_bytes(MP, XS) / NW;
    unsigned char *own = lds + w * region;
    const int tok = (MP == 8) ? (mcol & 7) : mcol;
    const int half = (MP == 8) ? (mcol >> 3) : 0;
    u32x4 xr[XS][NB * XP];
    // through LDS in whole cache lines, as in stream_direct.hpp
    auto fetch_x = [&](int at) {
        fetch_rows<MP, 256>(p.x, p.ldx, p.M, first + at, p.S - 1, min(kPass, XS - at), lds_address_of(lds) + (unsigned int)(w * region), lane);
    };
    auto read_x = [&](int at) {
#pragma unroll
        for (int i = 0; i < kPass; ++i)
            if (at + i < XS)
#pragma unroll
                for (int nb = 0; nb < NB; ++nb)
#pragma unroll
                    for (int j = 0; j < XP; ++j) {
                        const int t = tok + 16 * nb;
                        const int c = MP == 8 ? 4 * (2 * j + half) + g : 4 * j + g;
                        xr[at + i][nb * XP + j] = *reinterpret_cast<const u32x4 *>(own + row_piece<MP, 256>(t, i, c, min(kPass, XS - at)));
                    }
    };
    if constexpr (kPass > 0) {
        fetch_x(0);
    } else {
        const uint16_t *row = p.x + (long long)min(tok, p.M - 1) * p.ldx + 32 * half + 8 * g;
#pragma unroll
        for (int i = 0; i < XS; ++i)
#pragma unroll
            for (int j = 0; j < XP; ++j) xr[i][j] = *reinterpret_cast<const u32x4 *>(row + 128 * step[i] + (MP == 8 ? 64 : 32) * j);
    }

    // ---- weight ring: codes and the rows' step sizes of a slot
    const unsigned long long wbase = reinterpret_cast<unsigned long long>(p.w);
    const unsigned int tile_bytes = (unsigned int)p.S * (unsigned int)kStepBytes4;
    u32x4 ring[RD];
    u32x2 scl[RD];
    auto refill = [&](int d, int tl, int i) {
        const bool real = tl < ntiles;
        const unsigned long long a = real ? wbase + (unsigned long long)(unsigned int)share.tile(tl) * tile_bytes + (unsigned int)step[i] * (unsigned int)kStepBytes4
                                          : reinterpret_cast<unsigned long long>(p.x);
        unsigned int oc = real ? 16u * lane : 0u, os = real ? 1024u + 8u * g : 0u;
        ring[d] = ring_refill_at(a, oc, ring[d]);
        scl[d] = ring_refill2_at(a, os, scl[d]);
    };
#pragma unroll
    for (int d = 0; d < RD; ++d) {
        ring[d] = u32x4{0u, 0u, 0u, 0u};
        scl[d] = u32x2{0u, 0u};
        refill(d, d / XS, d % XS);
    }
    if constexpr (kPass > 0) {
        // (the direct-to-LDS loads are older than the ring's and loads return in order; only this wave reads them)
        asm volatile("s_waitcnt vmcnt(%0)" ::"n"(2 * RD) : "memory");
        read_x(0);
#pragma unroll
        for (int at = kPass; at < XS; at += kPass) {
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
            fetch_x(at);
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
            read_x(at);
        }
    }
    // two slots of 8 tokens: the rotated operands are kept, eight instructions a slot and tile less (25600 x 4096, M = 5 13.5 us, 13.1 so;
    // forms of more slots have no registers for them)
    constexpr bool KEEP = MP == 8 && XS == 2;
    [[maybe_unused]] u32x4 xrot[XS][XP];
    if constexpr (KEEP)
#pragma unroll
        for (int i = 0; i < XS; ++i)
#pragma unroll
            for (int j = 0; j < XP; ++j) {
                xrot[i][j] = rotate_half_row(xr[i][j]);
                asm volatile("" : "+v"(xrot[i][j].x), "+v"(xrot[i][j].y), "+v"(xrot[i][j].z), "+v"(xrot[i][j].w));
            }
    auto operand = [&](int i, int nb, int j) {          // operand j (0 .. 3) of slot i
        if constexpr (KEEP) {
            return __builtin_bit_cast(bf16x8, (j & 1) ? xrot[i][j >> 1] : xr[i][j >> 1]);
        } else if constexpr (MP == 8) {
            const u32x4 v = xr[i][j >> 1];
            return __builtin_bit_cast(bf16x8, (j & 1) ? rotate_half_row(v) : v);
        } else {
            return __builtin_bit_cast(bf16x8, xr[i][nb * XP + j]);
        }
    };
    // group offsets: every row of A is -136 (bf16 0xC308), so every row of the product is the token's offset
    float gofs[XS][NB];
    {
        const u32x4 k136 = {0xC308C308u, 0xC308C308u, 0xC308C308u, 0xC308C308u};
#pragma unroll
        for (int i = 0; i < XS; ++i)
#pragma unroll
            for (int nb = 0; nb < NB; ++nb) {
                f32x4 o = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    o = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, k136), operand(i, nb, j), o, 0, 0, 0);
                gofs[i][nb] = o.x;
            }
    }

    f32x4 acc[NB];
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) acc[nb] = f32x4{0.f, 0.f, 0.f, 0.f};
    float bestv[NB];
    unsigned int besti[NB];
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) { bestv[nb] = -__builtin_inff(); besti[nb] = 0x7FFFFFFFu; }
    int parity = 0;
    unsigned int nib_mask, nib_magic;
    w4_constants(nib_mask, nib_magic);

    auto slot = [&](int d, int i) {
        const unsigned int wd[4] = {ring[d].x, ring[d].y, ring[d].z, ring[d].w};
        f32x4 grp[NB];
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) grp[nb] = f32x4{gofs[i][nb], gofs[i][nb], gofs[i][nb], gofs[i][nb]};
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const bf16x8 a = w4_to_bf16x8(wd[j], nib_mask, nib_magic);
#pragma unroll
            for (int nb = 0; nb < NB; ++nb) grp[nb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, operand(i, nb, j), grp[nb], 0, 0, 0);
        }
        const float s0 = __uint_as_float(scl[d].x << 16), s1 = __uint_as_float(scl[d].x & 0xFFFF0000u);
        const float s2 = __uint_as_float(scl[d].y << 16), s3 = __uint_as_float(scl[d].y & 0xFFFF0000u);
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) {
            acc[nb].x = __builtin_fmaf(s0, grp[nb].x, acc[nb].x);
            acc[nb].y = __builtin_fmaf(s1, grp[nb].y, acc[nb].y);
            acc[nb].z = __builtin_fmaf(s2, grp[nb].z, acc[nb].z);
            acc[nb].w = __builtin_fmaf(s3, grp[nb].w, acc[nb].w);
        }
    };
    // tile end: cross-wave sum through LDS, fixed order, eight partial tiles requested together: left to itself the compiler read one after
    // the other in most forms, 16 trips to LDS at every tile (us: 25600 x 2176, M = 1 11.4 so, 10.2 now; 25600 x 1024, M = 16 9.7, 8.4).
    // Forms of more slots have no registers for eight (12288 x 4096 at M = 32, four slots: 10.8, 13.0 with them)
    constexpr bool TOGETHER = XS <= (MP == 8 ? 4 : 3);
    auto tile_end = [&](int tl) {
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) {
            *reinterpret_cast<f32x4 *>(own + ((parity * NB + nb) * 64 + lane) * 16) = acc[nb];
            acc[nb] = f32x4{0.f, 0.f, 0.f, 0.f};
        }
        lds_barrier();
        if (w == (tl % NW)) {
            f32x4 rsum[NB];
#pragma unroll
            for (int nb = 0; nb < NB; ++nb) {
                const unsigned char *st = lds + ((parity * NB + nb) * 64 + lane) * 16;
                rsum[nb] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll 1
                for (int w0 = 0; w0 < NW; w0 += 8) {           // (a loop: bounds the registers of the reads in flight)
                    if constexpr (TOGETHER) {
                        f32x4 v[8];
#pragma unroll
                        for (int j = 0; j < 8; ++j) v[j] = *reinterpret_cast<const f32x4 *>(st + (w0 + j) * region);
                        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                        for (int j = 0; j < 8; ++j) rsum[nb] += v[j];
                    } else {
#pragma unroll
                        for (int ww = w0; ww < w0 + 8; ++ww) rsum[nb] += *reinterpret_cast<const f32x4 *>(st + ww * region);
                    }
                }
            }
            const u32x2 none[NB] = {};
            finish_tile<true, EPI, false, NB>(p, rsum, share.tile(tl), nullptr, none, nullptr, 0, lane, bestv, besti);
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
                if (i < n && (U == 1 || tl < ntiles)) slot(j % RD, i);
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

template <int MP, int EPI, int... XS>
int launch_w4_forms(int xs, int grid, int lds_bytes, hipStream_t stream, const GemmParams &p) {
    int rc = QUASAR_ERR_SHAPE;
    ((xs == XS ? (void)(rc = launch(stream_direct_w4_kernel<MP, EPI, XS>, grid, w4_waves(MP, XS) * 64, lds_bytes, stream, p)) : (void)0), ...);
    return rc;
}
template <int EPI>
int launch_w4_as(const GemmParams &p, int MP, const DirectPlan &d, hipStream_t stream) {
    if (MP == 8) return launch_w4_forms<8, EPI, 1, 2, 3, 4, 6>(d.XS, d.groups, d.lds_bytes, stream, p);
    if (MP == 16) return launch_w4_forms<16, EPI, 1, 2, 3, 4, 12>(d.XS, d.groups, d.lds_bytes, stream, p);
    return launch_w4_forms<32, EPI, 1, 2, 3, 4, 5>(d.XS, d.groups, d.lds_bytes, stream, p);
}

}  // namespace quasar
