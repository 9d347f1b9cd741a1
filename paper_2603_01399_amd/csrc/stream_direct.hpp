// Skinny-M weight streaming with the activations held in registers (gfx950).
//
// The 16 waves of a workgroup split K, so a wave meets the same activations at every weight tile: its K slice of all
// M tokens.  That slice is M x K / 16 values - at M = 8, K = 4096 sixteen registers a lane - and this kernel loads it
// once into the matrix instruction's B operand registers: no staging for the workgroup and no barrier in front of the
// stream, no LDS reads in the main loop; the weight loads are requested in the same breath as the activations.  The kernel that stages x in LDS (stream_gemm.hpp) remains for shapes whose slice
// does not fit the registers.
//
// At M <= 8 half of the B operand's 16 columns have no token.  A slot's 64 k of a token are two operands of 32; lanes
// of columns 0 .. 7 load the first and lanes of columns 8 .. 15 the second, one full 1 KB load a slot, and the second
// operand is the same register rotated by eight lanes (the unused columns multiply rubbish that nobody reads).
//
// What bounds it: a launch whose compute units read nothing but the 16 MB of a 4096 x 4096 matrix takes 3.9 us back to
// back (48 MB: 8.6 us); the rest is the fetch of x (as many bytes per compute unit as its weights at M = 8) and the
// tile end.  Back to back, HBM-cold, int8, us a launch, staged kernel -> this one:
//     M = 8:  1024 x 1024 5.1 -> 3.2, 4096 x 4096 7.2 -> 5.3, 12288 x 4096 11.7 -> 10.0, 4096 x 12288 13.9 -> 11.1
//     M = 16: 4096 x 4096 9.4 -> 6.5, 12288 x 4096 14.8 -> 11.3, 4096 x 8192 14.3 -> 9.9
//     M = 32: 4096 x 4096 13.0 -> 7.9, 12288 x 4096 22.9 -> 12.5
// Fetching x: straight into the registers, or, for more of it, in whole cache lines through the wave's own piece of LDS
// (direct_pass).  Weights requested before x: 0.4 us slower; workgroups that start at different K slices, rows of x at
// other strides: no difference.
#pragma once

#include "launch.hpp"

namespace quasar {

// Slots in flight per wave: a compute unit accepts about 32 KB of outstanding loads, so three or four 1 KB loads in
// each of 16 waves keep it full; up to eight where the registers allow.
constexpr int direct_ring(int MP, int slots) {
    return slots <= 7 ? slots : (slots == 8 ? (MP == 16 ? 4 : 8) : (slots % 5 == 0 ? 5 : (slots == 24 ? 6 : 4)));
}

// A slot is 64 k: one 1 KB load of int8 codes or two of bf16 weights.
// XS: slots of a tile a wave may have (its activations are held in XS x (MP == 8 ? 4 : MP / 2) registers).
// CH: the bits of the kernels that stage x, whose order of the sum is one of 16 waves.  Up to 16 tokens: K is summed in p.C
//     chunks, each reduced over the waves by itself and added in chunk order.  32 tokens (PAIR): a wave of the eight takes two
//     neighbouring shares of sixteen of each chunk, CH slots each, and hands over the sum of the two, which is what that order adds
//     first; slots of bf16 weights are 32 k there, as the shares are.  The chunks are XS / (2 CH), as many as p.C; slots that a
//     share does not have read one line and are not multiplied.  0: one sum a wave.
// 32 tokens in chunks, V = 151936, staged -> so: int8 K = 4096 255 -> 109 us, K = 5120 314 -> 190; bf16 K = 4096 290 -> 196, K = 5120 359 -> 256
// LDS: [a region per wave: activations on their way in, then 2 x C x NB partial tiles of 1 KB][row scales][kept gate tile (EPI_SWIGLU)][16 x MP sums (PRE)]
template <int MP, bool W16, int EPI, int XS, int CH = 0, int PRE = PRE_NONE, bool RES = false>
__global__ __launch_bounds__(direct_waves(MP, XS) * 64) void stream_direct_kernel(const GemmParams p0) {
    extern __shared__ __align__(16) unsigned char lds[];
    constexpr int NW = direct_waves(MP, XS);
    constexpr int NB = (MP == 32) ? 2 : 1;          // 16-token blocks
    constexpr bool PAIR = CH > 0 && MP == 32;
    constexpr int CC = PAIR ? XS / (2 * CH) : 1;    // chunks of the pair form
    constexpr int PARS = CC > 4 ? 1 : 2;            // sets of partial tiles (five chunks: two sets do not fit the LDS)
    constexpr int KS = PAIR && W16 ? 32 : 64;       // k of a slot
    constexpr int XP = (MP == 8 || KS == 32) ? 1 : 2;   // loads of x per slot and token block
    constexpr int WL = W16 && KS == 64 ? 2 : 1;     // weight loads per slot
    constexpr int U = KS == 32 ? (XS >= 6 ? 1 : 2) : (XS >= 4 ? 1 : 4 / XS);    // tiles per round: at least four slots in flight
    constexpr int RD = KS == 32 ? (CC == 1 ? XS * U : (XS == 12 ? 6 : (XS == 20 ? 10 : 8))) : direct_ring(MP, XS * U);                  // ring depth in slots
    static_assert((XS * U) % RD == 0, "a round is whole turns of the ring");
    constexpr int kSlotBytes = WL * kStepBytes;

    constexpr int TU = EPI == EPI_SWIGLU ? 2 : 1;   // tiles are handed out in units of TU
    using Share = TileShare<TU, EPI != EPI_LOGITS && deal_tiles(W16 ? FMT_BF16 : FMT_INT8, MP, NW, PAIR ? XS * KS / 64 : XS, EPI == EPI_ARGMAX),
                            EPI == EPI_ARGMAX || EPI == EPI_LOGITS>;
    const int slice = blockIdx.x, b = blockIdx.y;
    GemmParams p = p0;
    loaded_together<Share>(p, p.x, p.ldx, p.w, p.scales, p.M, p.S, p.Srow, p.slice_steps, CH ? p.SC : p.sc_bytes);
    const int s0 = slice * p0.slice_steps;          // (all step counts here are in slots of 64 k)
    p.S = min(p0.slice_steps, p0.S - s0);
    p.w = p0.w + (long long)s0 * (64 * WL);
    p.x = p0.x + (long long)s0 * 64;
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int g = lane >> 4, mcol = lane & 15;

    const Share share(p, b);
    const int ntiles = TU * share.units;
    const int C = PAIR ? CC : (CH ? p.C : 1);

    // per wave: [2][C][NB][64] partial tiles, over the activations' way into the registers
    // (bf16 weights keep the gather at four slots, where LDS is as fast or faster call after call in a graph - 168 shapes of K 3328 to 4096
    // 0.99 on average, 1024 x 4096 M = 8 6.2 -> 5.6 us - but slower eagerly up to five tokens: 4096 x 4096 M = 1 7.53, 7.69, M = 5 7.85,
    // 7.95; seven linears of an 8B layer, M = 5 79.1, 79.6)
    constexpr int kPass = (KS == 32 && CC > 1) || (W16 && MP == 8 && XS == 4) ? 0 : direct_pass(MP, XS);
    static_assert(KS == 64 || CC > 1 || XS / 2 + 1 <= kPass, "slots of 32 k come in one pass of whole lines");
    const int region = max(kPass * MP * 128, PARS * C * NB * 1024);
    unsigned char *own = lds + w * region;
    uint16_t *sc_lds = reinterpret_cast<uint16_t *>(lds + NW * region);                // [tiles][16]
    [[maybe_unused]] f32x4 *gate_keep = reinterpret_cast<f32x4 *>(lds + NW * region + p.sc_bytes - NB * 1024);

    // ---- the wave's slots: slot i of a tile is step[i] of it.  Chunk c covers steps c * SC .., wave w takes the w-th of
    // 16 shares of each.  Slots beyond the wave's last step repeat its first: their loads hit lines it has just
    // requested, and they are not multiplied.
    int n = 0, first = 0, bound0 = 0;
    int step[XS];
    [[maybe_unused]] unsigned int have = 0;         // PAIR: the slots that carry a step
    if constexpr (PAIR) {
#pragma unroll
        for (int c = 0; c < CC; ++c) {
            const int scc = CC == 1 ? p.S : min(p.SC, p.S - c * p.SC);
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const int lo = (scc * (2 * w + h)) / 16, count = (scc * (2 * w + h + 1)) / 16 - lo;
                if (c == 0 && h == 0) first = lo;
#pragma unroll
                for (int j = 0; j < CH; ++j) {
                    const int i = (2 * c + h) * CH + j;
                    if (j < count) have |= 1u << i;
                    step[i] = j < count ? (CC == 1 ? lo : c * p.SC + lo) + j : min(first, p.S - 1);
                }
            }
        }
    } else if constexpr (CH) {
        int c = 0, at = 0, left = 0;
        first = (min(p.SC, p.S) * w) / NW;
#pragma unroll
        for (int i = 0; i < XS; ++i) {
            if (left == 0 && c < C) {
                const int scc = min(p.SC, p.S - c * p.SC);
                at = c * p.SC + (scc * w) / NW;
                left = (scc * (w + 1)) / NW - (scc * w) / NW;     // >= 1: chunks have at least 16 steps
                if (c == 0) bound0 = left;
                ++c;
            }
            step[i] = left > 0 ? at : first;
            if (left > 0) { ++n; ++at; --left; }
        }
    } else {
        first = (p.S * w) / NW;
        n = (p.S * (w + 1)) / NW - first;
#pragma unroll
        for (int i = 0; i < XS; ++i) step[i] = i < n ? first + i : min(first, p.S - 1);
    }

    // ---- requests: activations, row scales, weight ring
    const int tok = (MP == 8) ? (mcol & 7) : mcol;
    u32x4 xr[XS][NB * XP];
    const int kofs = W16 ? 8 * g + ((MP == 8) ? 32 * (mcol >> 3) : 0) : 16 * g + ((MP == 8) ? 8 * (mcol >> 3) : 0);
    const uint16_t *xrow[NB];
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) xrow[nb] = p.x + (long long)min(tok + 16 * nb, p.M - 1) * p.ldx + kofs;
    auto load_x = [&](int i) {
#pragma unroll
        for (int nb = 0; nb < NB; ++nb)
#pragma unroll
            for (int q = 0; q < XP; ++q)
                xr[i][nb * XP + q] = *reinterpret_cast<const u32x4 *>(xrow[nb] + KS * step[i] + (W16 ? 32 : 8) * q);
    };
    // through LDS: slots at .. at + kPass - 1, each instruction 128 bytes of eight tokens' rows, piece c of token t at
    // position c ^ (t & 7) of its 128 bytes (the lanes that read one column of pieces meet different banks)
    constexpr bool RANGE = CH == 0 && KS == 64;      // the wave's slots are one range of K: fetch_rows
    [[maybe_unused]] auto fetch_x = [&](int at) {
        const unsigned int base = lds_address_of(lds) + (unsigned int)(w * region);
        const unsigned long long xa = reinterpret_cast<unsigned long long>(p.x);
        if constexpr (RANGE) {
            fetch_rows<MP, 128>(p.x, p.ldx, p.M, first + at, p.S - 1, min(kPass, XS - at), base, lane);
            return;
        }
#pragma unroll
        for (int t8 = 0; t8 < MP / 8; ++t8) {
            const int t = (lane >> 3) + 8 * t8;
            const unsigned int off = (unsigned int)min(t, p.M - 1) * (unsigned int)(2 * p.ldx) + (unsigned int)(((lane & 7) ^ (t & 7)) * 16);
#pragma unroll
            for (int i = 0; i < kPass; ++i) {
                // (slots of 32 k: the lines of 64 that hold them)
                const int s64 = KS == 64 ? step[min(at + i, XS - 1)] : min((min(first, p.S - 1) >> 1) + i, (p.S - 1) >> 1);
                if (KS == 64 ? at + i < XS : i <= XS / 2)
                    load_to_lds_16(xa + 128ull * (unsigned int)s64, off, base + (i * (MP / 8) + t8) * 1024);
            }
        }
    };
    [[maybe_unused]] auto read_x = [&](int at) {
        if constexpr (KS == 32) {
#pragma unroll
            for (int i = 0; i < XS; ++i)
#pragma unroll
                for (int nb = 0; nb < NB; ++nb) {
                    const int t = tok + 16 * nb, c = 4 * (step[i] & 1) + g;
                    xr[i][nb] = *reinterpret_cast<const u32x4 *>(own + (((step[i] >> 1) - (min(first, p.S - 1) >> 1)) * (MP / 8) + (t >> 3)) * 1024 +
                                                                 (t & 7) * 128 + ((c ^ (t & 7)) * 16));
                }
            return;
        }
#pragma unroll
        for (int i = 0; i < kPass; ++i)
            if (at + i < XS)
#pragma unroll
                for (int nb = 0; nb < NB; ++nb)
#pragma unroll
                    for (int q = 0; q < XP; ++q) {
                        const int t = tok + 16 * nb, half = MP == 8 ? mcol >> 3 : q;
                        const int c = W16 ? 4 * half + g : 2 * g + half;
                        const int where = RANGE ? row_piece<MP, 128>(t, i, c, min(kPass, XS - at))
                                                : (i * (MP / 8) + (t >> 3)) * 1024 + (t & 7) * 128 + ((c ^ (t & 7)) * 16);
                        xr[at + i][nb * XP + q] = *reinterpret_cast<const u32x4 *>(own + where);
                    }
    };
    if constexpr (kPass > 0) {
        fetch_x(0);
    } else {
        // the slots of the first turn of the ring before the ring's loads, the others behind them
#pragma unroll
        for (int i = 0; i < (XS < RD || PRE != PRE_NONE ? XS : RD); ++i) load_x(i);
    }
    // gamma: requested with the activations where the registers hold both, else when the row sums are known
    constexpr bool kGammaEarly = 4 * XS * (NB + 1) * XP + 4 * RD <= (MP == 32 ? 160 : 84);
    [[maybe_unused]] u32x4 gm[PRE == PRE_RMSNORM ? XS : 1][XP];
    [[maybe_unused]] auto load_gamma = [&](int i) {
#pragma unroll
        for (int q = 0; q < XP; ++q) gm[i][q] = *reinterpret_cast<const u32x4 *>(p.pre_arg + kofs + 64 * step[i] + 8 * q);
    };
    if constexpr (PRE == PRE_RMSNORM && kGammaEarly)
#pragma unroll
        for (int i = 0; i < XS; ++i) load_gamma(i);
    [[maybe_unused]] unsigned int sc_first = 0;
    if constexpr (!W16) {
        if (2 * tid < ntiles * kTileRows)
            sc_first = *reinterpret_cast<const unsigned int *>(p.scales + (long long)share.tile(tid >> 3) * kTileRows + 2 * (tid & 7));
    }
    u32x2 resid[NB];
    load_residual<RES, NB>(p, share.tile(min(w, ntiles - 1)), lane, resid);

    const unsigned long long wbase = reinterpret_cast<unsigned long long>(p.w);
    const unsigned int tile_bytes = (unsigned int)p.Srow * (unsigned int)kSlotBytes;
    auto mine = [&](int i) { return PAIR ? (have >> i & 1u) != 0u : i < n; };
    u32x4 ring[RD][WL];
    // refill of ring entry d with slot i of tile tl; beyond the workgroup's last tile every lane reads the same 16 bytes
    auto refill = [&](int d, int tl, int i) {
        const bool real = tl < ntiles && (CC == 1 || mine(i));
        const unsigned long long a = real ? wbase + (unsigned long long)(unsigned int)share.tile(tl) * tile_bytes + (unsigned int)step[i] * (unsigned int)kSlotBytes
                                          : reinterpret_cast<unsigned long long>(p.x);
        unsigned int off = real ? 16u * lane : 0u;
#pragma unroll
        for (int j = 0; j < WL; ++j) ring[d][j] = ring_refill_at(a + (real ? j * kStepBytes : 0), off, ring[d][j]);
    };
#pragma unroll
    for (int d = 0; d < RD; ++d) {
#pragma unroll
        for (int j = 0; j < WL; ++j) ring[d][j] = u32x4{0u, 0u, 0u, 0u};
        refill(d, d / XS, d % XS);
    }
    if constexpr (kPass > 0) {
        // the direct-to-LDS loads were issued first and loads return in order: once no more than the ring's are
        // outstanding they are in LDS, where only this wave reads them
        asm volatile("s_waitcnt vmcnt(%0)" ::"n"(RD * WL) : "memory");
        read_x(0);
#pragma unroll
        for (int at = kPass; KS == 64 && at < XS; at += kPass) {
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
            fetch_x(at);
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
            read_x(at);
        }
    } else if constexpr (PRE == PRE_NONE) {
#pragma unroll
        for (int i = RD; i < XS; ++i) load_x(i);
    }

    // ---- what the activations need before they are operands
    if constexpr (!W16) {
        if (2 * tid < ntiles * kTileRows) reinterpret_cast<unsigned int *>(sc_lds)[tid] = sc_first;
        for (int i = 2 * (tid + NW * 64); i < ntiles * kTileRows; i += 2 * NW * 64)
            reinterpret_cast<unsigned int *>(sc_lds)[i >> 1] =
                *reinterpret_cast<const unsigned int *>(p.scales + (long long)share.tile(i >> 4) * kTileRows + (i & 15));
    }
    if constexpr (PRE == PRE_RMSNORM) {
        // sum of squares per token: this lane's values, the lanes of the token, then the waves in order
        float *red = reinterpret_cast<float *>(lds + NW * region + p.sc_bytes);    // [NW][MP]
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) {
            float ss = 0.f;
#pragma unroll
            for (int i = 0; i < XS; ++i)
#pragma unroll
                for (int q = 0; q < XP; ++q) {
                    const float s = piece_sumsq(xr[i][nb * XP + q]);
                    ss += i < n ? s : 0.f;
                }
            ss += __shfl_xor(ss, 16, 64);
            ss += __shfl_xor(ss, 32, 64);
            if constexpr (MP == 8) ss += __shfl_xor(ss, 8, 64);
            if (lane < (MP == 8 ? 8 : 16)) red[w * MP + lane + 16 * nb] = ss;
        }
        lds_barrier();
        float r[NB];
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) {
            float tot = 0.f;
#pragma unroll
            for (int ww = 0; ww < NW; ++ww) tot += red[ww * MP + tok + 16 * nb];
            r[nb] = __fdiv_rn(1.0f, __fsqrt_rn(__fdiv_rn(tot, (float)p.K) + p.eps));
        }
#pragma unroll
        for (int i = 0; i < XS; ++i) {
            if constexpr (!kGammaEarly) load_gamma(i);
#pragma unroll
            for (int nb = 0; nb < NB; ++nb)
#pragma unroll
                for (int q = 0; q < XP; ++q) xr[i][nb * XP + q] = pre_rmsnorm_piece(xr[i][nb * XP + q], gm[i][q], r[nb]);
        }
    }

    f32x4 acc[NB];
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) acc[nb] = f32x4{0.f, 0.f, 0.f, 0.f};
    float bestv[NB];
    unsigned int besti[NB];
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) { bestv[nb] = -__builtin_inff(); besti[nb] = 0x7FFFFFFFu; }
    [[maybe_unused]] float sume[NB] = {};            // EPI_LOGITS: sum of exp(z - bestv)
    int parity = 0;

    [[maybe_unused]] f32x4 share1[NB];               // PAIR: the second of the two shares
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) share1[nb] = f32x4{0.f, 0.f, 0.f, 0.f};
    // one slot: 64 k of a tile into the accumulators
    auto slot = [&](int d, int i) {
        bf16x8 a[2];
        if constexpr (W16) {
            a[0] = __builtin_bit_cast(bf16x8, ring[d][0]);
            a[1] = __builtin_bit_cast(bf16x8, ring[d][WL - 1]);
        } else {
            a[0] = codes_to_bf16x8(ring[d][0].x, ring[d][0].y);
            a[1] = codes_to_bf16x8(ring[d][0].z, ring[d][0].w);
        }
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) {
            const u32x4 b0 = xr[i][nb * XP];
            const u32x4 b1 = MP == 8 ? rotate_half_row(b0) : xr[i][nb * XP + XP - 1];
            f32x4 &to = PAIR && (i / (PAIR ? CH : 1)) % 2 == 1 ? share1[nb] : acc[nb];
            to = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[0], __builtin_bit_cast(bf16x8, b0), to, 0, 0, 0);
            if constexpr (KS == 64) to = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[1], __builtin_bit_cast(bf16x8, b1), to, 0, 0, 0);
        }
    };
    auto hand_over = [&](int c) {
        f32x4 *st = reinterpret_cast<f32x4 *>(own) + (parity * C + c) * NB * 64;
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) {
            st[nb * 64 + lane] = PAIR ? acc[nb] + share1[nb] : acc[nb];
            acc[nb] = f32x4{0.f, 0.f, 0.f, 0.f};
            if constexpr (PAIR) share1[nb] = f32x4{0.f, 0.f, 0.f, 0.f};
        }
    };
    // tile end: cross-wave sum through LDS, neighbouring waves in pairs, the pair sums in order, the chunks in order
    auto tile_end = [&](int tl) {
        lds_barrier();
        if (w == (tl % NW)) {
            f32x4 rsum[NB];
            for (int c = 0; c < C; ++c) {
                const unsigned char *st = lds + ((parity * C + c) * NB * 64 + lane) * 16;
#pragma unroll
                for (int nb = 0; nb < NB; ++nb, st += 1024) {
                    f32x4 s = {0.f, 0.f, 0.f, 0.f};
#pragma unroll 1
                    for (int w0 = 0; w0 < NW; w0 += 8)         // (a loop: bounds the registers of the reads in flight)
#pragma unroll
                        for (int ww = w0; ww < w0 + 8; ww += 2) {
                            const f32x4 s0 = *reinterpret_cast<const f32x4 *>(st + ww * region);
                            const f32x4 s1 = *reinterpret_cast<const f32x4 *>(st + (ww + 1) * region);
                            if constexpr (PAIR) s = (s + s0) + s1;           // (each the sum of a pair already)
                            else s += s0 + s1;
                        }
                    rsum[nb] = c > 0 ? s + rsum[nb] : s;
                }
            }
            if constexpr (PARS == 1) lds_barrier();          // (the others wait below: the one set of partial tiles is free again)
            finish_tile<W16, EPI, RES, NB>(p, rsum, share.tile(tl), sc_lds + tl * kTileRows, resid, gate_keep, slice, lane, bestv, besti);
            if constexpr (EPI == EPI_LOGITS) {
                if (p.soft_stats) {
                    // the logits of finish_tile once more: a running (max, sum) per lane and token
                    const u32x2 sb = *reinterpret_cast<const u32x2 *>(sc_lds + tl * kTileRows + 4 * g);
#pragma unroll
                    for (int nb = 0; nb < NB; ++nb)
                        softmax_add(bestv[nb], sume[nb], rsum[nb].x * bf16_bits_to_float(sb.x & 0xFFFFu) * p.inv_t,
                                    rsum[nb].y * bf16_bits_to_float(sb.x >> 16) * p.inv_t,
                                    rsum[nb].z * bf16_bits_to_float(sb.y & 0xFFFFu) * p.inv_t,
                                    rsum[nb].w * bf16_bits_to_float(sb.y >> 16) * p.inv_t);
                }
            }
            if (RES) load_residual<RES, NB>(p, share.tile(min(tl + NW, ntiles - 1)), lane, resid);      // of this wave's next tile
        } else if constexpr (PARS == 1) {
            lds_barrier();
        }
        if constexpr (PARS == 2) parity ^= 1;
    };
    auto round = [&](int tl0, auto last) {
        constexpr bool kLast = decltype(last)::value;
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int tl = tl0 + u;
            int c = 0;
            [[maybe_unused]] int bound = bound0;
#pragma unroll
            for (int i = 0; i < XS; ++i) {
                constexpr int R = RD;
                const int j = u * XS + i;
                if (mine(i) && (U == 1 || tl < ntiles)) slot(j % R, i);
                if (!kLast || j + R < U * XS) {
                    const int jn = j + R;
                    refill(j % R, tl0 + (jn / (U * XS)) * U + (jn % (U * XS)) / XS, jn % XS);
                }
                if constexpr (CC > 1) {
                    if ((i + 1) % (2 * CH) == 0) hand_over(i / (2 * CH));
                }
                if constexpr (CH && !PAIR) {
                    if (i + 1 == bound) {
                        hand_over(c);
                        ++c;
                        if (c < C) {
                            const int scc = min(p.SC, p.S - c * p.SC);
                            bound += (scc * (w + 1)) / NW - (scc * w) / NW;
                        }
                    }
                }
            }
            if (U == 1 || tl < ntiles) {
                if constexpr (!CH || (PAIR && CC == 1)) hand_over(0);
                tile_end(tl);
            }
        }
    };
    int tl0 = 0;
    for (; tl0 + U < ntiles; tl0 += U) round(tl0, std::false_type{});
    round(tl0, std::true_type{});

    if constexpr (EPI == EPI_ARGMAX) publish_argmax<MP, NB, NW>(bestv, besti, lds, p.partial + (long long)b * MP);
    if constexpr (EPI == EPI_LOGITS) {
        if (p.soft_stats) {
            float *red = reinterpret_cast<float *>(lds);             // [NW][MP] (max, sum)
            lds_barrier();   // all tile-end reads of the partial tiles are done
#pragma unroll
            for (int nb = 0; nb < NB; ++nb) {
#pragma unroll
                for (int off = 16; off <= 32; off <<= 1) {
                    const float m2 = __shfl_xor(bestv[nb], off, 64), s2 = __shfl_xor(sume[nb], off, 64);
                    softmax_merge(bestv[nb], sume[nb], m2, s2);
                }
                if (g == 0 && (MP != 8 || mcol < 8)) {
                    red[(w * MP + mcol + 16 * nb) * 2] = bestv[nb];
                    red[(w * MP + mcol + 16 * nb) * 2 + 1] = sume[nb];
                }
            }
            lds_barrier();
            if (tid < p.M) {
                float m = red[2 * tid], s = red[2 * tid + 1];
                for (int ww = 1; ww < NW; ++ww) softmax_merge(m, s, red[(ww * MP + tid) * 2], red[(ww * MP + tid) * 2 + 1]);
                p.soft_stats[((long long)tid * p.groups + b) * 2] = m;
                p.soft_stats[((long long)tid * p.groups + b) * 2 + 1] = s;
            }
        }
    }
}

// ---- dispatch over the built forms ----

template <int MP, bool W16, int EPI, int CH, int PRE, bool RES, int... XS>
int launch_direct_forms(int xs, dim3 grid, int lds_bytes, hipStream_t stream, const GemmParams &p) {
    int rc = QUASAR_ERR_SHAPE;
    ((xs == XS ? (void)(rc = launch(stream_direct_kernel<MP, W16, EPI, XS, CH, PRE, RES>, grid, direct_waves(MP, XS) * 64, lds_bytes,
                                    stream, p))
               : (void)0), ...);
    return rc;
}
template <bool W16, int EPI, int PRE, bool RES>
int launch_direct_as(const GemmParams &base, int MP, const DirectPlan &d, hipStream_t stream) {
    GemmParams p = base;
    p.S = p.Srow = p.K / 64;
    p.SC = d.SC;
    p.C = d.C;
    p.ksplit = d.ksplit;
    p.slice_steps = d.ksplit > 1 ? d.slice_steps : p.S;
    p.sc_bytes = d.sc_bytes;
    p.xs_bytes = 0;
    share_tiles(p, d.groups, d.ksplit, EPI == EPI_SWIGLU ? 2 : 1);
    const dim3 grid((unsigned int)d.ksplit, (unsigned int)d.groups);
    if constexpr (PRE == PRE_NONE && !RES && (EPI == EPI_LINEAR || EPI == EPI_ARGMAX)) {
        // (CH: slots of a share)
        if (d.pair) {
            if constexpr (W16) {
                p.S = p.Srow = p.slice_steps = p.K / 32;
                if constexpr (EPI == EPI_ARGMAX)
                    if (d.C > 1) return launch_direct_forms<32, W16, EPI, 2, PRE, RES, 8, 12, 16, 20>(d.XS, grid, d.lds_bytes, stream, p);
                if (d.XS == 2) return launch_direct_forms<32, W16, EPI, 1, PRE, RES, 2>(d.XS, grid, d.lds_bytes, stream, p);
                if (d.XS == 4) return launch_direct_forms<32, W16, EPI, 2, PRE, RES, 4>(d.XS, grid, d.lds_bytes, stream, p);
                return launch_direct_forms<32, W16, EPI, 3, PRE, RES, 6>(d.XS, grid, d.lds_bytes, stream, p);
            } else {
                if constexpr (EPI == EPI_ARGMAX)
                    if (d.C > 1) return launch_direct_forms<32, W16, EPI, 1, PRE, RES, 4, 6, 8, 10>(d.XS, grid, d.lds_bytes, stream, p);
                if (d.XS == 2) return launch_direct_forms<32, W16, EPI, 1, PRE, RES, 2>(d.XS, grid, d.lds_bytes, stream, p);
                return launch_direct_forms<32, W16, EPI, 2, PRE, RES, 4>(d.XS, grid, d.lds_bytes, stream, p);
            }
        }
        if (d.C > 1) {
            if (MP == 8) return launch_direct_forms<8, W16, EPI, 1, PRE, RES, 8, 10, 12>(d.XS, grid, d.lds_bytes, stream, p);
            // (bf16 weights: chunks of whole slots for every wave, K = 4096 and 6144)
            if constexpr (W16) return launch_direct_forms<16, W16, EPI, 1, PRE, RES, 4, 6>(d.XS, grid, d.lds_bytes, stream, p);
            else return launch_direct_forms<16, W16, EPI, 1, PRE, RES, 4, 5, 6, 8>(d.XS, grid, d.lds_bytes, stream, p);
        }
    }
    if constexpr (EPI == EPI_ARGMAX) {
        // the order of the staged kernel: K in one piece is 120 slots at 8 tokens, 60 at 16
        if (MP == 8) return launch_direct_forms<8, W16, EPI, 0, PRE, RES, 1, 2, 3, 4, 5, 6, 7, 8>(d.XS, grid, d.lds_bytes, stream, p);
        return launch_direct_forms<16, W16, EPI, 0, PRE, RES, 1, 2, 3, 4>(d.XS, grid, d.lds_bytes, stream, p);
    } else if constexpr (PRE != PRE_NONE) {
        if (MP == 8) return launch_direct_forms<8, W16, EPI, 0, PRE, RES, 1, 2, 3, 4, 5, 6, 7, 8>(d.XS, grid, d.lds_bytes, stream, p);
        if (MP == 16) return launch_direct_forms<16, W16, EPI, 0, PRE, RES, 1, 2, 3, 4, 5>(d.XS, grid, d.lds_bytes, stream, p);
        return launch_direct_forms<32, W16, EPI, 0, PRE, RES, 2, 4, 6, 8, 10>(d.XS, grid, d.lds_bytes, stream, p);
    } else {
        if (MP == 8) return launch_direct_forms<8, W16, EPI, 0, PRE, RES, 1, 2, 3, 4, 5, 6, 7, 8, 10, 12>(d.XS, grid, d.lds_bytes, stream, p);
        if (MP == 16) {
            if constexpr (W16) return launch_direct_forms<16, W16, EPI, 0, PRE, RES, 1, 2, 3, 4, 5, 6, 8, 20>(d.XS, grid, d.lds_bytes, stream, p);
            else return launch_direct_forms<16, W16, EPI, 0, PRE, RES, 1, 2, 3, 4, 5, 6, 8, 20, 24>(d.XS, grid, d.lds_bytes, stream, p);
        }
        return launch_direct_forms<32, W16, EPI, 0, PRE, RES, 2, 4, 6, 8, 10>(d.XS, grid, d.lds_bytes, stream, p);
    }
}

}  // namespace quasar
