// Skinny-M weight streaming with K outermost (gfx950): W8A8 and 4-bit weights.
//
// A workgroup's NT weight tiles are walked side by side: a pass is one slot of K - 64 k, 128 of 4-bit weights - of every
// tile, so a slot of activations is fetched when its pass is near, serves the NT tiles and is forgotten.  The kernels that
// hold a wave's whole slice of x (stream_direct_a8.hpp, stream_direct_w4.hpp) run out of registers where M x K is large; this one
// takes the registers of a few slots whatever K is, and the waves meet once, behind the last pass, where the tiles'
// cross-wave sums are taken by as many waves as there are tiles.  Wave w takes the slots w, w + NW, .. of a tile, so a pass
// of the workgroup is NW contiguous KB of each tile and of x.
//
// Everything a lane loads is ordinary vector loads of constant number per pass, so the compiler waits on counts.
//
// W8A8: the activations come as int8 codes in operand order from a launch of their own (quantize_operand_kernel), 64 bytes
// a token and slot in contiguous KB.  Quantising in every workgroup costs eight vector instructions an element, 256
// times over; the launch costs 2.8 us once.
//
// 4-bit weights: x is read in place, eight tokens' 128 bytes an instruction; an eight-lane rotation with a bank mask turns the
// two halves of 16 tokens into two operands, and the group's offset is a matrix product a pass (stream_direct_w4.hpp).
//
// What bounds it: the weight stream and, in the same in-order queue of the compute unit, x at about 50 KB/us; nothing of x is
// hidden behind the weights (int8 weights with bf16 activations were slower so: 12288 x 4096, M = 32 13.9 -> 16.3 us).
// us a call against the kernels that hold x: at the rules that choose between them (plan_w8a8_apart, plan_w4_outer).
#pragma once

#include "launch.hpp"
#include "stream_w4.hpp"
#include "stream_w8a8.hpp"

namespace quasar {

// lanes 8..15 of every row of 16 <- lanes 0..7 of `hi`; the others keep `lo`
__device__ __forceinline__ unsigned int low_halves(unsigned int lo, unsigned int hi) {
    return (unsigned int)__builtin_amdgcn_update_dpp((int)lo, (int)hi, 0x128, 0xf, 0xc, false);
}
// lanes 0..7 <- lanes 8..15 of `lo`; the others keep `hi`
__device__ __forceinline__ unsigned int high_halves(unsigned int lo, unsigned int hi) {
    return (unsigned int)__builtin_amdgcn_update_dpp((int)hi, (int)lo, 0x128, 0xf, 0x3, false);
}

// A load of activations, its address tied to the registers it replaces as in ring_refill_at; cached, every compute unit reads it.
__device__ __forceinline__ u32x4 x_refill_at(unsigned long long base, unsigned int lane_offset, const u32x4 &used) {
    asm volatile("" : "+v"(lane_offset) : "v"(used.x), "v"(used.y), "v"(used.z), "v"(used.w));
    return *reinterpret_cast<global_u32x4_ptr>(base + lane_offset);
}

// LDS: [NW waves x NT tiles x NB partial tiles of 1 KB][row scales]
// p.S, p.Srow, p.slice_steps: in slots.  FMT_A8: p.x is the codes of quantize_operand_kernel, p.dx their step sizes.
template <int FMT, int MP, int NT>
__global__ __launch_bounds__(outer_waves(MP) * 64) void stream_outer_kernel(const GemmParams p0) {
    extern __shared__ __align__(16) unsigned char lds[];
    constexpr int NW = outer_waves(MP);
    constexpr int NB = MP == 32 ? 2 : 1;
    constexpr int D = outer_depth(FMT, MP, NT);              // passes the weights are ahead
    constexpr int PB = D == 1 ? 2 : D;                       // passes of a round = passes x is ahead
    constexpr int XL = outer_x_loads(FMT, MP);               // 16-byte loads of x a lane and slot
    constexpr int SB = FMT == FMT_W4 ? kStepBytes4 : kStepBytes;
    constexpr int OPS = FMT == FMT_W4 ? 4 : 1;               // B operands a slot and 16 tokens
    typedef std::conditional_t<FMT == FMT_A8, i32x4, f32x4> sum_t;

    const int slice = blockIdx.x, b = blockIdx.y;
    const GemmParams &p = p0;
    loaded_together<TileShare<1, false, false>>(p, p.x, p.w, p.scales, p.ldx, p.S, p.Srow, p.slice_steps, p.M);
    const int s0 = slice * p.slice_steps;
    const int S = min(p.slice_steps, p.S - s0);

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int g = lane >> 4, mcol = lane & 15;
    const int t0 = share_begin(p.tq, p.tr, b), ntiles = share_count(p.tq, p.tr, b);       // <= NT
    const int n = (S - w + NW - 1) / NW;                     // the wave's slots: w, w + NW, ..

    // ---- where the lane reads x
    unsigned int xofs[FMT == FMT_A8 ? 1 : MP / 8];
    const unsigned long long xbase = reinterpret_cast<unsigned long long>(p.x);
    constexpr unsigned int kXSlot = FMT == FMT_A8 ? 64u * MP : 256u;
    if constexpr (FMT == FMT_A8) {
        xofs[0] = MP == 8 ? 16u * (8 * g + (mcol & 7)) : 16u * lane;
    } else {
        const unsigned int kofs = 16u * g + 64u * (mcol >> 3);
#pragma unroll
        for (int j = 0; j < MP / 8; ++j)
            xofs[j] = (unsigned int)min((mcol & 7) + 8 * j, p.M - 1) * (unsigned int)(2 * p.ldx) + kofs;
    }
    [[maybe_unused]] unsigned int sc_own = 0;                // two row scales of the workgroup's tiles
    if constexpr (FMT == FMT_A8) {
        if (2 * tid < ntiles * kTileRows) sc_own = *reinterpret_cast<const unsigned int *>(p.scales + (long long)t0 * kTileRows + 2 * tid);
    }
    u32x4 xb[PB][XL];
    auto load_x = [&](int d, int i) {
        const bool real = i < n;                             // (else one line, 16 bytes for all lanes)
        const unsigned long long a = real ? xbase + (unsigned long long)(unsigned int)(s0 + w + i * NW) * kXSlot : xbase;
        const unsigned int all = real ? ~0u : 0u;
#pragma unroll
        for (int l = 0; l < XL; ++l) {
            if constexpr (FMT == FMT_A8) xb[d][l] = x_refill_at(a + 1024 * l, xofs[0] & all, xb[d][l]);
            else xb[d][l] = x_refill_at(a + 128 * (l & 1), xofs[l >> 1] & all, xb[d][l]);
        }
    };

    // ---- the weight ring: D passes of NT slots
    const unsigned int tile_bytes = (unsigned int)p.Srow * (unsigned int)SB;
    const unsigned long long wbase = reinterpret_cast<unsigned long long>(p.w) + (unsigned long long)t0 * tile_bytes +
                                     (unsigned long long)(unsigned int)(s0 + w) * (unsigned int)SB;
    u32x4 ring[D][NT];
    [[maybe_unused]] u32x2 scl[D][NT];
    auto refill = [&](int d, int u, int i) {
        const bool real = i < n && u < ntiles;               // (else one line that every compute unit holds)
        const unsigned long long a = real ? wbase + (unsigned long long)u * tile_bytes + (unsigned int)(i * NW) * (unsigned int)SB : xbase;
        unsigned int off = real ? 16u * lane : 0u;
        ring[d][u] = ring_refill_at(a, off, ring[d][u]);
        if constexpr (FMT == FMT_W4) {
            unsigned int os = real ? 1024u + 8u * g : 0u;
            scl[d][u] = ring_refill2_at(a, os, scl[d][u]);
        }
    };
#pragma unroll
    for (int d = 0; d < PB; ++d) {
#pragma unroll
        for (int l = 0; l < XL; ++l) xb[d][l] = u32x4{0u, 0u, 0u, 0u};
        load_x(d, d);
        if (d < D)
#pragma unroll
            for (int u = 0; u < NT; ++u) {
                ring[d][u] = u32x4{0u, 0u, 0u, 0u};
                if constexpr (FMT == FMT_W4) scl[d][u] = u32x2{0u, 0u};
                refill(d, u, d);
            }
    }
    sum_t acc[NT][NB];
#pragma unroll
    for (int u = 0; u < NT; ++u)
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) acc[u][nb] = sum_t{};
    [[maybe_unused]] unsigned int nib_mask, nib_magic;
    if constexpr (FMT == FMT_W4) w4_constants(nib_mask, nib_magic);

    auto pass = [&](int q, int i) {
        u32x4 op[NB][OPS];
        [[maybe_unused]] float gofs[NB];
        if constexpr (FMT == FMT_A8) {
#pragma unroll
            for (int nb = 0; nb < NB; ++nb) op[nb][0] = xb[q][nb];
        } else {
            constexpr int H = OPS / 2;                       // 128-byte lines a token and slot
#pragma unroll
            for (int nb = 0; nb < NB; ++nb)
#pragma unroll
                for (int h = 0; h < H; ++h) {
                    if constexpr (MP == 8) {
                        op[0][2 * h] = xb[q][h];
                        op[0][2 * h + 1] = rotate_half_row(xb[q][h]);
                    } else {
                        const u32x4 lo = xb[q][(2 * nb) * H + h], hi = xb[q][(2 * nb + 1) * H + h];
                        op[nb][2 * h] = u32x4{low_halves(lo.x, hi.x), low_halves(lo.y, hi.y), low_halves(lo.z, hi.z), low_halves(lo.w, hi.w)};
                        op[nb][2 * h + 1] = u32x4{high_halves(lo.x, hi.x), high_halves(lo.y, hi.y), high_halves(lo.z, hi.z), high_halves(lo.w, hi.w)};
                    }
                }
        }
        load_x(q, i + PB);       // (in front of the pass's weights: what it waits for then leaves D passes of weights in flight)
        if constexpr (FMT == FMT_W4) {
            // the group's offset -136 * (sum of its activations), in every row (stream_direct_w4.hpp)
            const u32x4 k136 = {0xC308C308u, 0xC308C308u, 0xC308C308u, 0xC308C308u};
#pragma unroll
            for (int nb = 0; nb < NB; ++nb) {
                f32x4 o = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int j = 0; j < OPS; ++j)
                    o = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, k136), __builtin_bit_cast(bf16x8, op[nb][j]), o, 0, 0, 0);
                gofs[nb] = o.x;
            }
        }
#pragma unroll
        for (int u = 0; u < NT; ++u) {
            const int d = q % D;
            if (u < ntiles) {
                if constexpr (FMT == FMT_A8) {
#pragma unroll
                    for (int nb = 0; nb < NB; ++nb)
                        acc[u][nb] = __builtin_amdgcn_mfma_i32_16x16x64_i8(__builtin_bit_cast(i32x4, ring[d][u]),
                                                                           __builtin_bit_cast(i32x4, op[nb][0]), acc[u][nb], 0, 0, 0);
                } else {
                    const u32x4 wd = ring[d][u];
                    const unsigned int wds[4] = {wd.x, wd.y, wd.z, wd.w};
                    f32x4 grp[NB];
#pragma unroll
                    for (int nb = 0; nb < NB; ++nb) grp[nb] = f32x4{gofs[nb], gofs[nb], gofs[nb], gofs[nb]};
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        const bf16x8 a = w4_to_bf16x8(wds[j], nib_mask, nib_magic);
#pragma unroll
                        for (int nb = 0; nb < NB; ++nb)
                            grp[nb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, __builtin_bit_cast(bf16x8, op[nb][j]), grp[nb], 0, 0, 0);
                    }
                    const u32x2 sc = scl[d][u];
                    const float f0 = __uint_as_float(sc.x << 16), f1 = __uint_as_float(sc.x & 0xFFFF0000u);
                    const float f2 = __uint_as_float(sc.y << 16), f3 = __uint_as_float(sc.y & 0xFFFF0000u);
#pragma unroll
                    for (int nb = 0; nb < NB; ++nb) {
                        acc[u][nb].x = __builtin_fmaf(f0, grp[nb].x, acc[u][nb].x);
                        acc[u][nb].y = __builtin_fmaf(f1, grp[nb].y, acc[u][nb].y);
                        acc[u][nb].z = __builtin_fmaf(f2, grp[nb].z, acc[u][nb].z);
                        acc[u][nb].w = __builtin_fmaf(f3, grp[nb].w, acc[u][nb].w);
                    }
                }
            }
            refill(d, u, i + D);
        }
    };
    for (int r = 0; r < n; r += PB) {
#pragma unroll
        for (int q = 0; q < PB; ++q) {
            if (q > 0 && r + q >= n) break;
            pass(q, r + q);
        }
    }

    // ---- the waves meet: wave w sums the partial tiles of tile w (and w + NW ..), neighbouring waves in pairs
    f32x4 *part = reinterpret_cast<f32x4 *>(lds);
    uint16_t *sc_lds = reinterpret_cast<uint16_t *>(lds + NW * NT * NB * 1024);
    if constexpr (FMT == FMT_A8) {
        if (2 * tid < ntiles * kTileRows) reinterpret_cast<unsigned int *>(sc_lds)[tid] = sc_own;
    }
#pragma unroll
    for (int u = 0; u < NT; ++u)
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) part[((w * NT + u) * NB + nb) * 64 + lane] = __builtin_bit_cast(f32x4, acc[u][nb]);
    lds_barrier();
    for (int tl = w; tl < ntiles; tl += NW) {
        sum_t sum[NB];
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) {
            sum[nb] = sum_t{};
#pragma unroll
            for (int ww = 0; ww < NW; ww += 2)
                sum[nb] += __builtin_bit_cast(sum_t, part[((ww * NT + tl) * NB + nb) * 64 + lane]) +
                           __builtin_bit_cast(sum_t, part[(((ww + 1) * NT + tl) * NB + nb) * 64 + lane]);
        }
        if constexpr (FMT == FMT_A8) {
            const int n0 = (t0 + tl) * kTileRows + 4 * g;
            const u32x2 sb = *reinterpret_cast<const u32x2 *>(sc_lds + tl * kTileRows + 4 * g);
#pragma unroll
            for (int nb = 0; nb < NB; ++nb) {
                const int m = mcol + 16 * nb;
                if (m >= p.M) continue;
                if (p.ksplit > 1) {
                    *reinterpret_cast<i32x4 *>(reinterpret_cast<int *>(p.part32) + ((long long)slice * p.M + m) * p.N + n0) = sum[nb];
                } else {
                    const float dx = p.dx[m];
                    *reinterpret_cast<u32x2 *>(p.y + m * p.ldy + n0) = a8_outputs(sum[nb], sb, dx);
                }
            }
        } else {
            const u32x2 none[NB] = {};
            float bestv[NB];
            unsigned int besti[NB];
            finish_tile<true, EPI_LINEAR, false, NB>(p, sum, t0 + tl, nullptr, none, nullptr, slice, lane, bestv, besti);
        }
    }
}

// y[m, n] = bf16( (sum over K slices, in slice order, of part[slice][m][n]) * step size ): the second launch of a K split.
// One thread per four consecutive outputs of a token; blockIdx.y is the token.  Launch-sized: what a thread waits for is one
// trip to memory, so the slices are requested together and added in order (one after the other they cost 0.6 us each); two, four or
// eight of them, for requests that only repeat the last slice take their turn too (us a call, eight requested, two or four: bf16 2048 x 12288 M = 4, two slices 12.65, 12.3; int8 1024 x 12288 M = 16, four 8.1, 7.9).
template <int FMT>
__global__ __launch_bounds__(256) void splitk_finalize_kernel(const float *part, int ksplit, int M, int N, const uint16_t *scales,
                                                              const float *dx, const uint16_t *resid, long long ldr, uint16_t *y,
                                                              long long ldy) {
    typedef std::conditional_t<FMT == FMT_A8, i32x4, f32x4> sum_t;
    const int n0 = 4 * (blockIdx.x * 256 + threadIdx.x), m = blockIdx.y;
    if (n0 >= N) return;
    const float *mine = part + (long long)m * N + n0;
    u32x2 sb = {0u, 0u};
    if constexpr (FMT == FMT_INT8 || FMT == FMT_A8) sb = *reinterpret_cast<const u32x2 *>(scales + n0);
    sum_t acc = {};
    auto add = [&](int base, auto together) {
        constexpr int R = decltype(together)::value;
        sum_t v[R];
#pragma unroll
        for (int j = 0; j < R; ++j) v[j] = *reinterpret_cast<const sum_t *>(mine + (long long)min(base + j, ksplit - 1) * M * N);
#pragma unroll
        for (int j = 0; j < R; ++j)
            if (base + j < ksplit) acc = base + j == 0 ? v[j] : acc + v[j];
    };
    if (ksplit <= 2) add(0, std::integral_constant<int, 2>{});
    else if (ksplit <= 4) add(0, std::integral_constant<int, 4>{});
    else
        for (int base = 0; base < ksplit; base += 8) add(base, std::integral_constant<int, 8>{});
    u32x2 o;
    if constexpr (FMT == FMT_A8) {
        o = a8_outputs(acc, sb, dx[m]);
    } else {
        float s4[4] = {1.f, 1.f, 1.f, 1.f};
        if constexpr (FMT == FMT_INT8) {
            s4[0] = bf16_bits_to_float(sb.x & 0xFFFFu);
            s4[1] = bf16_bits_to_float(sb.x >> 16);
            s4[2] = bf16_bits_to_float(sb.y & 0xFFFFu);
            s4[3] = bf16_bits_to_float(sb.y >> 16);
        }
        o.x = float_to_bf16_bits(acc.x * s4[0]) | (float_to_bf16_bits(acc.y * s4[1]) << 16);
        o.y = float_to_bf16_bits(acc.z * s4[2]) | (float_to_bf16_bits(acc.w * s4[3]) << 16);
    }
    if constexpr (FMT == FMT_INT8) {
        if (resid) {                                         // (may be y itself: read here, by the thread that writes)
            const u32x2 rr = *reinterpret_cast<const u32x2 *>(resid + m * ldr + n0);
            const float r0 = bf16_bits_to_float(o.x & 0xFFFFu) + bf16_bits_to_float(rr.x & 0xFFFFu);
            const float r1 = __uint_as_float(o.x & 0xFFFF0000u) + __uint_as_float(rr.x & 0xFFFF0000u);
            const float r2 = bf16_bits_to_float(o.y & 0xFFFFu) + bf16_bits_to_float(rr.y & 0xFFFFu);
            const float r3 = __uint_as_float(o.y & 0xFFFF0000u) + __uint_as_float(rr.y & 0xFFFF0000u);
            o.x = float_to_bf16_bits(r0) | (float_to_bf16_bits(r1) << 16);
            o.y = float_to_bf16_bits(r2) | (float_to_bf16_bits(r3) << 16);
        }
    }
    *reinterpret_cast<u32x2 *>(y + m * ldy + n0) = o;
}

// ---- dispatch over the built forms ----

template <int FMT, int MP, int... NT>
int launch_outer_forms(int nt, dim3 grid, int lds_bytes, hipStream_t stream, const GemmParams &p) {
    int rc = QUASAR_ERR_SHAPE;
    ((nt == NT ? (void)(rc = launch(stream_outer_kernel<FMT, MP, NT>, grid, outer_waves(MP) * 64, lds_bytes, stream, p)) : (void)0), ...);
    return rc;
}
template <int FMT>
int launch_outer_as(const GemmParams &base, int MP, const DirectPlan &d, hipStream_t stream) {
    GemmParams p = base;
    p.S = p.Srow = p.K / outer_slot_k(FMT);
    p.ksplit = d.ksplit;
    p.slice_steps = d.ksplit > 1 ? d.slice_steps : p.S;
    share_tiles(p, d.groups, d.ksplit, 1);
    const dim3 grid((unsigned int)d.ksplit, (unsigned int)d.groups);
    if (MP == 8) return launch_outer_forms<FMT, 8, 1, 2, 3, 4, 5, 6, 7, 8>(d.XS, grid, d.lds_bytes, stream, p);
    if (MP == 16) {
        if constexpr (outer_tiles(FMT, 16) == 6) return launch_outer_forms<FMT, 16, 1, 2, 3, 4, 5, 6>(d.XS, grid, d.lds_bytes, stream, p);
        else return launch_outer_forms<FMT, 16, 1, 2, 3, 4, 5, 6, 7, 8>(d.XS, grid, d.lds_bytes, stream, p);
    }
    return launch_outer_forms<FMT, 32, 1, 2, 3, 4, 5, 6, 7, 8>(d.XS, grid, d.lds_bytes, stream, p);
}

}  // namespace quasar
