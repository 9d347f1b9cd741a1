// Offline weight preparation kernels: quantise + pack, unpack, bf16 pack (gfx950).
//
// Packed order (both dtypes): a "step" is 1024 contiguous bytes read by one wave-wide
// 128-bit load; lane l = 16*g + i of step s of tile t holds, for int8,
//     W[16 t + i][64 s + 16 g + 0..15]        (16 codes)
// and for bf16
//     W[16 t + i][32 s +  8 g + 0..7]         (8 values).
// Steps of a tile are contiguous, tiles follow each other, so a workgroup that owns a
// tile range streams one contiguous address range.
#pragma once

#include "quasar_device.hpp"

namespace quasar {

template <bool SRC_BF16>
__device__ __forceinline__ float load_w(const void *w, long long idx) {
    if constexpr (SRC_BF16)
        return bf16_bits_to_float(reinterpret_cast<const uint16_t *>(w)[idx]);
    else
        return reinterpret_cast<const float *>(w)[idx];
}

// rint(v / s) of the quotient of one IEEE division.  v * inv, inv the rounded reciprocal, is within 2^-23 of the quotient
// relatively, the rounded quotient within 2^-24: below 256 that is 4.6e-5, so both round alike unless the product lies closer
// than that to a half (one element in ten thousand), where the division is made.  Not-finite products make it too.
__device__ __forceinline__ float rounded_ratio(float v, float s, float inv) {
    const float q = v * inv;
    float r = rintf(q);
    if (!(fabsf(q - r) < 0.49995f)) r = rintf(__fdiv_rn(v, s));
    return r;
}

// One workgroup of 8 waves per 16-row tile; a wave owns two rows.  Bound by memory (4 or 2 bytes in, 1 out per weight), so
// a row is read once, 16 bytes a lane and load, and kept in registers (NJ loads a lane) from its maximum to its codes; of
// longer rows the maximum is taken first and the row read again.  The tile's codes meet in LDS in packed order - slots of
// 16 rows x 16 k, 16 bytes further apart than their length, so that the lanes of a store meet different banks - and leave in
// contiguous 16-byte pieces.  Up to K = 4096 two workgroups share a compute unit: one converts while the other's rows
// arrive.  With scalar loads, two passes and 16-byte
// pieces stored row by row -> now, us: 12288 x 4096 fp32 240 -> 47 (5.4 TB/s), bf16 165 -> 33, fp32 smoothed 209 -> 67;
// 25600 x 5120 fp32 632 -> 162, bf16 (read twice) 432 -> 135; 1024 x 1024 fp32 15.6 -> 8.5.
// VEC: rows (and smooth) start on 16 bytes; otherwise the same elements are read one by one.
constexpr int kQuantWaves = 8;
constexpr int kQuantSlotBytes = kTileRows * 16 + 16;

template <bool SRC_BF16, bool SMOOTH, bool VEC, int NJ>
__global__ __launch_bounds__(kQuantWaves * 64, NJ > 16 ? 2 : 4) void quantize_pack_kernel(const void *w, long long ldw, int K,
                                                                                        const float *smooth, u32x4 *packed,
                                                                                        uint16_t *scales) {
    extern __shared__ __align__(16) unsigned char lds[];
    constexpr int VE = SRC_BF16 ? 8 : 4;              // elements per lane and load
    constexpr int kSpan = NJ * 64 * VE;               // k of a row that a wave holds
    const int tid = threadIdx.x, lane = tid & 63;
    const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int t = blockIdx.x;

    u32x4 raw[NJ];
    auto load_row = [&](int row, int k0) {
        // (a wave-uniform address and the lane's offset: no address registers per load)
        const long long base = (long long)(t * kTileRows + row) * ldw + k0;
        const unsigned long long at = reinterpret_cast<unsigned long long>(w) + base * (SRC_BF16 ? 2 : 4);
#pragma unroll
        for (int j = 0; j < NJ; ++j) {
            raw[j] = u32x4{0u, 0u, 0u, 0u};
            if (lane * VE < K - k0 - 64 * j * VE) {
                if constexpr (VEC) {
                    typedef const __attribute__((address_space(1))) u32x4 *vec_ptr;
                    raw[j] = __builtin_nontemporal_load(reinterpret_cast<vec_ptr>(at + 1024u * j + 16u * (unsigned int)lane));
                } else {
                    const int k = (64 * j + lane) * VE;
                    unsigned int u[4];
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        if constexpr (SRC_BF16) {
                            const uint16_t *p = reinterpret_cast<const uint16_t *>(w) + base + k + 2 * e;
                            u[e] = p[0] | ((unsigned int)p[1] << 16);
                        } else {
                            u[e] = reinterpret_cast<const unsigned int *>(w)[base + k + e];
                        }
                    }
                    raw[j] = u32x4{u[0], u[1], u[2], u[3]};
                }
            }
        }
    };
    // the VE values of raw[j] with the offline side of the smoothing transformation (W diag(s)^-1, one fp32 division)
    auto values = [&](int j, int k, float (&v)[VE]) {
        const unsigned int u[4] = {raw[j].x, raw[j].y, raw[j].z, raw[j].w};
#pragma unroll
        for (int e = 0; e < VE; ++e)
            v[e] = !SRC_BF16 ? __uint_as_float(u[e & 3])
                             : ((e & 1) ? __uint_as_float(u[e >> 1] & 0xFFFF0000u) : __uint_as_float(u[e >> 1] << 16));
        if constexpr (SMOOTH) {
            if (k < K) {
                float sm[VE];
                if constexpr (VEC) {
#pragma unroll
                    for (int e = 0; e < VE; e += 4) {
                        const f32x4 s4 = *reinterpret_cast<const f32x4 *>(smooth + k + e);
                        sm[e] = s4.x; sm[e + 1] = s4.y; sm[e + 2] = s4.z; sm[e + 3] = s4.w;
                    }
                } else {
#pragma unroll
                    for (int e = 0; e < VE; ++e) sm[e] = smooth[k + e];
                }
#pragma unroll
                for (int e = 0; e < VE; ++e) v[e] = __fdiv_rn(v[e], sm[e]);
            }
        }
    };
    // largest magnitude of the held span; fp32 values are kept smoothed
    auto held_amax = [&](int k0, float amax) {
#pragma unroll
        for (int j = 0; j < NJ; ++j) {
            float v[VE];
            values(j, k0 + (64 * j + lane) * VE, v);
            if constexpr (SMOOTH && !SRC_BF16)
                raw[j] = u32x4{__float_as_uint(v[0]), __float_as_uint(v[1]), __float_as_uint(v[2]), __float_as_uint(v[3])};
#pragma unroll
            for (int e = 0; e < VE; ++e) amax = fmaxf(amax, fabsf(v[e]));
            if constexpr (SMOOTH) __builtin_amdgcn_sched_barrier(0);       // one load's quotients at a time
        }
        return amax;
    };
    // the row's step size (stored), 0 for a row without one
    auto step_size = [&](int row, float amax) {
#pragma unroll
        for (int off = 32; off >= 1; off >>= 1) amax = fmaxf(amax, __shfl_xor(amax, off, 64));
        unsigned int sb = float_to_bf16_bits(__fdiv_rn(amax, 127.0f));
        float s = bf16_bits_to_float(sb);
        if (!(s > 0.f)) { sb = 0; s = 0.f; }
        if (lane == 0) scales[t * kTileRows + row] = (uint16_t)sb;
        return s;
    };
    auto codes_to_lds = [&](int row, int k0, float s, bool smoothed) {
        const float inv = __fdiv_rn(1.0f, s);
        // bf16, smoothed: the quotients are formed again from the held words (kept from the maximum they spill)
        if constexpr (SRC_BF16 && SMOOTH) asm volatile("" ::: "memory");
#pragma unroll
        for (int j = 0; j < NJ; ++j) {
            const int kk = (64 * j + lane) * VE;
            if constexpr (SRC_BF16 && SMOOTH) asm volatile("" : "+v"(raw[j].x), "+v"(raw[j].y), "+v"(raw[j].z), "+v"(raw[j].w));
            float v[VE];
            if (SMOOTH && !SRC_BF16 && smoothed) {
                v[0] = __uint_as_float(raw[j].x); v[1] = __uint_as_float(raw[j].y);
                v[2] = __uint_as_float(raw[j].z); v[3] = __uint_as_float(raw[j].w);
            } else {
                values(j, k0 + kk, v);
            }
            unsigned int word[VE / 4];
#pragma unroll
            for (int q = 0; q < VE / 4; ++q) {
                word[q] = 0;
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const float r = fminf(fmaxf(rounded_ratio(v[4 * q + e], s, inv), -127.f), 127.f);
                    word[q] |= ((unsigned int)(int)r & 0xffu) << (8 * e);
                }
                if (!(s > 0.f)) word[q] = 0;
            }
            if (lane * VE < K - k0 - 64 * j * VE) {
                unsigned char *dst = lds + j * (4 * VE * kQuantSlotBytes) + row * 16 + ((lane * VE) >> 4) * kQuantSlotBytes + ((lane * VE) & 15);
                if constexpr (VE == 4) *reinterpret_cast<unsigned int *>(dst) = word[0];
                else *reinterpret_cast<u32x2 *>(dst) = u32x2{word[0], word[VE / 4 - 1]};
            }
            __builtin_amdgcn_sched_barrier(0);               // (bounds the registers of codes in the making)
        }
    };
    auto store_span = [&](int k0) {
        u32x4 *out = packed + ((long long)t * K + k0);               // 16 rows x 1 k per 16 bytes
        const int n = min(kSpan, K - k0);
        for (int q = tid; q < n; q += kQuantWaves * 64)
            __builtin_nontemporal_store(*reinterpret_cast<const u32x4 *>(lds + (q >> 4) * kQuantSlotBytes + (q & 15) * 16), out + q);
    };

    if (K <= kSpan) {
#pragma unroll 1
        for (int row = 2 * wv; row < 2 * wv + 2; ++row) {
            load_row(row, 0);
            codes_to_lds(row, 0, step_size(row, held_amax(0, 0.f)), true);
        }
        __syncthreads();
        store_span(0);
        return;
    }
    float s[2];
#pragma unroll
    for (int rr = 0; rr < 2; ++rr) {
        float amax = 0.f;
#pragma unroll 1
        for (int k0 = 0; k0 < K; k0 += kSpan) {
            load_row(2 * wv + rr, k0);
            amax = held_amax(k0, amax);
        }
        s[rr] = step_size(2 * wv + rr, amax);
    }
#pragma unroll 1
    for (int k0 = 0; k0 < K; k0 += kSpan) {
#pragma unroll
        for (int rr = 0; rr < 2; ++rr) {
            load_row(2 * wv + rr, k0);
            codes_to_lds(2 * wv + rr, k0, s[rr], false);
        }
        __syncthreads();
        store_span(k0);
        __syncthreads();
    }
}

__global__ __launch_bounds__(256) void unpack_kernel(const u32x4 *packed, int N, int K, int8_t *q) {
    const int S = K / kStepK8;
    const long long nslots = (long long)(N / kTileRows) * S * 64;
    for (long long slot = (long long)blockIdx.x * 256 + threadIdx.x; slot < nslots;
         slot += (long long)gridDim.x * 256) {
        const int l = (int)(slot & 63);
        const long long ts = slot >> 6;
        const int s = (int)(ts % S);
        const long long t = ts / S;
        const int g = l >> 4, i = l & 15;
        const u32x4 v = packed[slot];
        *reinterpret_cast<u32x4 *>(q + (t * kTileRows + i) * (long long)K + (long long)s * kStepK8 + 16 * g) = v;
    }
}

template <bool SRC_BF16>
__global__ __launch_bounds__(256) void pack_bf16_kernel(const void *w, long long ldw, int N, int K,
                                                        u32x4 *packed) {
    const int S = K / kStepK16;
    const long long nslots = (long long)(N / kTileRows) * S * 64;
    for (long long slot = (long long)blockIdx.x * 256 + threadIdx.x; slot < nslots;
         slot += (long long)gridDim.x * 256) {
        const int l = (int)(slot & 63);
        const long long ts = slot >> 6;
        const int s = (int)(ts % S);
        const long long t = ts / S;
        const int g = l >> 4, i = l & 15;
        const long long base = (t * kTileRows + i) * ldw + (long long)s * kStepK16 + 8 * g;
        unsigned int h[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            if constexpr (SRC_BF16)
                h[e] = reinterpret_cast<const uint16_t *>(w)[base + e];
            else
                h[e] = float_to_bf16_bits(reinterpret_cast<const float *>(w)[base + e]);
        }
        packed[slot] = u32x4{h[0] | (h[1] << 16), h[2] | (h[3] << 16), h[4] | (h[5] << 16), h[6] | (h[7] << 16)};
    }
}

// ---- 4-bit group-wise weights -------------------------------------------------------------
// Packed order: step s of tile t is 1056 contiguous bytes: 16 rows x 128 k of codes (lane
// l = 16*g + i holds row i; dword j of the lane holds k = 32 j + 8 g + e, e = 0..7, as
// code + 8 in nibble (e >> 1) + 4 (e & 1)), then the rows' 16 bf16 step sizes of this group.
constexpr int kW4StepK = 128;
constexpr int kW4StepBytes = 1056;

// One workgroup (256 threads) per 16-row tile; 16 threads per row, each owns 8 consecutive k of
// the current group, which is exactly one dword of the packed step.
template <bool SRC_BF16>
__global__ __launch_bounds__(256) void quantize_pack_w4_kernel(const void *w, long long ldw, int N, int K,
                                                               unsigned char *packed) {
    const int tid = threadIdx.x;
    const int t = blockIdx.x;
    const int S = K / kW4StepK;
    const int r = tid >> 4, c = tid & 15;
    const long long base = (long long)(t * kTileRows + r) * ldw;
    for (int s = 0; s < S; ++s) {
        float v[8];
        float amax = 0.f;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            v[e] = load_w<SRC_BF16>(w, base + (long long)s * kW4StepK + 8 * c + e);
            amax = fmaxf(amax, fabsf(v[e]));
        }
#pragma unroll
        for (int off = 8; off >= 1; off >>= 1) amax = fmaxf(amax, __shfl_xor(amax, off, 64));
        unsigned int sb = float_to_bf16_bits(__fdiv_rn(amax, 7.0f));
        float sc = bf16_bits_to_float(sb);
        if (!(sc > 0.f)) { sb = 0; sc = 0.f; }
        unsigned int word = 0;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            int code = 0;
            if (sc > 0.f) {
                float q = rintf(__fdiv_rn(v[e], sc));           // round half to even
                q = fminf(fmaxf(q, -7.f), 7.f);
                code = (int)q;
            }
            word |= (unsigned int)(code + 8) << (4 * ((e >> 1) + 4 * (e & 1)));
        }
        unsigned char *step = packed + ((long long)t * S + s) * kW4StepBytes;
        const int j = c >> 2, g = c & 3;
        reinterpret_cast<unsigned int *>(step)[(16 * g + r) * 4 + j] = word;
        if (c == 0) reinterpret_cast<uint16_t *>(step + 1024)[r] = (uint16_t)sb;
    }
}

// codes -> q[N, K] int8 row-major, step sizes -> scales[N, K / 128] bf16 (for checking)
__global__ __launch_bounds__(256) void unpack_w4_kernel(const unsigned char *packed, int N, int K, int8_t *q,
                                                        uint16_t *scales) {
    const int S = K / kW4StepK;
    const long long nwords = (long long)(N / kTileRows) * S * 256;
    for (long long idx = (long long)blockIdx.x * 256 + threadIdx.x; idx < nwords; idx += (long long)gridDim.x * 256) {
        const int wd = (int)(idx & 255);
        const long long ts = idx >> 8;
        const int s = (int)(ts % S);
        const long long t = ts / S;
        const int l = wd >> 2, j = wd & 3;
        const int g = l >> 4, i = l & 15;
        const unsigned char *step = packed + ts * kW4StepBytes;
        const unsigned int word = reinterpret_cast<const unsigned int *>(step)[wd];
        int8_t *dst = q + (t * kTileRows + i) * (long long)K + (long long)s * kW4StepK + 32 * j + 8 * g;
#pragma unroll
        for (int e = 0; e < 8; ++e) dst[e] = (int8_t)((int)((word >> (4 * ((e >> 1) + 4 * (e & 1)))) & 15u) - 8);
        if (wd < kTileRows)
            scales[(t * kTileRows + wd) * (long long)S + s] = reinterpret_cast<const uint16_t *>(step + 1024)[wd];
    }
}

}  // namespace quasar
