// Launch helpers shared by the translation units of the library.
#pragma once

#include "../../include/quasar.h"

#include <hip/hip_runtime.h>

#include <mutex>
#include <type_traits>
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
int launch(KernelT kernel, dim3 grid, int block, int lds_bytes, hipStream_t stream, const GemmParams &p) {
    if (lds_bytes > kMaxLds) return QUASAR_ERR_SHAPE;
    if (!allow_large_lds(reinterpret_cast<const void *>(kernel))) return QUASAR_ERR_HIP;
    hipLaunchKernelGGL(kernel, grid, dim3(block), lds_bytes, stream, p);
    return hipGetLastError() == hipSuccess ? QUASAR_OK : QUASAR_ERR_HIP;
}

// ---- the kernels that hold the activations in registers (stream_direct*.hpp) ----

// lanes i of every row of 16 <- lanes (i + 8) mod 16
__device__ __forceinline__ u32x4 rotate_half_row(const u32x4 v) {
    u32x4 r;
    r.x = __builtin_amdgcn_update_dpp(0, (int)v.x, 0x128, 0xf, 0xf, true);
    r.y = __builtin_amdgcn_update_dpp(0, (int)v.y, 0x128, 0xf, 0xf, true);
    r.z = __builtin_amdgcn_update_dpp(0, (int)v.z, 0x128, 0xf, 0xf, true);
    r.w = __builtin_amdgcn_update_dpp(0, (int)v.w, 0x128, 0xf, 0xf, true);
    return r;
}


// A wave's range of K, `cnt` slots from `first` on, of MP token rows into its LDS region, in whole cache lines and as many of them in
// a row as a power of two allows: with one line of each of eight rows an instruction's lines, some KB apart, meet in one cache
// channel (4096 x 4096 at M = 8 6.5 -> 5.8 us, 1024 x 4096 5.1 -> 4.7, at M = 16 4096 x 12288 15.6 -> 14.7).  The addresses take one
// multiplication a wave and four additions a load (a division a load, for row segments as long as the range, cost 4096 x 6144
// 0.2 us).  Piece c of slot i of row t lies at piece c ^ (t & 7) of its slot: the lanes that read one column of pieces meet
// different banks.  Slots beyond `last` repeat it.
template <int SLOT>
constexpr int fetch_segment(int cnt) {               // slots of a row that an instruction takes
    int seg = 1;
    while (cnt % (2 * seg) == 0 && 2 * seg * SLOT <= 1024) seg *= 2;
    return seg;
}
template <int MP, int SLOT>
__device__ __forceinline__ void fetch_rows(const uint16_t *x, long long ldx, int M, int first, int last, int cnt, unsigned int lds_base, int lane) {
    constexpr int PS = SLOT / 16;
    const int seg = fetch_segment<SLOT>(cnt), rows = 64 / (PS * seg);
    const unsigned long long xa = reinterpret_cast<unsigned long long>(x);
    const unsigned int ld2 = (unsigned int)(2 * ldx), end = (unsigned int)(M - 1) * ld2;
    const int t0 = lane / (PS * seg), sl = (lane / PS) % seg;
    const unsigned int row0 = (unsigned int)t0 * ld2, c16 = (unsigned int)(((lane % PS) ^ t0) * 16);
#pragma unroll
    for (int i = 0; i < cnt / seg; ++i) {
        const unsigned int slot = (unsigned int)(min(first + i * seg + sl, last) * SLOT);
#pragma unroll
        for (int j = 0; j < MP / rows; ++j)
            load_to_lds_16(xa, min(row0 + (unsigned int)(j * rows) * ld2, end) + slot + (c16 ^ (unsigned int)(((j * rows) & 7) * 16)),
                           lds_base + 1024 * (i * (MP / rows) + j));
    }
}
// where piece c of slot i of row t lies, in bytes
template <int MP, int SLOT>
__device__ __forceinline__ int row_piece(int t, int i, int c, int cnt) {
    const int seg = fetch_segment<SLOT>(cnt), rows = 1024 / (SLOT * seg);
    return 1024 * ((i / seg) * (MP / rows) + t / rows) + ((t % rows) * seg + i % seg) * SLOT + ((c ^ (t & 7)) * 16);
}

// Waves of a workgroup by form (XS slots of 64 k per wave): where the activations take more than about half of a wave's
// 128 registers, eight waves of 256 - the ring, the accumulators and the addresses are then paid for half as often.
constexpr int direct_waves(int MP, int XS) { return MP == 32 || (MP == 16 && XS > 8) ? 8 : 16; }

// Slots of activations that pass through a wave's LDS region at a time (0: straight into registers).  Up to 48 KB of x a
// workgroup the gather of 16-byte pieces is as fast; beyond that the direct-to-LDS path, whose instructions read whole
// cache lines (fetch_rows), is.  128 KB a workgroup at most.
constexpr int direct_pass(int MP, int XS) {
    if (MP == 8 && XS <= 3) return 0;
    const int fit = 1024 / (direct_waves(MP, XS) * MP);
    return XS < fit ? XS : fit;
}
// LDS of the waves' regions (C chunks of partial tiles, two tiles' worth)
constexpr int direct_region_bytes(int MP, int XS, int C) {
    const int x = direct_pass(MP, XS) * MP * 128, tiles = 2 * C * (MP == 32 ? 2 : 1) * 1024;
    return direct_waves(MP, XS) * (x > tiles ? x : tiles);
}

// LDS of the waves' regions in the pair form of several chunks (32 tokens)
constexpr int direct_pair_bytes(int XS, int C, bool w16) {
    const int x = w16 ? 0 : direct_pass(32, XS) * 32 * 128, tiles = (C > 4 ? 1 : 2) * C * 2048;
    return 8 * (x > tiles ? x : tiles);
}

// The same for the 4-bit kernel (slots of 128 k): its waves, the slots that pass through LDS at a time, the regions.
constexpr int w4_waves(int MP, int XS) { return MP == 32 || (MP == 16 && XS > 4) ? 8 : 16; }
constexpr int w4_pass(int MP, int XS) {
    if (MP == 8 && XS <= 1) return 0;
    const int fit = 512 / (w4_waves(MP, XS) * MP);
    return XS < fit ? XS : fit;
}
constexpr int w4_region_bytes(int MP, int XS) {
    const int x = w4_pass(MP, XS) * MP * 256, tiles = 2 * (MP == 32 ? 2 : 1) * 1024;
    return w4_waves(MP, XS) * (x > tiles ? x : tiles);
}

// The W8A8 kernel (16 waves): whether the raw activations of a form stay in registers between the maximum and the codes (else
// they are read again), the slots that pass through LDS at a time on their way there, the regions.
constexpr bool a8_hold(int MP, int XS) { return XS * MP <= (MP == 8 ? 96 : 80) && MP != 32; }
constexpr int a8_pass(int MP, int XS) {
    if (!a8_hold(MP, XS) || (MP == 8 && XS <= 3)) return 0;
    return XS <= (MP == 8 ? 6 : 4) ? XS : (XS + 1) / 2;
}
constexpr int a8_region_bytes(int MP, int XS) {
    const int x = a8_pass(MP, XS) * MP * 128, tiles = 2 * (MP == 32 ? 2 : 1) * 1024;
    return 16 * (x > tiles ? x : tiles);
}

// What a kernel needs ahead of its first load, pinned so that it comes in one trip to the kernel arguments; the compiler otherwise loads
// each value in front of its first use, up to four trips one after the other.  That, the divisions of the tile shares and those
// of a K split (now a dimension of the grid) were why the last wave of a workgroup reached its first load 1.3 us after
// the kernel began (the first one 0.2 us: the set-up runs side by side, four waves to a SIMD).  us a launch, HBM-cold, one after the other,
// before -> so: int8, M = 8 1024 x 4096 4.89 -> 4.50, 4096 x 4096 5.69 -> 5.32, 12288 x 4096 10.54 -> 10.20; 4-bit 4096 x 4096 5.15 -> 4.87;
// W8A8 4096 x 4096 6.86 -> 6.65; bf16 1024 x 4096 6.33 -> 6.21.
// (one statement: in several, the loads of the later ones wait for the first.  What the kernel itself needs, then what its tile
// share does; constants need no register)
template <class Share, class A, class B, class C, class D, class E, class F = int, class G = int, class H = int, class I = int>
__device__ __forceinline__ void loaded_together(const GemmParams &p, A a, B b, C c, D d, E e, F f = 0, G g = 0, H h = 0, I i = 0) {
    constexpr bool deal = Share::kDeal;
    asm volatile("" ::"s"(a), "s"(b), "s"(c), "s"(d), "s"(e), "is"(f), "is"(g), "is"(h), "is"(i), "s"(p.tq), "s"(p.tr), "is"(deal ? p.groups : 0),
                 "is"(deal ? p.xcd_shift : 0));
}

// formats of weights and activations
enum { FMT_INT8 = 0, FMT_BF16 = 1, FMT_W4 = 2, FMT_A8 = 3 };

// Whether the workgroups of a register-resident form (XS slots a wave of NW) are dealt their tiles (TileShare).  Contiguous shares keep
// 256 streams some MB apart open, which costs address translation and leaves some XCDs behind the others by a tenth of a
// long stream.  us, contiguous, dealt, M = 8 unless said: vocabulary of 151936, K = 4096, int8 104.0, 98.5, W8A8 104.5, 97.9, bf16 195.6,
// 187.2, 4-bit 56.7, 53.6, K = 2560 int8 67.7, 62.2, 4-bit 43.7, 44.4 (K = 3072 50.0, 46.3); int8 12288 x 4096 10.24, 10.03, 65536 x 3072 34.7,
// 31.4, 25600 x 5120 22.6, 22.1, M = 32 26.6, 26.2, 16384 x 8192 23.4, 23.8, M = 32 28.9, 27.5; bf16 12288 x 4096 17.6, 16.9, 16384 x 8192
// 42.6, 41.4, 12288 x 4096 M = 32 19.5, 19.0.  One or two tiles a workgroup are the same either way (int8 4096 x 4096 5.35, 5.36), but int8
// and W8A8 of K just over 2048, up to 8 tokens: 8192 x 2112 6.26, 6.28, M = 1 5.36, 5.58, 16384 x 2112 W8A8 9.4, 9.9.
// Short K, where a tile is a slot or two a wave, stays contiguous: int8 16384 x 1024 6.75, 7.25, 20480 x 2048 9.27, 9.44 (a
// vocabulary of 100000 38.6, 36.2), bf16 16384 x 1024 8.53, 8.81, 65536 x 2048 40.4, 42.1.  4-bit linears too, but those of 9 to 16 tokens and two
// slots (25600 x 4096 13.25, 13.14, 10240 x 3072 7.95, 7.88): M = 1 12288 x 4096 7.98, 8.21, 25600 x 4096 11.83, 12.07, M = 8 12.15, 12.25, M = 32
// 16.1, 16.1, and of three slots and more 8192 x 8192 9.8, 10.6, 16384 x 8192 14.6, 15.1, 25600 x 5120 15.8, 15.4.
constexpr bool deal_tiles(int fmt, int MP, int NW, int XS, bool argmax) {
    const int k = (fmt == FMT_W4 ? 128 : 64) * NW * XS;      // the longest K of the form
    if (fmt == FMT_W4) return k > 2048 && (argmax || (MP == 16 && XS == 2));
    return k > 2048 || (argmax && fmt != FMT_BF16 && k > 1024);
}

// ---- the kernel with K outermost (stream_outer.hpp): FMT_A8 and FMT_W4 ----
// tiles a workgroup walks side by side, at most (4-bit weights, 9 to 16 tokens: seven spill 44 registers)
constexpr int outer_tiles(int fmt, int MP) { return fmt == FMT_W4 && MP == 16 ? 6 : 8; }
constexpr int outer_waves(int MP) { return MP == 32 ? 8 : 16; }             // (32 tokens: 256 registers a wave)
constexpr int outer_slot_k(int fmt) { return fmt == FMT_W4 ? 128 : 64; }    // k of a slot
// 16-byte loads of activations a lane and slot
constexpr int outer_x_loads(int fmt, int MP) { return fmt == FMT_A8 ? (MP == 32 ? 2 : 1) : MP / 4; }
// passes the weights are requested ahead: six to ten slots in flight a wave, in powers of two so that shares of 4 and 8 slots
// are whole rounds
constexpr int outer_depth(int fmt, int MP, int NT) {
    if (fmt == FMT_W4) return NT == 1 ? (MP == 32 ? 4 : 2) : (NT <= 3 ? 2 : 1);
    return NT <= 2 ? 4 : (NT <= (MP == 32 ? 6 : 4) ? 2 : 1);
}
constexpr int outer_lds_bytes(int MP, int NT) { return outer_waves(MP) * NT * (MP == 32 ? 2 : 1) * 1024; }

struct DirectPlan {
    int XS, SC, C, ksplit, slice_steps, groups, sc_bytes, lds_bytes;
    bool pair;       // 32 tokens in the order of sixteen waves
};

// p: as for the other kernels (its step counts are replaced by slots of 64 k).  epi, pre, resid: EPI_*, PRE_* and whether a
// residual is added.
int launch_direct_int8(int epi, int pre, bool resid, const GemmParams &p, int MP, const DirectPlan &d, hipStream_t stream);
int launch_direct_bf16(int epi, const GemmParams &p, int MP, const DirectPlan &d, hipStream_t stream);

int launch_direct_w8a8(int epi, const GemmParams &p, int MP, const DirectPlan &d, hipStream_t stream);

int launch_outer_w4(const GemmParams &p, int MP, const DirectPlan &d, hipStream_t stream);
int launch_quantize_operand(const GemmParams &p, int MP, unsigned char *codes, float *dx, hipStream_t stream);
int launch_outer_w8a8(const GemmParams &p, int MP, const DirectPlan &d, hipStream_t stream);

int launch_direct_w4(int epi, const GemmParams &p, int MP, const DirectPlan &d, hipStream_t stream);

inline int launch_direct(bool w16, int epi, int pre, bool resid, const GemmParams &p, int MP, const DirectPlan &d, hipStream_t stream) {
    return w16 ? launch_direct_bf16(epi, p, MP, d, stream) : launch_direct_int8(epi, pre, resid, p, MP, d, stream);
}

}  // namespace quasar
