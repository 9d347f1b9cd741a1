// Stochastic verification at temperature T > 0 on the fp32 logits of the M positions (gfx950):
// softmax statistics per position, the acceptance test r < min(1, p/q) against a deterministic
// drafter (q is a point mass on the proposed token), and the draw of the corrective or bonus
// token by inverse CDF in vocabulary order (Sec. 3.1, the acceptance and resampling rules;
// Sec. 3.3 "Lossless Rejection Sampling").  The logits come from the streaming kernel's fp32
// epilogue: [M, V] fp32 is a few MB beside the hundreds of MB of weights it was computed from.
//
// The vocabulary is cut into contiguous blocks of whole 16-row tiles.  Where the streaming kernel keeps its activations in
// registers its workgroups are the blocks and leave (max, sum of exp(z - max)) per position beside the logits they write;
// otherwise softmax_partial_kernel takes the statistics of kSampleBlocks blocks from the finished logits.
// speculative_sample_kernel (one workgroup) merges them, takes the acceptance decisions, locates the block in which the draw
// falls from the block masses and resolves the draw inside that block only.  What bounds it is a chain of dependent steps,
// so each of them is spread over the workgroup: statistics merged by 32 lanes a position, block masses and the stretch of the
// chosen block by prefix sums over all threads (a serial walk by one thread before).  After the logits of V = 151936, M = 8:
// two launches of 5.5 and 14 us before, now one of 6.6 us.
#pragma once

#include "quasar_device.hpp"
#include "stream_gemm.hpp"

namespace quasar {

constexpr int kSampleBlocks = 32;

// first quad of block b of nblk
__device__ __forceinline__ int sample_block_begin(int V, int b, int nblk) { return 4 * tile_split(V / kTileRows, b, nblk); }

// grid (kSampleBlocks, M), 256 threads.  partial[(m * kSampleBlocks + b) * 2] = max of z over the
// block, [.. + 1] = sum of exp(z - max); z = logit * inv_t.  V is a multiple of 16: rows are read
// as 16-byte quads.
__global__ __launch_bounds__(256) void softmax_partial_kernel(const float *logits, int V, float inv_t,
                                                             float *partial) {
    __shared__ float sm[4], ss[4];
    const int b = blockIdx.x, m = blockIdx.y, tid = threadIdx.x;
    const f32x4 *row4 = reinterpret_cast<const f32x4 *>(logits + (long long)m * V);
    const int q_lo = sample_block_begin(V, b, kSampleBlocks), q_hi = sample_block_begin(V, b + 1, kSampleBlocks);
    float mx = -__builtin_inff(), s = 0.f;
    for (int q0 = q_lo + tid; q0 < q_hi; q0 += 256 * 4) {
        f32x4 v[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int q = q0 + 256 * j;
            v[j] = q < q_hi ? row4[q] : f32x4{-__builtin_inff(), -__builtin_inff(), -__builtin_inff(), -__builtin_inff()};
        }
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            softmax_add(mx, s, v[j].x * inv_t, v[j].y * inv_t, v[j].z * inv_t, v[j].w * inv_t);
        }
    }
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) {
        const float m2 = __shfl_xor(mx, off, 64), s2 = __shfl_xor(s, off, 64);
        softmax_merge(mx, s, m2, s2);
    }
    if ((tid & 63) == 0) { sm[tid >> 6] = mx; ss[tid >> 6] = s; }
    __syncthreads();
    if (tid == 0) {
        float M0 = sm[0], S0 = ss[0];
        for (int w = 1; w < 4; ++w) softmax_merge(M0, S0, sm[w], ss[w]);
        partial[((long long)m * kSampleBlocks + b) * 2] = M0;
        partial[((long long)m * kSampleBlocks + b) * 2 + 1] = S0;
    }
}

// Inclusive prefix sum over the workgroup's 1024 threads (fixed order); total: the sum over all.
__device__ __forceinline__ float block_scan(float v, float *wave_tot, float &total) {
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const float t = __shfl_up(v, off, 64);
        if (lane >= off) v += t;
    }
    if (lane == 63) wave_tot[wv] = v;
    __syncthreads();
    float base = 0.f;
    total = 0.f;
#pragma unroll
    for (int i = 0; i < 16; ++i) {
        if (i < wv) base += wave_tot[i];
        total += wave_tot[i];
    }
    __syncthreads();
    return base + v;
}

// One workgroup of 1024 threads.  partial: [M][nblk] (max, sum of exp(z - max)).
__global__ __launch_bounds__(1024) void speculative_sample_kernel(const float *logits, int V, int M, float inv_t, int nblk,
                                                                 const int32_t *draft, int n_draft,
                                                                 const float *u_accept, const float *u_sample,
                                                                 const float *partial, int32_t *out_accept,
                                                                 int32_t *out_token, float *out_p_draft) {
    __shared__ float pos_max[32], pos_pd[32], pos_zd[32], pos_ua[32], pos_us[32];
    __shared__ int pos_draft[32];
    __shared__ float part[1024];
    __shared__ float wave_tot[16];
    __shared__ int blk_s, chunk_s;
    __shared__ float target_s;
    const int tid = threadIdx.x, lane = tid & 63;
    // per position: 32 lanes merge the block statistics; p of the proposed token
    {
        const int m = tid >> 5, j = tid & 31;
        float mx = -__builtin_inff(), s = 0.f, zd = -__builtin_inff();
        if (m < M && j == 0) pos_us[m] = u_sample[m];
        if (m < n_draft && j == 0) {
            const int d = draft[m];
            pos_draft[m] = d;
            if (d >= 0 && d < V) zd = logits[(long long)m * V + d] * inv_t;
            pos_ua[m] = u_accept[m];
        }
        // (eight statistics requested at a time; the maximum over all lanes first, then every sum once against it)
        const u32x2 *row = reinterpret_cast<const u32x2 *>(partial) + (long long)min(m, M - 1) * nblk;
        for (int b = j; b < nblk; b += 256) {
            u32x2 v[8];
#pragma unroll
            for (int i = 0; i < 8; ++i) v[i] = row[min(b + 32 * i, nblk - 1)];
            float m8 = mx;
#pragma unroll
            for (int i = 0; i < 8; ++i) m8 = fmaxf(m8, __uint_as_float(v[i].x));
            if (m8 > -__builtin_inff()) {
                s *= expf(mx - m8);
#pragma unroll
                for (int i = 0; i < 8; ++i)
                    if (b + 32 * i < nblk) s += __uint_as_float(v[i].y) * expf(__uint_as_float(v[i].x) - m8);
                mx = m8;
            }
        }
        float all = mx;
#pragma unroll
        for (int off = 16; off >= 1; off >>= 1) all = fmaxf(all, __shfl_xor(all, off, 64));
        s = mx > -__builtin_inff() ? s * expf(mx - all) : 0.f;
        mx = all;
#pragma unroll
        for (int off = 16; off >= 1; off >>= 1) s += __shfl_xor(s, off, 64);
        if (m < M && j == 0) {
            float pd = 0.f;
            if (m < n_draft) {
                if (zd > -__builtin_inff()) pd = expf(zd - mx) / s;
                if (out_p_draft) out_p_draft[m] = pd;
            }
            pos_zd[m] = zd;
            pos_max[m] = mx;
            pos_pd[m] = pd;
        }
    }
    __syncthreads();
    // leading accepted candidates (every wave for itself): q(x~) = 1
    const bool ok = lane < n_draft && pos_ua[lane & 31] < fminf(1.f, pos_pd[lane & 31]);
    const int pos = __builtin_ctzll(~__builtin_amdgcn_ballot_w64(ok));
    const float mx = pos_max[pos];
    const int banned = pos < n_draft ? pos_draft[pos] : -1;
    {
        // the draw at that position: masses of the blocks, the rejected token's mass removed (max(0, p - q) is 0 on the
        // proposed token and p elsewhere); each thread owns `per` neighbouring blocks
        const bool ban = banned >= 0 && banned < V;
        const float ban_mass = ban ? expf(pos_zd[pos] - mx) : 0.f;
        const int per = (nblk + 1023) / 1024;
        const int b0 = min(nblk, tid * per), b1 = min(nblk, b0 + per);
        auto mass = [&](int b) {
            const float pm = partial[((long long)pos * nblk + b) * 2];
            float v = pm > -__builtin_inff() ? partial[((long long)pos * nblk + b) * 2 + 1] * expf(pm - mx) : 0.f;
            if (ban && banned / 4 >= sample_block_begin(V, b, nblk) && banned / 4 < sample_block_begin(V, b + 1, nblk))
                v = fmaxf(0.f, v - ban_mass);
            return v;
        };
        float sum = 0.f;
        for (int b = b0; b < b1; ++b) sum += mass(b);
        float total;
        const float incl = block_scan(sum, wave_tot, total);
        part[tid] = incl;
        if (tid == 0) {
            out_accept[0] = pos;
            blk_s = -1;
            chunk_s = 1023;
        }
        __syncthreads();
        float target = pos_us[pos] * total;
        if (!(target < total)) target = total * (1.f - 1.f / 16777216.f);     // u * total rounded up to the total
        const float before = tid > 0 ? part[tid - 1] : 0.f;
        // the first thread whose blocks reach beyond the target; past them all through rounding: the last with mass
        if (incl > target && (tid == 0 || !(before > target))) {
            float run = before;
            int blk = b0;
            for (; blk + 1 < b1; ++blk) {
                const float v = mass(blk);
                if (run + v > target) break;
                run += v;
            }
            blk_s = blk;
            target_s = target - run;            // what is left to cover inside the block
        }
        __syncthreads();
        const bool none = blk_s < 0;
        __syncthreads();
        if (none) {
            if (sum > 0.f) atomicMax(&blk_s, b1 - 1);
            __syncthreads();
            if (tid == 0) {
                if (blk_s < 0) blk_s = 0;
                target_s = total;
            }
            __syncthreads();
        }
    }
    const int blk = blk_s;
    const float *row = logits + (long long)pos * V;
    // inside the block: contiguous stretches of quads per thread, prefix sums in vocabulary order
    const int q_lo = sample_block_begin(V, blk, nblk), q_hi = sample_block_begin(V, blk + 1, nblk);
    const int per = (q_hi - q_lo + 1023) / 1024;                  // quads per thread
    const int a0 = min(q_hi, q_lo + tid * per), a1 = min(q_hi, a0 + per);
    const f32x4 *row4 = reinterpret_cast<const f32x4 *>(row);
    float sum = 0.f;
    const f32x4 head = a0 < a1 ? row4[a0] : f32x4{0.f, 0.f, 0.f, 0.f};
    for (int q = a0; q < a1; ++q) {
        const f32x4 v = q == a0 ? head : row4[q];
        const float z4[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
        for (int e = 0; e < 4; ++e)
            if (4 * q + e != banned) sum += expf(z4[e] * inv_t - mx);
    }
    float total;
    const float incl = block_scan(sum, wave_tot, total);
    part[tid] = incl;
    float target = target_s;
    if (!(target < total)) target = total * (1.f - 1.f / 16777216.f);   // block mass and in-block sum differ by rounding
    if (target < 0.f) target = 0.f;
    __syncthreads();
    if (incl > target && (tid == 0 || !(part[tid - 1] > target))) chunk_s = tid;
    __syncthreads();
    if (tid == chunk_s) {
        float run = tid > 0 ? part[tid - 1] : 0.f;
        int tok = -1, last = -1;
        for (int q = a0; q < a1 && tok < 0; ++q) {
            const f32x4 v = q == a0 ? head : row4[q];
            const float z4[4] = {v.x, v.y, v.z, v.w};
            for (int e = 0; e < 4; ++e) {
                if (4 * q + e == banned) continue;
                const float ex = expf(z4[e] * inv_t - mx);
                if (ex > 0.f) last = 4 * q + e;
                run += ex;
                if (run > target) { tok = 4 * q + e; break; }
            }
        }
        if (tok < 0) tok = last;            // rounding at the very end of the stretch
        if (tok < 0) tok = a1 > a0 ? 4 * a1 - 1 : V - 1;
        out_token[0] = tok;
    }
}

}  // namespace quasar
