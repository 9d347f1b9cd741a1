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
// two launches of 5.5 and 14 us before, now one of 6.0 us.
#pragma once

#include "draw.hpp"
#include "quasar_device.hpp"
#include "stream_gemm.hpp"

namespace quasar {

constexpr int kSampleBlocks = 32;

// The vocabulary's blocks of whole tiles, cut where the workgroups of the streaming kernel are (tile_split): of n blocks of T
// tiles, block b begins at tile floor(T b / n) = (T / n) b + floor((T mod n) b / n).  n is at most 4096, so the second product is below
// 2^24: its quotient is taken in fp32, one off at most, and put right.  (The general integer divisions cost the one
// workgroup that draws 0.6 us.)
struct SampleBlocks {
    int n, each, rest;
    float inv_n;
    SampleBlocks(int V, int n_) : n(n_), each((V / kTileRows) / n_), rest((V / kTileRows) % n_), inv_n(1.0f / (float)n_) {}
    __device__ __forceinline__ int tile(int b) const {
        const int x = rest * b;
        int q = (int)((float)x * inv_n);
        const int left = x - q * n;
        q += left >= n ? 1 : 0;
        q -= left < 0 ? 1 : 0;
        return each * b + q;
    }
    __device__ __forceinline__ int quad(int b) const { return kTileRows / 4 * tile(b); }
};

// grid (kSampleBlocks, M), 256 threads.  partial[(m * kSampleBlocks + b) * 2] = max of z over the
// block, [.. + 1] = sum of exp(z - max); z = logit * inv_t.  V is a multiple of 16: rows are read
// as 16-byte quads.
__global__ __launch_bounds__(256) void softmax_partial_kernel(const float *logits, int V, SampleBlocks blocks, float inv_t,
                                                             float *partial) {
    __shared__ float sm[4], ss[4];
    const int b = blockIdx.x, m = blockIdx.y, tid = threadIdx.x;
    const f32x4 *row4 = reinterpret_cast<const f32x4 *>(logits + (long long)m * V);
    const int q_lo = blocks.quad(b), q_hi = blocks.quad(b + 1);
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

// Prefix sum over the workgroup's 1024 threads (fixed order): incl, this thread's inclusive sum; before, the sum of the waves in
// front of its own; behind, that and its own wave; total.  wave_tot: 16 floats, another 16 in the next call (the barrier
// of that call is behind the reads of this one).
struct BlockSums { float incl, before, behind, total; };
__device__ __forceinline__ BlockSums block_scan(float v, float *wave_tot) {
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const float t = __shfl_up(v, off, 64);
        if (lane >= off) v += t;
    }
    if (lane == 63) wave_tot[wv] = v;
    __syncthreads();
    BlockSums s = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int i = 0; i < 16; ++i) {
        if (i == wv) s.before = s.total;
        s.total += wave_tot[i];
        if (i == wv) s.behind = s.total;
    }
    s.incl = s.before + v;
    return s;
}

// Whether this thread owns the draw at the target (draw.hpp), and the sum in front of it.
__device__ __forceinline__ bool draw_mine(float sum, const BlockSums &s, float target, float &run) {
    const int lane = threadIdx.x & 63;
    run = __shfl_up(s.incl, 1, 64);
    if (lane == 0) run = s.before;
    const unsigned long long mass = __builtin_amdgcn_ballot_w64(sum > 0.f);
    const unsigned long long reach = __builtin_amdgcn_ballot_w64(sum > 0.f && s.incl > target);
    return draw_in_wave(s.before, s.behind, target) && lane == draw_lane(reach, mass);
}

// One workgroup of 1024 threads.  partial: [M][nblk] (max, sum of exp(z - max)).
__global__ __launch_bounds__(1024) void speculative_sample_kernel(const float *logits, int V, int M, float inv_t, SampleBlocks blocks,
                                                                 const int32_t *draft, int n_draft,
                                                                 const float *u_accept, const float *u_sample,
                                                                 const float *partial, int32_t *out_accept,
                                                                 int32_t *out_token, float *out_p_draft) {
    __shared__ float pos_max[32], pos_pd[32], pos_zd[32], pos_ua[32], pos_us[32];
    __shared__ int pos_draft[32];
    __shared__ float wave_tot[2][16];
    __shared__ int blk_s, thin_s;
    __shared__ float target_s;
    const int tid = threadIdx.x, lane = tid & 63, nblk = blocks.n;
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
        if (tid == 0) blk_s = 0, thin_s = -1, target_s = 0.f;
    }
    __syncthreads();
    // leading accepted candidates (every wave for itself): q(x~) = 1
    const bool ok = lane < n_draft && pos_ua[lane & 31] < fminf(1.f, pos_pd[lane & 31]);
    const int pos = __builtin_ctzll(~__builtin_amdgcn_ballot_w64(ok));
    const float mx = pos_max[pos];
    const int banned = pos < n_draft ? pos_draft[pos] : -1;
    if (tid == 0) out_accept[0] = pos;
    const float *row = logits + (long long)pos * V;
    const f32x4 *row4 = reinterpret_cast<const f32x4 *>(row);
    auto quad_mass = [&](int q) {
        const f32x4 v = row4[q];
        return f32x4{4 * q != banned ? expf(v.x * inv_t - mx) : 0.f, 4 * q + 1 != banned ? expf(v.y * inv_t - mx) : 0.f,
                     4 * q + 2 != banned ? expf(v.z * inv_t - mx) : 0.f, 4 * q + 3 != banned ? expf(v.w * inv_t - mx) : 0.f};
    };
    // quads a0 .. a1 - 1 of the row: this thread's stretch of quads q_lo .. q_hi - 1, and its mass (first quad's kept in `head`)
    auto stretch = [&](int q_lo, int q_hi, int &a0, int &a1, f32x4 &head) {
        const int per = (q_hi - q_lo + 1023) / 1024;
        a0 = min(q_hi, q_lo + tid * per);
        a1 = min(q_hi, a0 + per);
        float sum = 0.f;
        for (int q = a0; q < a1; ++q) {
            const f32x4 e = quad_mass(q);
            if (q == a0) head = e;
            sum += (e.x + e.y) + (e.z + e.w);
        }
        return sum;
    };
    // A block among all, each thread with a stretch of neighbouring ones; the rejected token's mass is removed (max(0, p - q) is 0
    // on the proposed token and p elsewhere).
    {
        const bool ban = banned >= 0 && banned < V;
        const int ban_tile = ban ? banned / kTileRows : -1;
        const float ban_mass = ban ? expf(pos_zd[pos] - mx) : 0.f;
        const u32x2 *stats = reinterpret_cast<const u32x2 *>(partial) + (long long)pos * nblk;
        const int per = (nblk + 1023) / 1024;
        const int b0 = min(nblk, tid * per), b1 = min(nblk, b0 + per);
        int ban_blk = -1;                        // the rejected token's block, if it is this thread's, and its other mass
        float ban_left = -1.f;
        auto mass = [&](int b) {
            if (b == ban_blk) return ban_left;
            const u32x2 st = stats[b];
            const float pm = __uint_as_float(st.x);
            const float v = pm > -__builtin_inff() ? __uint_as_float(st.y) * expf(pm - mx) : 0.f;
            if (!ban || ban_tile < blocks.tile(b) || ban_tile >= blocks.tile(b + 1)) return v;
            // where the token is nearly all of its block the difference is rounding: the other tokens are added up below
            ban_blk = b;
            ban_left = fmaxf(0.f, v - ban_mass);
            if (!(ban_left > v * (1.f / 1024.f))) thin_s = b;
            return ban_left;
        };
        float sum = 0.f;
        for (int b = b0; b < b1; ++b) sum += mass(b);
        BlockSums s = block_scan(sum, wave_tot[0]);
        const int thin = thin_s;                 // (set ahead of the scan's barrier, if at all)
        if (thin >= 0) {
            int a0, a1;
            f32x4 head;
            const float left = block_scan(stretch(blocks.quad(thin), blocks.quad(thin + 1), a0, a1, head), wave_tot[1]).total;
            if (ban_blk == thin) {
                ban_left = left;
                sum = 0.f;
                for (int b = b0; b < b1; ++b) sum += mass(b);
            }
            s = block_scan(sum, wave_tot[0]);
        }
        const float target = draw_point(pos_us[pos], s.total);
        float run;
        if (draw_mine(sum, s, target, run)) {
            blk_s = b1 - b0 == 1 ? b0 : max(b0, draw_walk(b0, b1, target, run, mass));
            target_s = fmaxf(0.f, target - run);                     // what is left to cover inside the block
        }
        if (tid == 0) out_accept[0] = pos;
        __syncthreads();
    }
    // a token of that block, each thread with a stretch of its quads, in vocabulary order
    int a0, a1;
    f32x4 head = {0.f, 0.f, 0.f, 0.f};
    const float sum = stretch(blocks.quad(blk_s), blocks.quad(blk_s + 1), a0, a1, head);
    const BlockSums s = block_scan(sum, wave_tot[1]);
    // (block mass and the sum inside the block differ by rounding)
    const float target = target_s < s.total ? target_s : draw_point(1.f, s.total);
    float run;
    if (draw_mine(sum, s, target, run)) {
        const int tok = draw_walk(4 * a0, 4 * a1, target, run, [&](int i) {
            const f32x4 e = (i >> 2) == a0 ? head : quad_mass(i >> 2);
            return (i & 2) ? ((i & 1) ? e.w : e.z) : ((i & 1) ? e.y : e.x);
        });
        out_token[0] = max(tok, 4 * a0);
    }
    if (tid == 0 && !(target < s.total)) out_token[0] = V - 1;          // (no mass in the row: not finite)
}

}  // namespace quasar
