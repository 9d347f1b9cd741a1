// CPU model of the sampler's draw: the workgroup's prefix sum as the GPU adds it (a shuffle scan in each wave of 64, the wave
// totals in order), then the library's own choice of the owner and its walk.
#include "../paper_2603_01399_amd/csrc/draw.hpp"

#include <vector>

using namespace quasar;

// The draw among n masses that 1024 threads share in stretches of whole units; returns the element, *rest: what is left of the
// target inside it.
extern "C" int draw_model(const float *mass, int n, int unit, float u, float *rest) {
    constexpr int kWaves = 16, kThreads = 64 * kWaves;
    const int units = n / unit, per = (units + kThreads - 1) / kThreads;
    std::vector<float> sum(kThreads, 0.f);
    auto lo = [&](int t) { return unit * (t * per < units ? t * per : units); };
    for (int t = 0; t < kThreads; ++t)
        for (int i = lo(t); i < lo(t + 1); ++i) sum[t] += mass[i];
    float incl[kWaves][64], before[kWaves + 1] = {0.f};
    for (int w = 0; w < kWaves; ++w) {
        float v[64], next[64];
        for (int l = 0; l < 64; ++l) v[l] = sum[64 * w + l];
        for (int off = 1; off < 64; off <<= 1) {
            for (int l = 0; l < 64; ++l) next[l] = l >= off ? v[l] + v[l - off] : v[l];
            for (int l = 0; l < 64; ++l) v[l] = next[l];
        }
        for (int l = 0; l < 64; ++l) incl[w][l] = before[w] + v[l];
        before[w + 1] = before[w] + v[63];
    }
    const float total = before[kWaves], target = draw_point(u, total);
    int owners = 0, at = -1;
    for (int w = 0; w < kWaves; ++w) {
        if (!draw_in_wave(before[w], before[w + 1], target)) continue;
        ++owners;
        unsigned long long some = 0, reach = 0;
        for (int l = 0; l < 64; ++l) {
            if (sum[64 * w + l] > 0.f) some |= 1ull << l;
            if (sum[64 * w + l] > 0.f && incl[w][l] > target) reach |= 1ull << l;
        }
        const int l = draw_lane(reach, some), t = 64 * w + l;
        float run = l > 0 ? incl[w][l - 1] : before[w];
        at = draw_walk(lo(t), lo(t + 1), target, run, [&](int i) { return mass[i]; });
        *rest = target - run;
    }
    return owners <= 1 ? at : -2;
}
