// Choosing where a draw falls among masses whose prefix sums come from a parallel scan.  Plain C++ for both sides: the sampler
// (sample.hpp) runs it on the GPU, the tests run the same functions on the CPU behind a model of the scan.
//
// A scan adds the same masses in another tree for every element, so its fp32 sums are not monotone: a sum may lie a few last
// places below the one in front of it, and an element without mass may seem to reach beyond the target.  What is monotone
// is the sequence of sums in front of the waves - their totals are added one after the other - so exactly one wave covers a
// target in [0, total); inside it the FIRST element that has mass and reaches beyond the target owns the draw and, where
// rounding leaves none, the last that has mass.
#pragma once

#if defined(__HIPCC__)
#define QUASAR_BOTH __host__ __device__ __forceinline__
#else
#define QUASAR_BOTH inline
#endif

namespace quasar {

// The point of the total mass that the number u in [0, 1) names: in [0, total) also where the product rounds up (total > 0).
QUASAR_BOTH float draw_point(float u, float total) {
    float t = u * total;
    if (!(t < total)) t = total * (1.f - 1.f / 16777216.f);
    return t > 0.f && t < total ? t : 0.f;
}

// Whether a wave covers the target: before, the sum of the waves in front of it; behind, that sum and its own total.
QUASAR_BOTH bool draw_in_wave(float before, float behind, float target) { return before <= target && target < behind; }

// The lane of the covering wave that owns the draw.  reach: its lanes with mass whose inclusive sum lies beyond the target;
// mass: those with mass (at least one, or the wave would cover nothing).
QUASAR_BOTH int draw_lane(unsigned long long reach, unsigned long long mass) {
    return reach ? __builtin_ctzll(reach) : 63 - __builtin_clzll(mass);
}

// The owner's walk over its elements lo .. hi - 1: the first with mass whose running sum lies beyond the target, else the last
// with mass; -1: none has mass.  run: the sum in front of lo, on return that in front of the element.
template <class Mass>
QUASAR_BOTH int draw_walk(int lo, int hi, float target, float &run, Mass mass) {
    int at = -1;
    float sum = run;
    for (int i = lo; i < hi; ++i) {
        const float v = mass(i);
        if (!(v > 0.f)) continue;
        at = i;
        run = sum;
        sum += v;
        if (sum > target) break;
    }
    return at;
}

}  // namespace quasar
