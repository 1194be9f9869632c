// Launch shapes that sums or indices of a kernel rely on, as plain host
// arithmetic (no HIP), so that their bounds can be checked without a GPU.
#pragma once

#include <algorithm>
#include <cstdint>

namespace fizi {

constexpr int kShapeWave = 64;
constexpr int kGainParts = 8192;       // partial sums of one k_gain_span launch, over all its frames

// A workgroup's sums of sampled luminance: with few parts one holds 2^23
// pixels of at most 1020 (256 frames of 8192 x 8192, every row sampled), 2^33.
using GainSum = unsigned long long;

// k_gain_span over n frames of `items` items each: `parts` workgroups of
// `threads` per frame, lane l of part p taking items p threads + l, + parts
// threads, ... (at most `rounds` of them).
struct GainShape {
    int parts, threads, rounds;
};

// Waves per frame: one item per lane, but no more than about eight waves per
// SIMD over the launch; in parts of four waves, more (up to kGainWaves) where
// 32 parts would not hold them. Over 50 frames of 1920x1080 (learning) parts
// of 4 / 8 / 16 waves take 19 / 23 / 27 us, half the waves 22. Frames too large
// for 32 parts of kGainWaves take more of these parts, up to kGainBusy waves
// over the launch, and as many rounds as remain, the same for every part: one
// frame of 7680x4320 10.4 us (27.5 in 32 parts), with every row sampled 34
// (197), one of 3840x2160 with every row 14 (52); with kGainBusy 2048 / 4096 /
// 8192 four frames of 7680x4320 28.7 / 18.7 / 20.3, eight of 3840x2160 11.6 /
// 11.5 / 13.2; parts of 4 / 8 / 16 waves, one frame of 7680x4320 20.9 / 13.5 /
// 10.4.
constexpr int kGainWaves = 16, kGainBusy = 4096;

inline GainShape gain_span_shape(long long items, int n)
{
    const int full = (int)((items + kShapeWave - 1) / kShapeWave);
    int waves_f = std::min(full, std::max(32, 8192 / n));
    if (waves_f > 32 * kGainWaves)
        waves_f = std::min(waves_f, std::max(32 * kGainWaves, kGainBusy / n));
    GainShape g;
    g.parts = std::max({1, std::min(32, (waves_f + 3) / 4), (waves_f + kGainWaves - 1) / kGainWaves});
    const int most = std::min(kGainWaves, (waves_f + g.parts - 1) / g.parts);
    g.rounds = (full + g.parts * most - 1) / (g.parts * most);
    g.threads = kShapeWave * ((full + g.parts * g.rounds - 1) / (g.parts * g.rounds));
    return g;
}

}  // namespace fizi
