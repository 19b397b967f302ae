// split.hpp -- how a persistent launch splits its walks over wavefronts and
// lanes: plain arithmetic, the same on the host, in kernels and in a CPU build.
#pragma once

#include <stdint.h>

namespace n2v {

constexpr uint32_t SPLIT_LANES = 64;  // lanes of a wavefront
constexpr uint32_t SPLIT_WAVES = 4;   // wavefronts of a workgroup
constexpr uint32_t POOL = 256;        // most walks a wavefront claims per atomic

// Workgroups of a launch of `walks` walks, at most `blocks` of them.  Small
// jobs: down to a wavefront per walk.  Past a walk per wavefront, a job with
// hardly any hub moves fills its lanes first (but for two wavefronts per SIMD,
// which hide each other's latency): rounds with part of the lanes cost as many
// instructions (112,086 walks on WeC-16, mean degree 100: spread over all the
// wavefronts that fit 1.01 ms, so 0.84; with weights, WeC-15, 2.01 and 1.80
// ms).  The wavefronts that hold the remainder are counted in: one walk past
// the lanes would wait for a whole other walk.
constexpr uint32_t split_blocks(uint64_t walks, uint64_t blocks, uint32_t cus, bool few_hubs)
{
    uint64_t waves = walks;
    if (few_hubs && walks > blocks * SPLIT_WAVES) {
        waves = (walks + SPLIT_LANES - 1) / SPLIT_LANES;
        if (waves < 8ull * cus) waves = 8ull * cus;
    }
    const uint64_t need = (waves + SPLIT_WAVES - 1) / SPLIT_WAVES;
    if (blocks > need) blocks = need;
    return blocks < 1 ? 1u : (uint32_t)blocks;
}

// Walks of the fullest of nwaves wavefronts when `total` are given out evenly.
constexpr uint32_t split_share(uint32_t total, uint32_t nwaves)
{
    return total / nwaves + (total % nwaves ? 1u : 0u);
}

// Lanes of a wavefront that take walks, for a fullest share of `share` walks.
// Where hub moves are common a wavefront makes them one after the other: the
// walks that share it wait for each other, and a wavefront that meets many
// holds up the launch's end.  So the more of the entries lie in hub rows
// (lane_div), the smaller a part of its walks a wavefront starts at once
// (eight where it has eight); the rest go to whoever is free.  Measured with
// all walks started by index / half / a quarter / an eighth of them: 48 walks
// per wavefront at scale 18 without sketches 34.8 / 34.2 / 29.2 / 28.6 ms, 8
// per wavefront at scale 16 1.41 / 1.38 / 1.43 / 1.61 ms.
constexpr uint32_t walk_lanes(uint32_t lane_div, uint32_t share)
{
    const uint32_t part = (share + lane_div - 1) / lane_div;
    return share < 8u || part > SPLIT_LANES ? SPLIT_LANES : (part < 8u ? 8u : part);
}

// Walks each of nwaves wavefronts takes by its own index; 0: all of them are
// given out so, evenly, which is only done where every wavefront starts its
// whole share at once.  (Lanes for the share rounded down left a remainder
// walk to run alone after the others: 110,592 walks on ER-18, 54 a wavefront,
// 0.60 ms, 112,086 0.83 ms, now 0.60; with weights, WeC-15, 1.78, 2.42, 1.79 ms.)
constexpr uint32_t first_share(uint32_t lane_div, uint32_t total, uint32_t nwaves, uint32_t lanes)
{
    if (lanes >= split_share(total, nwaves)) return 0;
    const uint32_t q = total / nwaves;
    return lane_div > 1 ? lanes : (q < POOL ? q : POOL);
}

// A walk alone on its wavefront lasts as long as its chain of attempts: under
// the default option the wavefront makes 64 of a move at once (t_wave 0; 1000
// walks of 40 moves on ER-20: 139 -> 75 us).  Not where hubs are common, whose
// lines the other 60 attempts' reads push out (100 walks at scale 16: 165
// against 194 us).  Any other t_wave is the caller's, and stays.
constexpr uint32_t T_WAVE_DEFAULT = 1024;

constexpr bool lone_walks(uint32_t walks, uint32_t blocks, uint32_t lane_div)
{
    return lane_div == 1 && walks <= blocks * SPLIT_WAVES;
}

constexpr uint32_t launch_t_wave(uint32_t t_wave, bool lone)
{
    return lone && t_wave == T_WAVE_DEFAULT ? 0u : t_wave;
}

}  // namespace n2v
