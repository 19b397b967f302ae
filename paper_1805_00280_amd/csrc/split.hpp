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

// Whether a plain superstep may make its hub moves itself, each with one
// wavefront: where they are rare (lane_div 1), and either the caller left t_wg
// at its default or no row can be longer than it (a longer one alone would have
// more entries than all hub rows).  At the default even long rows are better
// off so: walks of 40 moves from one of two adjacent hubs of 300,000, 100 / 5000
// / 60,000 of them, 0.33 / 0.49 / 3.13 ms against 0.59 / 0.85 / 3.50 ms queued.
// A t_wg of the caller's own asks for workgroups, which take queued moves.
constexpr uint32_t T_WG_DEFAULT = 65536;

constexpr bool plain_may_fuse(uint32_t lane_div, uint32_t t_wg, uint64_t hub_entries)
{
    return lane_div == 1 && (t_wg == T_WG_DEFAULT || hub_entries <= t_wg);
}

// Lanes that make a walk's attempts in a superstep of the plain form, and
// whether the superstep makes its hub moves in the same launch.
struct PlainSplit {
    int lanes;
    bool fused;
};

// A superstep lasts as long as its slowest chain of dependent reads: while
// the walks fill no more than the chip's 32 wavefronts per CU with 64 (8, 4)
// lanes each, as many take a walk's attempts.  Where hub moves are rare
// those wavefronts make them too, and the superstep is one launch (40,960
// walks of 80 moves at scale 12: 2.33 -> 1.35 ms; 10,000 of 40 on ER-18 0.70
// -> 0.28 ms).  Where they are common they are queued, each wavefront's with
// one atomic on the queue's counter, so groups pay off only for fewer
// walks: 1 / 4 / 8 / 64 lanes measured 2.98 / 2.62 / 2.84 / 3.40 ms for
// 20,000 walks at scale 16, 9.1 / 10.2 / 11.6 / 14.5 ms for 100,000, 2.47 /
// 1.87 / 1.77 / 1.84 ms for 3000.  Counting adds each workgroup's checksum at one
// address: no more of them than a quarter of the walks' wavefronts need.
constexpr PlainSplit plain_split(uint32_t walks, uint32_t cus, bool fuse, bool counts)
{
    const uint32_t slots = cus * 32u * SPLIT_LANES;
    int lanes = fuse ? (walks <= slots / 64 ? 64 : (walks <= slots / 8 ? 8 : (walks <= slots / 2 ? 4 : 1)))
                     : (walks <= slots / 64 ? 8 : (walks <= slots / 16 ? 4 : 1));
    if (counts && lanes > 4) lanes = walks <= slots / 512 ? 8 : 4;
    return PlainSplit{lanes, fuse && lanes >= 4};
}

}  // namespace n2v
