"""The persistent launch's split rule (csrc/split.hpp), built for the CPU: every
walk is given out once, and a wavefront that is given its walks by index has a
lane for each of them (a walk past them would start only after the others)."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1805_00280_amd", "csrc")

DRIVER = r"""
#include <stdio.h>
#include <algorithm>
#include "split.hpp"
using namespace n2v;
int main()
{
    const uint32_t cus = 256, totals[] = {1, 3, 5, 63, 255, 1023, 1024, 2049, 4999, 5119, 5120, 5121, 6143, 6144,
        6145, 7168, 9000, 10241, 12289, 16384, 16500, 20000, 24000, 40961, 49151, 49152, 49153, 50001, 110592, 112086,
        131071, 131072, 131073, 200001, 250007, 300000, 327679, 327680, 327681, 393215, 393216, 393217, 400000,
        1400003, 1u << 21, 2147483647u};
    for (uint32_t per_cu = 1; per_cu <= 6; ++per_cu)
        for (uint32_t lane_div = 1; lane_div <= 8; ++lane_div)
            for (int few = 0; few < 2; ++few)
                for (uint32_t total : totals) {
                    const uint32_t blocks = split_blocks(total, cus * per_cu, cus, few);
                    const uint32_t nwaves = blocks * SPLIT_WAVES;
                    const uint32_t lanes = walk_lanes(lane_div, split_share(total, nwaves));
                    const uint32_t share0 = first_share(lane_div, total, nwaves, lanes);
                    uint64_t most = share0, given = (uint64_t)share0 * nwaves;
                    if (!share0)
                        for (uint32_t w = 0; w < nwaves; ++w) {
                            const uint64_t k = (uint64_t)total * (w + 1) / nwaves - (uint64_t)total * w / nwaves;
                            most = std::max(most, k);
                            given += k;
                        }
                    const bool ok = blocks >= 1 && blocks <= cus * per_cu && lanes >= 1 && lanes <= SPLIT_LANES &&
                                    (share0 ? given <= total && share0 <= POOL : given == total && most <= lanes);
                    if (!ok)
                        printf("total %u: %u workgroups, lane_div %u: %u lanes, share0 %u, most %llu, given %llu\n",
                               total, blocks, lane_div, lanes, share0, (unsigned long long)most,
                               (unsigned long long)given);
                }
    return 0;
}
"""

T_WAVE = r"""
#include <stdio.h>
#include "split.hpp"
using namespace n2v;
int main()
{
    const uint32_t t_waves[] = {0, 1, 8, 512, 1023, 1024, 1025, 4096, 0xFFFFFFFFu};
    const uint32_t walk_counts[] = {1, 1000, 5120, 5121, 100000};
    for (uint32_t lane_div = 1; lane_div <= 8; ++lane_div)
        for (uint32_t walks : walk_counts)
            for (uint32_t t : t_waves) {
                const uint32_t blocks = split_blocks(walks, 1280, 256, lane_div == 1);
                const uint32_t got = launch_t_wave(t, lone_walks(walks, blocks, lane_div));
                const uint32_t want = t == 1024 && lane_div == 1 && walks <= 5120 ? 0 : t;
                if (got != want) printf("t_wave %u, %u walks, lane_div %u: %u\n", t, walks, lane_div, got);
            }
    return 0;
}
"""

PLAIN = r"""
#include <stdio.h>
#include "split.hpp"
using namespace n2v;
int main()
{
    const uint32_t t_wgs[] = {0, 100, 65535, 65536, 65537, 0xFFFFFFFFu};
    const uint64_t hubs[] = {0, 1, 100, 101, 65536, 65537, 1ull << 33};
    for (uint32_t lane_div = 1; lane_div <= 8; ++lane_div)
        for (uint32_t t : t_wgs)
            for (uint64_t he : hubs) {
                const bool may = plain_may_fuse(lane_div, t, he);
                // a caller's own t_wg that some row may exceed keeps its workgroups
                if (may && (lane_div > 1 || (t != 65536 && he > t))) printf("t_wg %u, %llu\n", t, (unsigned long long)he);
                if (!may && lane_div == 1 && he <= t) printf("t_wg %u, %llu not\n", t, (unsigned long long)he);
                for (uint32_t walks = 1; walks && walks < 0x80000000u; walks = walks * 2 + walks % 3)
                    for (int counts = 0; counts < 2; ++counts) {
                        const PlainSplit p = plain_split(walks, 256, may, counts);
                        // the instances that exist
                        const bool ok = p.lanes == 1 ? !p.fused : p.lanes == 64 ? p.fused && !counts : p.lanes == 4 || p.lanes == 8;
                        if (!ok || (p.fused && !may)) printf("%u walks: %d lanes, fused %d\n", walks, p.lanes, p.fused);
                    }
            }
    return 0;
}
"""


def run(tmp_path, text):
    if shutil.which("g++") is None:
        pytest.skip("g++ not available")
    src, exe = tmp_path / "split.cpp", tmp_path / "split"
    src.write_text(text)
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-I", CSRC, str(src), "-o", str(exe)])
    out = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60)
    assert out.returncode == 0 and out.stdout == "", out.stdout[:2000]


def test_a_wavefront_has_a_lane_for_every_walk_it_is_given(tmp_path):
    run(tmp_path, DRIVER)


def test_only_the_default_t_wave_changes_for_lone_walks(tmp_path):
    run(tmp_path, T_WAVE)


def test_plain_supersteps_queue_the_moves_a_callers_t_wg_asks_for(tmp_path):
    run(tmp_path, PLAIN)
