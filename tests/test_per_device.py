"""Values found once per device (csrc/perdev.hpp), built for the CPU: threads
that ask while the first one is still filling must get the whole value."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1805_00280_amd", "csrc")

DRIVER = r"""
#include <stdio.h>
#include <atomic>
#include <chrono>
#include <thread>
#include <vector>
#include "perdev.hpp"
struct Info {
    int a = 0, b = 0;
};
int main()
{
    static n2v::PerDevice<Info> info;
    std::atomic<int> fills{0}, partial{0};
    std::vector<std::thread> t;
    for (int i = 0; i < 16; ++i)
        t.emplace_back([&, i] {
            const int dev = i % 2;
            const Info &d = info.get(dev, [&](Info &v) {
                ++fills;
                v.a = 1 + dev;
                std::this_thread::sleep_for(std::chrono::milliseconds(50));
                v.b = 1 + dev;
            });
            if (d.a != 1 + dev || d.b != 1 + dev) ++partial;
        });
    for (std::thread &x : t) x.join();
    printf("%d %d\n", fills.load(), partial.load());
    return 0;
}
"""


def test_threads_never_see_a_partly_filled_value(tmp_path):
    if shutil.which("g++") is None:
        pytest.skip("g++ not available")
    src, exe = tmp_path / "once.cpp", tmp_path / "once"
    src.write_text(DRIVER)
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-pthread", "-I", CSRC, str(src), "-o",
                           str(exe)])
    out = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60)
    assert out.returncode == 0 and out.stdout.split() == ["2", "0"], (out.returncode, out.stdout)
