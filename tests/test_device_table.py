"""The per-GPU table behind the tile passes' launch (host code, no GPU): each
device forms its own value once, also from several threads."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = r"""
#include <atomic>
#include <cstdio>
#include <thread>
#include <vector>
#include "device_table.h"
int main() {
    lbmep::DeviceTable<int, 8> table;
    std::atomic<int> made[10] = {};
    std::vector<std::thread> threads;
    std::atomic<int> wrong{0};
    for (int t = 0; t < 8; ++t)
        threads.emplace_back([&] {
            for (int k = 0; k < 200; ++k) {
                const int dev = k % 10 - 1;  // -1 and 8 lie beyond the table
                const int v = table.get(dev, [&] { made[dev + 1]++; return 100 + dev; });
                if (v != 100 + dev) wrong++;
            }
        });
    for (auto &t : threads) t.join();
    std::printf("%d", wrong.load());
    for (auto &m : made) std::printf(" %d", m.load());
    return 0;
}
"""


def test_every_device_forms_its_own_value_once(tmp_path):
    src, exe = tmp_path / "t.cpp", tmp_path / "t"
    src.write_text(PROGRAM)
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-pthread", "-I",
                           os.path.join(ROOT, "paper_1708_08741_amd", "csrc"), "-o", str(exe), str(src)])
    out = [int(v) for v in subprocess.check_output([str(exe)], text=True).split()]
    assert out[0] == 0
    assert out[2:10] == [1] * 8  # devices 0 .. 7
    assert out[1] == 8 * 20      # no such device: formed on every call


def test_the_tile_launch_keeps_nothing_for_the_first_device_only():
    """No attribute or occupancy of a kernel sits in a plain static of a
    launcher."""
    import re
    src = open(os.path.join(ROOT, "paper_1708_08741_amd", "csrc", "sor_tile_impl.h")).read()
    body = src[src.index("void launch_tile("):src.index("void launch_tile_pass(")]
    assert "hipFuncSetAttribute" in body
    for line in re.findall(r"^\s*static .*$", body, flags=re.M):
        assert "DeviceTable" in line
