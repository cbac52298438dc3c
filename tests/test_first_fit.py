"""The allocator under the server's device arena and its pinned slabs (host
code, no GPU): runs never overlap, all of it comes back."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = r"""
#include <cstdio>
#include <map>
#include <random>
#include "first_fit.h"
using lbmep::FirstFit;
int main() {
    const size_t size = size_t(3) << 20;
    FirstFit f(size + 17);
    std::mt19937 rng(7);
    std::map<size_t, size_t> live;  // offset -> bytes asked for
    int refused = 0;
    for (int k = 0; k < 20000; ++k) {
        if (live.empty() || rng() % 5 < 3) {
            const size_t bytes = 1 + rng() % (rng() % 8 ? 60000 : 900000);
            const size_t off = f.alloc(bytes);
            if (off == FirstFit::kNone) {
                ++refused;
                continue;
            }
            if (off % FirstFit::kAlign || off + bytes > size) return 1;
            auto next = live.lower_bound(off);
            if (next != live.end() && next->first < off + bytes) return 2;
            if (next != live.begin() && std::prev(next)->first + std::prev(next)->second > off) return 3;
            live[off] = bytes;
        } else {
            auto it = live.begin();
            std::advance(it, rng() % live.size());
            f.release(it->first);
            f.release(it->first);  // a second release does nothing
            live.erase(it);
        }
        size_t used = 0;
        for (auto &l : live) used += (l.second + FirstFit::kAlign - 1) / FirstFit::kAlign * FirstFit::kAlign;
        if (used != f.used()) return 4;
    }
    for (auto &l : live) f.release(l.first);
    if (f.used() != 0 || f.size() != size || refused == 0) return 5;
    if (f.alloc(size) != 0 || f.alloc(1) != FirstFit::kNone) return 6;
    FirstFit none(100);
    return none.alloc(1) == FirstFit::kNone && none.size() == 0 ? 0 : 7;
}
"""


def test_runs_do_not_overlap_and_come_back(tmp_path):
    src, exe = tmp_path / "t.cpp", tmp_path / "t"
    src.write_text(PROGRAM)
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-I",
                           os.path.join(ROOT, "paper_1708_08741_amd", "csrc"), "-o", str(exe), str(src)])
    assert subprocess.call([str(exe)]) == 0


def test_results_of_a_server_free_no_pinned_memory_while_it_steps():
    """hipHostFree may wait for the device: only the server's end calls it."""
    src = open(os.path.join(ROOT, "paper_1708_08741_amd", "csrc", "lbmep_server.hip")).read()
    assert src.count("hipHostFree(") == 1
    body = src[src.index("~PinnedBlocks()"):src.index("void set_limit(")]
    assert "hipHostFree(" in body
