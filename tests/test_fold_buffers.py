"""Which buffer of tile sums a scored step takes (paper_2403_04206_amd/csrc/grawa_route.h): never the one that holds sums which
are not folded in yet, whatever is called, recorded and replayed after what (a small program plays random sequences); and the estimate where
the counts of steps pass 32 bits."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
pytestmark = pytest.mark.skipif(shutil.which("g++") is None, reason="no host compiler")

PROGRAM = r"""
#include <cstdio>
#include <cstdlib>
#include <vector>
#include "grawa_route.h"
struct Launch { unsigned buffer; bool at_once; };
int main()
{
    srand(5);
    long steps = 0, replays = 0;
    for (int trial = 0; trial < 2000; ++trial) {
        GrawaSteps host = {};
        std::vector<std::vector<Launch>> graphs;
        int pending = -1; // buffer, on the device
        unsigned long long id = rand() % 3 ? 1 : 1000;
        const auto run = [&](const Launch &l) {
            if ((int)l.buffer == pending || l.buffer >= GRAWA_SUM_BUFFERS) return false;
            pending = l.at_once ? -1 : (int)l.buffer;
            ++steps;
            return true;
        };
        for (int i = 0; i < 60; ++i) {
            const int what = rand() % 4;
            if (what == 0) { // a call
                Launch l;
                l.buffer = grawa_step_buffer(host, false, id, &l.at_once);
                grawa_step_sent(host, false, id);
                if (!run(l)) { std::printf("call finds its buffer pending, trial %d\n", trial); return 1; }
            } else if (what == 1) { // a recording of 1 to 5 steps; nothing runs
                ++id;
                std::vector<Launch> g(1 + rand() % 5);
                for (Launch &l : g) {
                    l.buffer = grawa_step_buffer(host, true, id, &l.at_once);
                    grawa_step_sent(host, true, id);
                    if (grawa_all_folded(host, true, id) != l.at_once) return 2;
                    if (grawa_all_folded(host, true, id + 1) || grawa_all_folded(host, false, id)) return 3;
                }
                graphs.push_back(g);
            } else if (what == 2 && !graphs.empty()) { // a replay
                ++replays;
                for (const Launch &l : graphs[rand() % graphs.size()])
                    if (!run(l)) { std::printf("replay finds its buffer pending, trial %d\n", trial); return 1; }
            } else if (rand() % 2) { // a communication uses up what is pending
                pending = -1;
            }
        }
    }
    std::printf("%d\n", steps > 10000 && replays > 10000);
    return 0;
}
"""


def test_a_step_never_finds_its_own_buffer_pending(tmp_path):
    src, out = str(tmp_path / "steps.cpp"), str(tmp_path / "steps")
    with open(src, "w") as f:
        f.write(PROGRAM)
    res = subprocess.run(["g++", "-std=c++17", "-Wall", "-Wextra", "-Werror", "-I", os.path.join(ROOT, "paper_2403_04206_amd", "csrc"),
                          src, "-o", out], capture_output=True, text=True)
    assert res.returncode == 0, res.stderr
    res = subprocess.run([out], capture_output=True, text=True)
    assert res.returncode == 0 and res.stdout.strip() == "1", res.stdout


COUNTS = r"""
#include <cmath>
#include <cstdio>
#include "grawa_route.h"
// A round of two steps before and after each of the four communications around step 2^32, noted by launches of the weights alone (what pulls
// noted stays 0) or by pulls alone: the estimate is that of the steps since the last communication.
int main()
{
    for (int by_pull = 0; by_pull < 2; ++by_pull)
        for (uint64_t first = 4294967288ull; first < 4294967298ull; ++first) {
            uint64_t noted = first;
            GrawaEstimate e = {7.0, 0.5, first, 0, 0}; // 7: left from the round before, which is used up
            for (int round = 0; round < 6; ++round) {
                for (int step = 1; step <= 2; ++step) {
                    const uint64_t used = by_pull ? grawa_last_used(0, noted) : grawa_last_used(noted, 0);
                    e.mvg = grawa_estimate_value(e, used, 1.0); // folded in by the next step: norm 1
                    e.n += 1;
                    e.left = 1;
                }
                const uint64_t used = by_pull ? grawa_last_used(0, noted) : grawa_last_used(noted, 0);
                const double v = grawa_estimate_value(e, used, 1.0);
                if (e.n - used != 2 || std::fabs(v - 0.75) > 1e-15) {
                    std::printf("step %llu, used %llu: %g\n", (unsigned long long)e.n, (unsigned long long)used, v);
                    return 1;
                }
                noted = e.n;
            }
        }
    std::puts("1");
    return 0;
}
"""


def test_estimate_where_the_counts_pass_32_bits(tmp_path):
    src, out = str(tmp_path / "counts.cpp"), str(tmp_path / "counts")
    with open(src, "w") as f:
        f.write(COUNTS)
    res = subprocess.run(["g++", "-std=c++17", "-Wall", "-Wextra", "-Werror", "-I", os.path.join(ROOT, "paper_2403_04206_amd", "csrc"),
                          src, "-o", out], capture_output=True, text=True)
    assert res.returncode == 0, res.stderr
    res = subprocess.run([out], capture_output=True, text=True)
    assert res.returncode == 0 and res.stdout.strip() == "1", res.stdout
