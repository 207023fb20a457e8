"""The direct solver's axis tables are made once per process, however many
axis lengths are in use."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2108_01186_amd", "csrc")

PROGRAM = r"""
#include "fdm_basis.h"
#include <cstdio>
#include <cstring>
#include <set>
#include <thread>
int main() {
    const double c2[2] = {-2.0, 1.0}, c4[3] = {-2.5, 4.0 / 3.0, -1.0 / 12.0};
    std::vector<const double *> first;
    for (int n = 8; n < 72; ++n) {
        first.push_back(fsic::fdm_axis(n, 1, c2).data());
        first.push_back(fsic::fdm_axis(n, 2, c4).data());
    }
    if (std::set<const double *>(first.begin(), first.end()).size() != first.size()) return 1;
    int moved = 0;
    std::thread t[4];
    for (auto &th : t)
        th = std::thread([&] {
            for (int n = 8; n < 72; ++n)
                if (fsic::fdm_axis(n, 1, c2).data() != first[2 * (n - 8)] || fsic::fdm_axis(n, 2, c4).data() != first[2 * (n - 8) + 1])
                    __atomic_fetch_add(&moved, 1, __ATOMIC_RELAXED);
        });
    for (auto &th : t) th.join();
    if (moved) return 2;
    const auto fresh = fsic::fdm_axis_table(40, 2, c4);
    return memcmp(fresh.data(), fsic::fdm_axis(40, 2, c4).data(), fresh.size() * sizeof(double)) ? 3 : 0;
}
"""


def test_tables_are_made_once(tmp_path):
    """64 lengths at two orders: the second round, in four threads, finds every
    table where the first one put it."""
    src, exe = tmp_path / "t.cpp", str(tmp_path / "t")
    src.write_text(PROGRAM)
    subprocess.run(["g++", "-O2", "-std=c++17", "-pthread", "-I" + CSRC, str(src), "-o", exe], check=True)
    assert subprocess.run([exe], timeout=60).returncode == 0
