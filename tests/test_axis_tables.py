"""The direct solver's axis tables: made once per process, however many axis
lengths are in use, and as accurate as their rounding."""
import os
import subprocess

import numpy as np

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


TABLE = r"""
#include "fdm_basis.h"
#include <cstdio>
#include <cstdlib>
int main(int, char **a) {
    const double c[2] = {-2.0, 1.0};
    const auto t = fsic::fdm_axis_table(atoi(a[1]), 1, c);
    fwrite(t.data(), 8, t.size(), stdout);
}
"""


def test_second_order_axes_are_the_sines(tmp_path):
    """At order 2 the eigenvectors are known, sqrt(2 / (n + 1)) times sines: the
    table holds them to half a unit in the last place of the largest entry
    (the rounding of the table) and as much again for what forms them."""
    src, exe = tmp_path / "t.cpp", str(tmp_path / "t")
    src.write_text(TABLE)
    subprocess.run(["g++", "-O2", "-std=c++17", "-I" + CSRC, str(src), "-o", exe], check=True)
    ld = np.longdouble
    for n in (8, 9, 31, 32, 33, 64, 96, 127, 160, 192):
        t = np.frombuffer(subprocess.run([exe, str(n)], check=True, capture_output=True, timeout=60).stdout)
        L = 16 * (((n + 1) // 2 + 15) // 16)
        for par in range(2):
            h = (n + 1) // 2 if par == 0 else n // 2
            lam = t[2 * L * L + par * L:][:h]
            C = t[:2 * L * L].reshape(2, L, L)[par, :h, :h][np.argsort(lam)]
            k, j = np.arange(h)[:, None], np.arange(h)[None]
            ref = np.sqrt(ld(2) / (n + 1)) * np.sin(ld("3.14159265358979323846264338327950288") * ld(1) / (n + 1)
                                                    * ((2 * k + par + 1) * (j + 1) % (2 * (n + 1))))
            sign = np.sign((C * ref).sum(1))[:, None]
            assert np.abs(sign * C - ref).max() <= np.spacing(float(np.abs(ref).max())), (n, par)
