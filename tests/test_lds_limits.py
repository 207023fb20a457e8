"""Dynamic LDS limits of the kernels, on the CPU: a host program puts its own
recording versions of the HIP calls in front of the library's (nothing reaches
a device) and drives the launchers through shapes of different size.  A launch
may not ask for more LDS than its kernel's limit on the device, whatever shapes
were queried or launched before it, and no call lowers a limit: another thread
may be between raising it and launching."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PKG = os.path.join(ROOT, "paper_2108_01186_amd")
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")

PROGRAM = r"""
#include <cstdio>
#include <cstring>
#include <map>
#include <vector>
#include "kernels.h"

static std::map<const void *, size_t> limit;
static int lowered = 0, over = 0, launches = 0;
static dim3 cg, cb;
static size_t cl;
static hipStream_t cst;
static size_t limit_of(const void *f) { return limit.count(f) ? limit[f] : 65536; }

extern "C" {
hipError_t hipFuncSetAttribute(const void *f, hipFuncAttribute, int v) {
    if ((size_t)v < limit_of(f) && limit.count(f)) ++lowered;
    limit[f] = (size_t)v;
    return hipSuccess;
}
hipError_t hipOccupancyMaxActiveBlocksPerMultiprocessor(int *n, const void *, int, size_t) {
    *n = 1;
    return hipSuccess;
}
hipError_t hipGetDevice(int *d) {
    *d = 0;
    return hipSuccess;
}
hipError_t hipDeviceGetAttribute(int *v, hipDeviceAttribute_t, int) {
    *v = 256;
    return hipSuccess;
}
hipError_t hipGetLastError(void) { return hipSuccess; }
hipError_t __hipPushCallConfiguration(dim3 g, dim3 b, size_t l, hipStream_t s) {
    cg = g; cb = b; cl = l; cst = s;
    return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3 *g, dim3 *b, size_t *l, hipStream_t *s) {
    *g = cg; *b = cb; *l = cl; *s = cst;
    return hipSuccess;
}
hipError_t hipLaunchKernel(const void *f, dim3, dim3, void **, size_t lds, hipStream_t) {
    ++launches;
    if (lds > limit_of(f)) ++over;
    return hipSuccess;
}
}

using namespace fsic;
static int bad = 0;
static void ok(hipError_t e) { bad += e != hipSuccess; }

static void fdm(int T, int two) {
    const FdmClass cl[2] = {{kFdmPassXY, T, two, 1, 0}, {kFdmPassZ, T, 0, 1, 0}};
    FdmPlan p{};
    p.cls = cl;
    p.ncls = 2;
    for (int sq = 0; sq < 2; ++sq) ok(launch_fdm(p, nullptr, nullptr, nullptr, nullptr, sq, 1.0, nullptr, nullptr, nullptr));
}
static void lowdin(int N) {
    LowdinBatch lb{};
    lb.n = 1;
    lb.N[0] = N;
    ok(launch_lowdin_batch(lb, nullptr, LowdinOffsets{}, nullptr, 0, 0.0, nullptr, nullptr));
    ok(launch_lowdin(N, nullptr, nullptr, nullptr, nullptr, nullptr, nullptr, nullptr, nullptr, 0.0, nullptr, nullptr, nullptr));
    LowdinBwdBatch bb{};
    bb.n = 1;
    bb.N[0] = N;
    ok(launch_lowdin_backward_batch(bb, nullptr, 0, nullptr, LowdinBwdOffsets{}, nullptr, 0, nullptr, nullptr));
}
static void octant(int lmax, int tiles) {
    oct_slots(0, lmax, tiles);
    oct_slots(1, lmax, tiles);
    ok(launch_sic_octant(lmax, nullptr, 1, nullptr, nullptr, tiles, tiles, nullptr, nullptr, nullptr, 0.0, 0, nullptr, nullptr, nullptr));
}
static void transform(int N) {
    ProdChan c{};
    c.N = N;
    c.M = 1000;
    ok(launch_transform(&c, 1, nullptr));
}
static void sine(int np, int variant, int npxy, bool two) {
    ok(dst_setup(np, variant, npxy, two));
    DstItems di{};
    di.nx = di.ny = di.nz = 1;
    di.fast = variant;
    di.np = np;
    di.blocks = 1;
    di.nxy = npxy > 0;
    di.two = two;
    di.npxy = npxy;
    for (int v = 0; v < 2; ++v)
        for (int o = 0; o < 2; ++o) {
            di.xyvec = v;
            di.xyocc2 = o;
            ok(launch_dst_precond<float>(di, nullptr, nullptr, nullptr, nullptr, nullptr, nullptr, nullptr, nullptr, nullptr));
            ok(launch_dst_pcg(di, nullptr, nullptr, nullptr, nullptr, nullptr, nullptr, nullptr, PcgOut{}, nullptr, nullptr));
        }
}
static void expand(int lmax) {
    for (int m = 0; m < 2; ++m) {
        harm_slots(2 + m, lmax);
        ok(launch_harm_expand(m, lmax, HarmTables{}, 6, nullptr, nullptr, nullptr, 1, nullptr, nullptr, nullptr));
    }
}

int main(int, char **a) {
    const char *const w = a[1];
    if (!strcmp(w, "fdm")) {
        // queries come with a batch's plan, the limits with its preparation
        auto batch = [](int T, int two) {
            fdm_occupancy(kFdmPassXY, T, two);
            fdm_occupancy(kFdmPassZ, T, 0);
            ok(fdm_setup());
            fdm(T, two);
        };
        for (int T = 1; T <= 3; ++T)
            for (int two : {1, 0, 1}) batch(T, two);
        batch(4, 0);
    } else if (!strcmp(w, "lowdin")) {
        for (int N : {128, 5, 64, 100, 64, 128}) lowdin(N);
    } else if (!strcmp(w, "octant")) {
        for (int lmax : {6, 8, 0, 6})
            for (int t : {16, 1, 4, 6, 2, 16}) octant(lmax, t);
    } else if (!strcmp(w, "transform")) {
        for (int N : {128, 33, 96, 128, 113, 97}) transform(N);
    } else if (!strcmp(w, "sine")) {
        struct { int np, v, npxy; bool two; } q[] = {{128, 1, 128, false}, {96, 1, 96, true}, {64, 1, 64, false},
            {128, 1, 128, false}, {96, 1, 96, true}, {160, 2, 0, false}, {192, 3, 0, false}, {192, 3, 128, false},
            {128, 1, 0, false}, {160, 2, 0, false}};
        for (auto &x : q) sine(x.np, x.v, x.npxy, x.two);
    } else {
        for (int l : {8, 0, 6, 8}) expand(l);
    }
    printf("%d launches, %d over their limit, %d limits lowered, %d errors\n", launches, over, lowered, bad);
    return launches == 0 || over || lowered || bad;
}
"""


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    if not os.path.exists(HIPCC):
        pytest.skip("hipcc not available")
    if not os.path.exists(os.path.join(PKG, "libfsic.so")):
        pytest.fail("libfsic.so is not built (run __graft_entry__.build())")
    d = tmp_path_factory.mktemp("lds")
    src, exe = d / "lds.hip", str(d / "lds")
    src.write_text(PROGRAM)
    obj = str(d / "lds.o")
    subprocess.run([HIPCC, "-x", "hip", "--offload-arch=gfx950", "--offload-host-only", "-O1", "-std=c++17",
                    "-I" + os.path.join(PKG, "csrc"), "-c", str(src), "-o", obj], check=True)
    # (the program's symbols are found before the HIP runtime's)
    subprocess.run([HIPCC, obj, os.path.join(PKG, "libfsic.so"), "-rdynamic", "-Wl,-rpath," + PKG, "-o", exe], check=True)
    return exe


@pytest.mark.parametrize("launcher", ["fdm", "lowdin", "octant", "transform", "sine", "expand"])
def test_limits_hold_and_are_never_lowered(program, launcher):
    r = subprocess.run([program, launcher], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stdout + r.stderr
