"""Element index of the brick passes at the largest grid they accept, on the host.

A Dirichlet grid may hold 2^31 cells (its work items count cells in an int); with
the ghost shell that is more than 2^31 elements, past a signed 32-bit offset.
The 24-bit index (small_index) is compared with the 64-bit one (cell_index's
arithmetic, the strides of a level) at the corners, shell included, and at random
cells, for such grids, for small ones and for periodic levels.
"""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")

PROGRAM = r"""
#include <hip/hip_runtime.h>
#include <cstdio>
#include <random>
#include "%s/vmg_internal.h"
#include "%s/device_common.h"
using namespace vmg;

static Geom level(int n0, int n1, int n2, int dir, int64_t base) {
    Geom g{};
    g.n0 = n0; g.n1 = n1; g.n2 = n2; g.dir = dir; g.base = base;
    g.sy = n0 + 2 * dir;
    g.sz = g.sy * (n1 + 2 * dir);
    g.off0 = base + (dir ? 1 + g.sy + g.sz : 0);
    return g;
}

template <int DIR>
static long check(const Geom& g) {
    std::mt19937 rng(7);
    const int n[3] = {g.n0, g.n1, g.n2};
    long bad = 0;
    for (int t = 0; t < 20064; ++t) {
        int c[3];
        for (int a = 0; a < 3; ++a) {
            const int lo = DIR ? -1 : 0, hi = n[a] - 1 + (DIR ? 1 : 0);
            const int at[4] = {lo, lo + 1, hi - 1, hi};
            c[a] = t < 64 ? at[(t >> (2 * a)) & 3] : lo + (int)(rng() %% (unsigned)(hi - lo + 1));
        }
        const int64_t want = g.off0 + c[0] + c[1] * g.sy + c[2] * g.sz;
        if (small_index<DIR>(g, c[0], c[1], c[2]) != want) ++bad;
    }
    return bad;
}

int main() {
    const int d[][3] = {{2048, 1024, 1024}, {1024, 2048, 1024}, {1024, 1024, 2048}, {2048, 2048, 512}, {512, 2048, 2048},
                        {64, 64, 64}, {24, 40, 32}, {2, 3, 5}};
    for (auto& n : d)
        for (int64_t base : {(int64_t)0, (int64_t)1 << 33})
            std::printf("dirichlet %%dx%%dx%%d base %%lld: %%ld bad\n", n[0], n[1], n[2], (long long)base,
                        check<1>(level(n[0], n[1], n[2], 1, base)));
    const int p[][3] = {{1024, 1024, 1024}, {64, 64, 64}, {20, 24, 28}, {4, 6, 8}};
    for (auto& n : p)
        std::printf("periodic %%dx%%dx%%d: %%ld bad\n", n[0], n[1], n[2], check<0>(level(n[0], n[1], n[2], 0, 0)));
    return 0;
}
"""


def test_small_index_equals_the_64_bit_index(tmp_path):
    if not os.path.exists(HIPCC):
        pytest.skip("no hipcc")
    csrc = os.path.join(ROOT, "paper_1303_0008_amd", "csrc")
    src, exe = tmp_path / "index.cpp", tmp_path / "index"
    src.write_text(PROGRAM % (csrc, csrc))
    r = subprocess.run([HIPCC, "-x", "hip", "--cuda-host-only", "-O1", "-std=c++17", str(src), "-o", str(exe)],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    out = subprocess.run([str(exe)], capture_output=True, text=True)
    print(out.stdout)
    assert out.returncode == 0
    lines = out.stdout.splitlines()
    assert len(lines) == 20 and all(line.endswith(": 0 bad") for line in lines)
