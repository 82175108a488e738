"""The tile plan of the resident time loop on the host: what the kernel takes
for granted of it (tile heights, thread and word counts, that every LDS
element a thread reads lies in the block's tiles), and which plans the
grids of the GPU tests get."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2304_00233_amd", "csrc")

# (shape, rd, nb, ne) -> planes per thread, one thread group or several
GRIDS = [((37, 29, 23), 2, 10, 7, 3, False), ((21, 45, 64), 2, 10, 8, 4, False), ((26, 44, 55), 1, 10, 8, 4, True),
         ((25, 40, 82), 3, 6, 8, 3, True), ((48, 48, 48), 2, 10, 7, 5, False), ((9, 60, 40), 1, 3, 2, 1, True),
         # one update plane (two per thread where that lets it receive more words)
         ((61, 42, 5), 2, 0, 0, 2, False), ((45, 58, 7), 3, 0, 0, 2, False)]

PROGRAM = r"""
#include "emm_resident_plan.h"
#include <algorithm>
#include <cstdio>
#include <cstdlib>
#include <random>
using namespace emm;
static long check(int r, int n1, int n2, int n3, const ResidentPlan &p) {
    const int L = 2 * r, nx = n1 - L, ny = n2 - L, nz = n3 - L;
    const long zs = (long)(p.ty + L - 1) * n1;
    long reach = 0;
    if (p.gy * p.gz > 256 || p.threads % (64 * p.groups) || p.threads > resident_threads(p.planes)) return 1;
    if (p.threads / p.groups < nx * p.ty || p.groups * p.planes < p.tz || p.tz > kResTall) return 2;
    if (2 * (L - 1) * (p.ty + p.tz) * nx > p.threads * resident_words(p.planes)) return 3;
    for (int bz = 0; bz < p.gz; ++bz)
        for (int by = 0; by < p.gy; ++by) {
            const int ty = ny * (by + 1) / p.gy - ny * by / p.gy, tz = nz * (bz + 1) / p.gz - nz * bz / p.gz;
            if (ty > p.ty || tz > p.tz || (p.gy > 1 && ty < r) || (p.gz > 1 && tz < r)) return 4;
            // every element that the threads of every group read, E (h = 0, r - 1
            // halo rows and planes below) and H (h = 1, r below)
            for (int h = 0; h < 2; ++h)
                for (int yy : {0, ty - 1})
                    for (int i : {r, n1 - 1 - r})
                        for (int pl = 0; pl < p.groups * p.planes; ++pl) {
                            const int HL = h ? r : r - 1;
                            const long o = 3l * h * kResSlot + (HL + pl) * zs + (yy + HL) * (long)n1 + i;
                            for (int m = 0; m < L; ++m)
                                for (long at : {o + 2 * kResSlot + (m - HL) * (long)n1, o + 2 * kResSlot + m - HL,
                                                o + kResSlot + (m - HL) * zs, o + kResSlot + m - HL,
                                                o + (m - HL) * zs, o + (m - HL) * (long)n1}) {
                                    if (at < 0 || at >= 6l * kResSlot) return 5;
                                    reach = std::max(reach, at);
                                }
                        }
        }
    return reach == resident_reach(r, n1, p) ? 0 : 6;
}
int main(int argc, char **argv) {
    if (argc == 5) {
        const ResidentPlan p = resident_plan(atoi(argv[1]), atoi(argv[2]), atoi(argv[3]), atoi(argv[4]), 256);
        printf("%d %d\n", p.planes, p.groups);
        return 0;
    }
    std::mt19937 g(1);
    int plans = 0;
    for (int t = 0; t < 20000; ++t) {
        const int r = 1 + g() % 3, top = t % 2 ? 110 : 250;
        const int n1 = 2 * r + 1 + g() % top, n2 = 2 * r + 1 + g() % top, n3 = 2 * r + 1 + g() % top;
        const ResidentPlan p = resident_plan(r, n1, n2, n3, 256);
        if (!p.gy) continue;
        ++plans;
        if (long e = check(r, n1, n2, n3, p)) {
            printf("r%d %d %d %d: %ld\n", r, n1, n2, n3, e);
            return 1;
        }
    }
    printf("%d\n", plans);
    return plans > 1000 ? 0 : 1;
}
"""


@pytest.fixture(scope="module")
def plan(tmp_path_factory):
    d = tmp_path_factory.mktemp("plan")
    (d / "plan.cpp").write_text(PROGRAM)
    exe = d / "plan"
    subprocess.run(["g++", "-O2", "-std=c++17", "-I", CSRC, str(d / "plan.cpp"),
                    os.path.join(CSRC, "emm_resident_plan.cpp"), "-o", str(exe)], check=True)
    return lambda *a: subprocess.run([str(exe), *map(str, a)], capture_output=True, text=True)


def test_plans_keep_what_the_kernel_assumes(plan):
    res = plan()
    assert res.returncode == 0, res.stdout


@pytest.mark.parametrize("shape,rd,nb,ne,planes,several", GRIDS)
def test_plans_of_the_gpu_cases(plan, shape, rd, nb, ne, planes, several):
    p, g = map(int, plan(rd, *(n + 2 * (nb + ne) for n in shape)).stdout.split())
    assert p == planes and (g > 1) == several
