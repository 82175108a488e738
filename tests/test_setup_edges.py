"""Point stencils and source control volumes at the ends of an axis, on the
host, with the standard library's own bounds checks."""
import os
import subprocess

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2304_00233_amd", "csrc")

PROGRAM = r"""
#include "emm_setup.h"
#include <cmath>
#include <cstdio>
using namespace emm;
int main() {
    for (int nbe = 0; nbe < 4; ++nbe)
        for (int r = 1; r <= 4; ++r) {
            std::vector<double> in;
            for (int i = 0; i < 2 * r + 3; ++i) in.push_back(i + 0.1 * i * i);
            const std::vector<double> x = pad_axis(in.data(), (int)in.size(), nbe), h = half_nodes(x);
            const int n = (int)x.size();
            for (int staggered = 0; staggered < 2; ++staggered)
                for (double p = in[0] - 1.0; p < in.back() + 1.0; p += 0.01) {
                    const std::vector<double> &c = staggered ? h : x;
                    double w[8];
                    for (double &v : w) v = NAN;
                    const int base = point_stencil(c, p, r, w);
                    if (!stencil_inside(c, base, r, n, nbe)) continue;
                    double sum = 0.0;
                    for (int q = 0; q < 2 * r; ++q) {
                        sum += w[q];                       // filled: the weights sum to one
                        if (base + q < nbe || base + q > n - 1 - nbe) return 1;
                        const double e = source_extent(x, h, base + q, staggered);
                        if (!(e > 0.0)) return 2;
                        if (!staggered && base + q > 0 && base + q < n - 1 && e != h[base + q] - h[base + q - 1]) return 3;
                    }
                    if (!(std::fabs(sum - 1.0) < 1e-9)) return 4;
                }
        }
    return 0;
}
"""


def test_points_at_the_ends_of_an_axis(tmp_path):
    (tmp_path / "t.cpp").write_text(PROGRAM)
    subprocess.run(["g++", "-O1", "-std=c++17", "-D_GLIBCXX_ASSERTIONS", "-I", CSRC, str(tmp_path / "t.cpp"),
                    os.path.join(CSRC, "emm_setup.cpp"), "-o", str(tmp_path / "t")], check=True)
    assert subprocess.run([str(tmp_path / "t")]).returncode == 0
