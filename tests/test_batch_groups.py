"""Grouping on the host.  A batch's jobs: consecutive groups that cover every
job, none beyond the cache budget once its jobs fill the chip, except for two
jobs of one or two sources.  A forward's sources: loops of even size within
the budget."""
import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2304_00233_amd", "csrc")
BUDGET, PAIR, FILL = 240.0, 560.0, 2.5               # MB, million cells

PROGRAM = r"""
#include "emm_groups.h"
#include <cstdio>
#include <cstdlib>
int main(int argc, char **argv) {
    if (argc == 4) {
        printf("%d ", emm::source_group(1e6 * atof(argv[1]), 1e6 * atof(argv[2]), atoi(argv[3])));
        return 0;
    }
    std::vector<double> need, cells;
    std::vector<int> nsrc;
    for (int a = 1; a + 2 < argc; a += 3) {
        need.push_back(1e6 * atof(argv[a]));
        cells.push_back(1e6 * atof(argv[a + 1]));
        nsrc.push_back(atoi(argv[a + 2]));
    }
    for (int g : emm::batch_groups(need, cells, nsrc)) printf("%d ", g);
}
"""


@pytest.fixture(scope="module")
def groups(tmp_path_factory):
    d = tmp_path_factory.mktemp("groups")
    (d / "g.cpp").write_text(PROGRAM)
    subprocess.run(["g++", "-O1", "-std=c++17", "-I", CSRC, str(d / "g.cpp"), "-o", str(d / "g")], check=True)

    def call(jobs, source=False):
        args = [str(v) for job in jobs for v in job] + ([] if source else ["end"])
        return [int(v) for v in subprocess.run([str(d / "g"), *args], capture_output=True, text=True,
                                               check=True).stdout.split()]
    return call


# (MB, million cells, sources) of each job -> group sizes
CASES = [([(150, 4, 1)] * 4, [2, 2]),                      # pairs, though beyond the budget
         ([(150, 4, 2)] * 5, [2, 2, 1]),
         ([(150, 4, 3)] * 4, [1, 1, 1, 1]),                # not with more sources
         ([(150, 4, 1), (150, 4, 3), (150, 4, 1)], [1, 1, 1]),
         ([(300, 8, 1)] * 2, [1, 1]),                      # nor far beyond it
         ([(97, 2.6, 1)] * 3, [2, 1]),                     # three together exceed it
         ([(97, 2.6, 4)] * 7, [2, 1, 2, 2]),
         ([(76, 2.1, 1)] * 4, [2, 2]),                     # even, not 3 + 1
         ([(76, 2.1, 1)] * 7, [2, 3, 2]),
         ([(64, 1.6, 1)] * 12, [3, 3, 3, 3]),
         ([(46, .9, 1), (50, 1.1, 1), (55, 1.3, 1), (60, 1.5, 1), (66, 1.7, 1), (71, 2.0, 1), (96, 2.2, 1),
           (103, 2.5, 1)], [4, 2, 2]),
         ([(20, 0.5, 1), (230, 6, 1), (20, 0.5, 1), (20, 0.5, 1)], [2, 2]),
         ([(30, 0.5, 1)] * 9, [5, 4]),
         ([(20, 0.3, 1)] * 12, [12]),
         ([(10, 0.1, 1)], [1])]


@pytest.mark.parametrize("jobs,want", CASES)
def test_batch_groups(groups, jobs, want):
    got = groups(jobs)
    assert got == want
    j = 0
    for size in got:
        part = jobs[j:j + size]
        j += size
        held = sum(b for b, _, _ in part)
        assert (held <= BUDGET or size == 1 or sum(c for _, c, _ in part[:-1]) < FILL or
                (size == 2 and held <= PAIR and max(s for _, _, s in part) <= 2))
    assert j == len(jobs)


# MB of a source, MB shared by all, sources -> sources per loop
@pytest.mark.parametrize("per,shared,nsrc,want", [(23, 3, 9, 9), (23, 3, 10, 10), (23, 3, 11, 6), (23, 3, 16, 8),
                                                  (35, 4, 12, 6), (62, 24, 6, 3), (153, 62, 4, 1), (200, 60, 4, 4),
                                                  (239, 1, 3, 1), (5, 1, 1, 1)])
def test_source_groups(groups, per, shared, nsrc, want):
    assert groups([(per, shared, nsrc)], source=True) == [want]
