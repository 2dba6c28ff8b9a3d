"""What a context remembers of the cells that a device build's groups opened,
and the level walk's capacity of the next build (OctMemory in
csrc/bhq_internal.h), compiled for the host."""
import os
import subprocess

import pytest

from conftest import ROOT

CSRC = os.path.join(ROOT, "paper_1812_07313_amd", "csrc")

MAIN = r"""
#include <cstdio>
#include <cstdlib>
#include "bhq_internal.h"
// arguments: theta ncrit opened ...; prints each build's capacity
int main(int argc, char **argv)
{
    bhq::OctMemory m;
    for (int i = 1; i + 2 < argc; i += 3) {
        const double theta = atof(argv[i]);
        const int ncrit = atoi(argv[i + 1]);
        printf("%d ", m.capacity(theta, ncrit));
        m.built(theta, ncrit, atoll(argv[i + 2]));
    }
    return 0;
}
"""


@pytest.fixture(scope="module")
def capacities(tmp_path_factory):
    d = tmp_path_factory.mktemp("walk")
    src, exe = str(d / "main.cpp"), str(d / "main")
    with open(src, "w") as f:
        f.write(MAIN)
    subprocess.run(["g++", "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-I", "/opt/rocm/include",
                    "-I", CSRC, "-I", os.path.join(ROOT, "include"), "-o", exe, src], check=True)

    def run(builds):
        args = [str(v) for b in builds for v in b]
        return [int(v) for v in subprocess.check_output([exe] + args).split()]
    return run


def test_capacity_follows_the_last_build(capacities):
    same = [(0.3, 64, opened) for opened in (100, 1000, 1500, 2000, 3500, 4080, 4000, 10)]
    # 1024 first, then 1.25 times the last build's and 8 more, at most 4080: a
    # build that outgrew its capacity (1500 after 1258) is counted too
    assert capacities(same) == [1024, 133, 1258, 1883, 2508, 4080, 4080, 4080]


def test_too_many_cells(capacities):
    """A group that opens more than 4080 cells leaves the octet walk (0) to
    the builds of its opening criterion until one opens fewer."""
    assert capacities([(0.0, 8, 5000), (0.0, 8, 9000), (0.0, 8, 1200), (0.0, 8, 1200)]) == \
        [1024, 0, 0, 1508]
    assert capacities([(0.0, 8, 5000), (0.5, 8, 300), (0.5, 8, 300)]) == [1024, 1024, 383]
    assert capacities([(0.0, 8, 5000), (0.0, 64, 5000), (0.0, 64, 5000)]) == [1024, 1024, 0]
    assert capacities([(0.0, 8, 1 << 40), (0.0, 8, 1)]) == [1024, 0]
