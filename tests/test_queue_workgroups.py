"""Wavefronts per workgroup of the batch's ready queue, on the CPU: whatever a cell's LDS is, the choice keeps as many
wavefronts on a CU as workgroups of one would, and takes four where that costs none."""
import subprocess

import pytest

from paper_1409_6948_amd import build as B

PROGRAM = r"""
#include <cstdio>
#include <cstdlib>
#include "ec_internal.h"
int main(int argc, char** argv) { std::printf("%d\n", ec::queue_cells_per_block(std::atoi(argv[1]), std::atoi(argv[2]))); }
"""


@pytest.fixture(scope="module")
def choose(tmp_path_factory):
    d = tmp_path_factory.mktemp("queue")
    (d / "q.cpp").write_text(PROGRAM)
    r = subprocess.run(["g++", "-O2", "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-I", B.CSRC, "-I", "/opt/rocm/include",
                        "-o", str(d / "q"), str(d / "q.cpp")], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]
    return lambda one, four: int(subprocess.run([str(d / "q"), str(one), str(four)], capture_output=True, text=True).stdout)


# per CU: 160 KiB of LDS, 12 wavefronts by their registers, 256 CUs
@pytest.mark.parametrize("lds,want", [(6000, 4), (12240, 4), (13600, 4), (14500, 1), (20816, 1), (26704, 1), (31700, 1),
                                      (33232, 4), (40960, 4), (41424, 1), (55440, 1), (100000, 1)])
def test_no_resident_wavefront_is_given_up(choose, lds, want):
    one, four = 256 * min(163840 // lds, 12), 256 * 4 * min(163840 // (4 * lds), 3)
    got = choose(one, four)
    assert got == want
    assert (four if got == 4 else one) >= one
