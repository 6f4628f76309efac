"""The pair histogram's workgroups, on the CPU: no 32-bit bin of a workgroup can overflow, whatever the number of disks
and the range that the library accepts, and the ordinary ranges keep their 1,024 workgroups."""
import math
import subprocess

import pytest

from paper_1409_6948_amd import build as B

PROGRAM = r"""
#include <cstdio>
#include <cstdlib>
#include "ec_internal.h"
int main(int argc, char** argv) {
  for (int i = 1; i + 1 < argc; i += 2)
    std::printf("%lld\n", (long long)ec::histogram_groups(std::atoll(argv[i]), std::atof(argv[i + 1])));
}
"""


@pytest.fixture(scope="module")
def groups(tmp_path_factory):
    d = tmp_path_factory.mktemp("groups")
    (d / "g.cpp").write_text(PROGRAM)
    r = subprocess.run(["g++", "-O2", "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-I", B.CSRC, "-I", "/opt/rocm/include",
                        "-o", str(d / "g"), str(d / "g.cpp")], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]

    def ask(n, u):
        return int(subprocess.run([str(d / "g"), str(n), repr(u)], capture_output=True, text=True).stdout)
    return ask


# 2^29 - 4 disks are the most of a walled system, 61 diameters the widest cell; 2048 disks the most of one periodic cell
@pytest.mark.parametrize("n", [1, 256, 257, 2048, 1 << 18, (1 << 18) + 1, 10 ** 6, 1 << 24, (1 << 29) - 4])
@pytest.mark.parametrize("u", [1.001, 1.5, 6.0, 30.0, 61.0, 500.0])
def test_no_bin_can_overflow(groups, n, u):
    g = groups(n, u)
    blocks = -(-n // 256)
    assert 1 <= g <= blocks
    # the busiest workgroup's disks, each with all its neighbours in one bin: a triangular packing's
    # (2 pi / sqrt 3) u^2 and the rim's pi u, every pair adding 2
    disks = min(n, 256 * -(-blocks // g))
    most = disks * 2 * min(n, 2 * math.pi / math.sqrt(3) * u * u + math.pi * u)
    assert most < 2 ** 32 or g == blocks
    if most * 2 < 2 ** 32 * (1024 / max(blocks, 1024)):
        assert g == min(blocks, 1024)


def test_ordinary_ranges_keep_their_workgroups(groups):
    assert groups(1 << 20, 1.5) == 1024
    assert groups(1 << 24, 4.0) == 1024
    assert groups(100000, 6.0) == 391
