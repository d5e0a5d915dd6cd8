"""Edge positions at the end of the largest graphs (2^31 - 1 edges): the first edge of every wavefront of a range
(csrc/edge_range.h) against whole numbers of any size."""
import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_1701_01170_amd", "csrc")
MAIN = """
#include <cstdio>
#include <cstdlib>
#include "edge_range.h"
int main(int argc, char** argv) {
  std::printf("%lld", (long long)gr::wave_first_edge((int32_t)std::atoll(argv[1]), std::atoi(argv[2])));
}
"""


@pytest.fixture(scope="module")
def first_edge(tmp_path_factory):
    d = tmp_path_factory.mktemp("range")
    (d / "m.cpp").write_text(MAIN)
    # (the overflow of a 32-bit sum is defined to wrap here, so that it shows as a wrong number)
    subprocess.run(["g++", "-std=c++17", "-O1", "-fwrapv", f"-I{CSRC}", str(d / "m.cpp"), "-o", str(d / "m")], check=True)
    return lambda lo, wave: int(subprocess.run([str(d / "m"), str(lo), str(wave)], capture_output=True, text=True).stdout)


@pytest.mark.parametrize("back", [0, 1, 63, 64, 127, 128, 191, 192, 193, 4096])
@pytest.mark.parametrize("wave", [0, 1, 2, 3])
def test_first_edge_at_the_end(first_edge, back, wave):
    lo = 2 ** 31 - 1 - back
    assert first_edge(lo, wave) == lo + 64 * wave
