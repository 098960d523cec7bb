"""How many blocks of sweeps a patch solve queues before the host looks at its
state again (csrc/patch_schedule.hpp, host code without HIP): compiled with the
host compiler and asked directly."""
import math
import os
import shutil
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))),
                    "paper_1307_6748_amd", "csrc")
MAIN = """
#include <cstdio>
#include <cstdlib>
#include "patch_schedule.hpp"
int main(int argc, char** argv)
{
    for (int i = 1; i + 3 < argc; i += 4)
        std::printf("%d\\n", isis::next_patch_batch(std::atoi(argv[i]), std::atof(argv[i + 1]),
                                                   std::atof(argv[i + 2]), std::atof(argv[i + 3])));
}
"""


@pytest.fixture(scope="module")
def rule(tmp_path_factory):
    cxx = shutil.which("g++")
    if cxx is None:
        pytest.skip("g++ is needed")
    d = tmp_path_factory.mktemp("patch")
    (d / "main.cpp").write_text(MAIN)
    exe = str(d / "rule")
    subprocess.run([cxx, "-std=c++17", "-I", CSRC, "-o", exe, str(d / "main.cpp")], check=True)

    def ask(*cases):
        args = [repr(v) for c in cases for v in c]
        out = subprocess.run([exe, *args], check=True, capture_output=True, text=True).stdout
        return [int(v) for v in out.split()]
    return ask


def test_as_many_blocks_as_the_factor_predicts(rule):
    # halved by a block of one; 3 and 2.9 blocks left, 40 left, 0.5 per two blocks
    assert rule((1, 1.0, 0.5, 0.5 / 8.001), (1, 1.0, 0.5, 0.5 / 2 ** 2.9), (1, 1.0, 0.5, 1e-12),
                (2, 1.0, 0.5, 0.5 / 8.001)) == [4, 3, 4, 7]
    assert rule((4, 1.0, 0.5, 1e-30), (16, 1.0, 0.5, 1e-30), (64, 1.0, 0.5, 1e-80),
                (1, 1.0, 0.5, 0.0)) == [16, 64, 64, 4]


@pytest.mark.parametrize("batch", [1, 2, 4, 8, 64])
def test_one_block_where_less_than_one_is_left_or_nothing_fell(rule, batch):
    """More would run past the end: a block may be hundreds of launches."""
    rho = 0.25
    near = [(batch, 1.0, rho ** batch, rho ** (batch + f)) for f in (0.01, 0.5, 0.99)]
    rising = [(batch, 1.0, 1.0, 1e-8), (batch, 1.0, 3.0, 1e-8), (batch, 1.0, math.inf, 1e-8),
              (batch, math.inf, 1.0, 1e-8), (batch, 1.0, math.nan, 1e-8)]
    assert rule(*near, *rising) == [1] * (len(near) + len(rising))
