"""How an epoch is cut into segments (csrc/segments.hpp), compiled for the host: no GPU is needed."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
MAIN = r"""
#include <cstdio>
#include "segments.hpp"
int main() {
  long long t0, t1, T;
  while (std::scanf("%lld %lld %lld", &t0, &t1, &T) == 3) std::printf("%d\n", halp::segment_steps(t0, t1, T));
}
"""


@pytest.fixture(scope="module")
def steps(tmp_path_factory):
    tmp = tmp_path_factory.mktemp("segments")
    (tmp / "main.cpp").write_text(MAIN)
    subprocess.run(["g++", "-std=c++17", "-Wall", "-Werror", "-I", os.path.join(ROOT, "paper_1803_03383_amd", "csrc"),
                    "-o", str(tmp / "main"), str(tmp / "main.cpp")], check=True)

    def run(cases):
        text = "".join("%d %d %d\n" % c for c in cases)
        out = subprocess.run([str(tmp / "main")], input=text, capture_output=True, text=True, check=True).stdout
        return [int(v) for v in out.split()]
    return run


def test_steps_of_a_segment(steps):
    """A chain that ended more than 2^31 steps before the segment takes none of it (the 32-bit difference wraps)."""
    ends = [0, 1, 7, 8, 100000, 2 ** 31 - 1, 2 ** 31, 2 ** 31 + 5, 3 * 10 ** 9, 3 * 10 ** 9 + 17, 2 ** 32 - 1]
    begins = [0, 8, 99992, 2 ** 31 - 8, 2 ** 31, 3 * 10 ** 9, 2 ** 32 - 8]
    cases = [(t0, t0 + S, T) for t0 in begins for S in (8, 8192, 1 << 20) for T in ends]
    assert (3 * 10 ** 9, 3 * 10 ** 9 + 8192, 100000) in cases
    assert steps(cases) == [max(0, min(t1, T) - t0) for t0, t1, T in cases]
