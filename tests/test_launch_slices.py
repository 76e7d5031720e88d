"""The slices of a launch of more threads than HIP takes in one (csrc/launch.hpp), at
counts just below, at and above the limit.  Host code; no GPU."""
import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2411_02268_amd", "csrc")
PROGRAM = """
#include <cstdio>
#include <cstdlib>
#include "launch.hpp"
int main(int, char **v) {
  mgcd::launch_slices(std::atoll(v[1]), std::atoi(v[2]), [](int64_t first, unsigned count) {
    std::printf("%lld %u\\n", (long long)first, count);
  });
}
"""


@pytest.fixture(scope="module")
def slices(tmp_path_factory):
    d = tmp_path_factory.mktemp("slices")
    (d / "s.cpp").write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-Wall", "-Werror", "-I", CSRC, str(d / "s.cpp"), "-o", str(d / "s")],
                   check=True)

    def run(blocks, threads):
        out = subprocess.run([str(d / "s"), str(blocks), str(threads)], check=True, capture_output=True, text=True)
        return [tuple(map(int, line.split())) for line in out.stdout.splitlines()]
    return run


@pytest.mark.parametrize("threads", [64, 256, 512, 1024])
@pytest.mark.parametrize("around", [0, 1, 2, 7])
@pytest.mark.parametrize("off", [-2, -1, 0, 1, 2])
def test_slices(slices, threads, around, off):
    limit = 1 << 32
    blocks = max(around * (limit // threads) + off, 0)
    got = slices(blocks, threads)
    at = 0
    for first, count in got:  # consecutive, none empty, each a launch that HIP takes
        assert first == at and count > 0 and count * threads < limit
        at += count
    assert at == blocks
    assert len(got) == -(-blocks // (limit // threads - 1))  # no more of them than needed
