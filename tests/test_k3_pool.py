"""The arithmetic of K3's walk over the pool of candidates, compiled for the CPU: it
visits every place once and ends, up to the most units a controller takes.  In
int32 the walk over 2^31 - 1,023 units and more had no end, and the one over
2^31 - 255 units and more visited nothing."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2606_00539_amd", "csrc")
MOST = 2**31 - 1                      # units

PROGRAM = """
#include <cstdio>
#include <cstdlib>
#include "k3_pool.h"
int main(int argc, char** argv) {
  const int wgs = atoi(argv[1]), shift = atoi(argv[2]);
  const uint32_t places = gnmr::pool_places(wgs, shift), n = gnmr::pool_rounds(places, 1024);
  uint32_t next = 0, r = 0;   // the kernel's places: r * 1024 + thread, those below `places`
  for (; r < n; ++r) {
    if (r * 1024u != next) return 1;
    next += 1024;
  }
  printf("%u %u\\n", places, r);
}
"""


@pytest.fixture(scope="module")
def walk(tmp_path_factory):
    d = tmp_path_factory.mktemp("pool")
    (d / "walk.cpp").write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-fsanitize=undefined",
                    "-fno-sanitize-recover=undefined", "-I", CSRC, "-o", str(d / "walk"),
                    str(d / "walk.cpp")], check=True)
    return lambda *a: tuple(map(int, subprocess.run(
        [str(d / "walk"), *map(str, a)], check=True, capture_output=True, text=True,
        timeout=60).stdout.split()))


# K2 workgroups of 256, 4 and 1 units
@pytest.mark.parametrize("units,shift", [
    (1, 8), (16385, 8), (MOST // 2, 8), (MOST - 1279, 8), (MOST - 1023, 8), (MOST - 256, 8),
    (MOST - 255, 8), (MOST, 8), (524288, 2), (32768, 0)])
def test_the_walk_covers_the_places_and_ends(walk, units, shift):
    wgs = -(-units // (1 << shift))
    places, rounds = walk(wgs, shift)
    assert places == wgs << shift and units <= places < units + (1 << shift)
    assert rounds == -(-places // 1024)
