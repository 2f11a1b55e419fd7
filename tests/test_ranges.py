"""Index arithmetic near lists of 2^31 - 1 entries: evaluated by the host compiler, for which a sum that does
not fit 32 bits is no constant, so that it does not compile."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

CHECKS = r"""
#include "pipad_ranges.h"
using namespace pipad;
constexpr int32_t most = 2147483647;
// a tile's 64 lanes of 10 entries (8 in the base), from the last places on that a list can have
static_assert(!reaches(most - 512, 63 * 10 + 10, most));
static_assert(!reaches(most - 513, 63 * 8 + 10, most));
static_assert(reaches(most - 514, 63 * 8 + 10, most));
static_assert(!reaches(most, 1, most) && reaches(most, 0, most) && reaches(0, most, most));
static_assert(reaches(0, 514, 514) && !reaches(0, 514, 513) && !reaches(0, 1, 0));
static_assert(place_in(most - 1, 639, most) == most - 1);
static_assert(place_in(most - 512, 639, most) == most - 1 && place_in(most - 512, 511, most) == most - 1);
static_assert(place_in(most - 512, 510, most) == most - 2 && place_in(0, most - 1, most) == most - 1);
static_assert(place_in(0, 0, 1) == 0 && place_in(0, 9, 1) == 0 && place_in(3, 4, 100) == 7);
int main() {}
"""


def test_indices_near_the_longest_list(tmp_path):
    source = tmp_path / "ranges.cpp"
    source.write_text(CHECKS)
    subprocess.run(["g++", "-std=c++17", "-fsyntax-only", "-I", os.path.join(ROOT, "paper_2301_00391_amd", "csrc"), str(source)],
                   check=True)
