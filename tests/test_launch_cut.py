"""The cut of a box kernel's (box, angle) workgroups into launches: every
launch stays below HIP's 2^32 lanes, the launches cover every box and angle
once, and what fits one launch stays one."""
import os
import subprocess

import pytest

import paper_2211_03516_amd as vam

CSRC = os.path.join(os.path.dirname(vam.__file__), "csrc")
PROGRAM = r"""
#include <cstdio>
#include <cstdlib>
#include "launch_cut.h"
int main(int, char** v) {
  const vam::LaunchCut c = vam::launch_cut(atoll(v[1]), atoll(v[2]), atoi(v[3]));
  printf("%d %d\n", c.boxes, c.angles);
}
"""


@pytest.fixture(scope="module")
def cut(tmp_path_factory):
    d = tmp_path_factory.mktemp("cut")
    (d / "cut.cpp").write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-Wall", "-I", CSRC, str(d / "cut.cpp"), "-o", str(d / "cut")], check=True)

    def run(*a):
        out = subprocess.run([str(d / "cut")] + [str(x) for x in a], check=True, capture_output=True, text=True)
        return tuple(int(x) for x in out.stdout.split())
    return run


# 41 811 boxes: a refracting vial at 512^3; 65 000: an index-matched one
@pytest.mark.parametrize("boxes,angles,threads", [
    (1, 1, 256), (770, 180, 768), (41811, 90, 768), (41811, 200, 512), (41811, 201, 512), (41811, 270, 512),
    (41811, 359, 512), (41811, 360, 512), (41811, 180, 768), (65000, 129, 512), (65000, 257, 256), (65000, 258, 256),
    (24700, 359, 512), (13000000, 1, 512), (13000000, 3, 512), (40000000, 7, 768), (3, 65535, 512),
    (8388600, 1, 512), (8388601, 1, 512), (8388608, 1, 512), (16777208, 1, 256), (5592400, 1, 768), (5592401, 1, 768),
    (2000000000, 2, 768),
])
def test_launches_stay_below_the_lane_limit(cut, boxes, angles, threads):
    nb, na = cut(boxes, angles, threads)
    assert 1 <= nb <= boxes and 1 <= na <= angles
    lanes = (nb * na + 7) // 8 * 8 * threads      # grids are padded to a multiple of 8 workgroups
    assert lanes < 2 ** 32
    fits = (boxes * angles + 7) // 8 * 8 * threads < 2 ** 32
    assert fits == ((nb, na) == (boxes, angles))
    if nb < boxes:                                # boxes are cut only where one angle's do not fit
        assert na == 1 and (boxes + 7) // 8 * 8 * threads >= 2 ** 32
    # the parts are alike: none of them is empty
    for n, part in ((boxes, nb), (angles, na)):
        parts = -(-n // part)
        assert (parts - 1) * part < n <= parts * part
