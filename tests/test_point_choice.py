"""The launch of the pointwise convolution (csrc/tern_point_choice.h, host code) over the sizes that it takes."""
import os
import shutil
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_1801_09449_amd", "csrc")

SOURCE = r"""
#include "tern_point_choice.h"
#include <cstdio>
#include <random>
using namespace tern;

int main()
{
    long lost = 0, odd = 0, late = 0, uneven = 0;
    std::mt19937_64 r(4);
    for (int i = 0; i < 200000; ++i) {
        const int64_t voxels = 1 + (int64_t)(r() % ((uint64_t)0x7fffffff >> (r() % 31)));
        const int layers = r() % 4 ? 1 : 1 + (int)(r() % (65535 >> (r() % 16))), words = 1 + (int)(r() % 8);
        const int c_out = 1 + (int)(r() % ((1u << 19) >> (r() % 19)));
        const bool packed = layers == 1 && r() % 3;
        const PointLaunch l = point_launch(voxels, layers, c_out, words, packed);
        const int64_t blocks = (voxels + 31) / 32, waves = l.gx * kPointWaves * l.groups;
        // every block of every filter is some wave's, and the grid is one
        lost += l.gx * kPointWaves * l.blocks_per_wave < blocks || l.blocks_per_wave < 1 || l.gx < 1 || l.gx > 0x7fffffff ||
                (int64_t)l.groups * l.nb * 32 < c_out || (l.nb == 2 && words > 4);
        odd += packed && words <= 4 && l.groups > 1 && l.gx % 8 != 0;
        // no wave of a large packed launch waits for another's end, unless waves are as long as they get
        late += l.six && waves > 4096 + 4 * l.groups && l.blocks_per_wave < 256 && l.gx > 8;
    }
    // a block fewer than an even number of them is the same launch
    for (int words = 1; words <= 4; ++words)
        for (int c_out : {64, 128, 192, 256})
            for (int64_t even : {131072, 262144, 524288}) {
                const PointLaunch a = point_launch(even, 1, c_out, words, true), b = point_launch(even - 32, 1, c_out, words, true);
                uneven += a.blocks_per_wave != b.blocks_per_wave || a.six != b.six || a.nb != b.nb;
            }
    printf("%ld %ld %ld %ld\n", lost, odd, late, uneven);
}
"""


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")
def test_pointwise_launches(tmp_path):
    """All blocks covered, workgroups of a voxel on one XCD, no wave more than are resident, and no size that is
    launched unlike the one beside it."""
    (tmp_path / "t.cpp").write_text(SOURCE)
    subprocess.run(["g++", "-O2", "-std=c++17", "-I", CSRC, str(tmp_path / "t.cpp"), "-o", str(tmp_path / "t")], check=True)
    out = subprocess.run([str(tmp_path / "t")], check=True, capture_output=True, text=True, timeout=300).stdout
    assert out.split() == ["0", "0", "0", "0"]
