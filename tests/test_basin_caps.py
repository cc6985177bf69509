"""Sizes of the basins' lists (basin.hip) over the shapes an image may have: the
places fit 32 bits, and the scratch follows the image's voxels, however thin it is."""
import os
import subprocess

import numpy as np
import pytest

from paper_2101_03240_amd import build

SHAPES = [(512, 512, 512), (16, 16, 16), (64, 64, 64), (1, 500, 500), (500, 1, 500), (500, 500, 1), (1, 1, 7),
          (9, 33, 9), (20000, 20000, 1), (20000, 1, 20000), (65535, 1, 32767), (65535, 32767, 1), (1, 65535, 32767),
          (9, 65535, 3640), (65535, 9, 3640), (65535, 992, 33), (1290, 1290, 1290), (2, 32767, 32767)]

SOURCE = r"""
#include <cstdio>
#include <cstdlib>
#include "basin.h"
int main(int n, char** v) {
    for (int i = 1; i + 2 < n; i += 3) {
        ibip::BasinArgs a{};
        ibip::basin_caps(a, ibip_dims{atoi(v[i]), atoi(v[i + 1]), atoi(v[i + 2])});
        printf("%u %u %u %u %zu\n", a.pcap, a.pall, a.ecap, a.eall, ibip::basin_bytes(a));
    }
}
"""


@pytest.fixture(scope="module")
def caps(tmp_path_factory):
    d = tmp_path_factory.mktemp("caps")
    (d / "caps.hip").write_text(SOURCE)
    subprocess.run([build.HIPCC, "-std=c++17", "--offload-host-only", "-I", build.CSRC, str(d / "caps.hip"), "-L",
                    build.HERE, "-l:" + os.path.basename(build.LIB), f"-Wl,-rpath,{build.HERE}", "-o", str(d / "caps")], check=True)
    out = subprocess.run([str(d / "caps"), *(str(q) for s in SHAPES for q in s)], capture_output=True, text=True,
                         check=True)
    return dict(zip(SHAPES, ([int(x) for x in line.split()] for line in out.stdout.splitlines())))


@pytest.mark.parametrize("shape", SHAPES)
def test_lists_fit(caps, shape):
    pcap, pall, ecap, eall, size = caps[shape]
    n = int(np.prod(shape))
    slots = pall // pcap
    assert 1 <= slots <= 64 and pall == slots * pcap and eall == slots * ecap  # (no product of them wrapped)
    assert 2 * (pall + 1) < 2 ** 32 and pall < 2 ** 31 and eall < 2 ** 32
    if n <= 2 ** 18:
        assert pall >= n and eall >= 4 * n  # whatever the image holds
        assert size <= 80 * 2 * n + 20000  # 76 B a voxel, and the last tiles
    else:
        assert 8 * pall >= 0.99 * n and 2 * eall >= 0.99 * n
    if n > 2 ** 20:
        assert size <= 2 * 13 * n
