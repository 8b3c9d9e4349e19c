"""How the tap-product kernel cuts inputs into tiles (csrc/kernels.hpp: tap_tiles, taps_fit_input),
compiled for the host: several small images share a tile, and the byte offset of a staged pixel from
the tile's first image has 32 bits, so an input that fits must not pass them."""

import ctypes
import os
import subprocess

import pytest

from conftest import ROOT

SOURCE = """
#include <hip/hip_runtime.h>
#include "kernels.hpp"
using namespace patdnn;
static ConvShape shape(int n, int c_in, int c_out, int h, int w, int pad, int pool)
{
    ConvShape s{n, c_in, c_out, h, w, h + 2 * pad - 2, w + 2 * pad - 2, 1, pad, 0};
    s.pool = pool;
    return s;
}
extern "C" int fit(int n, int c_in, int c_out, int h, int w, int pad, int pool) { return taps_fit_input(shape(n, c_in, c_out, h, w, pad, pool)); }
// images of the fullest tile, by the kernel's own placement of a tile's pixels
extern "C" int images(int h, int w, int pad, int pool)
{
    const TapTiles t = tap_tiles(shape(1, 1, 1, h, w, pad, pool));
    int most = 0;
    for (int i = 0; i < kTile; ++i)
        for (int j = 0; j < kTile; ++j) {
            const int si = i / t.py, sj = j / t.px, y = i - si * t.py - pad, x = j - sj * t.px - pad;
            if (si < t.sy && sj < t.sx && y >= 0 && y < h && x >= 0 && x < w) most = std::max(most, si * t.sx + sj + 1);
        }
    return most;
}
"""


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    d = tmp_path_factory.mktemp("tap_tiles")
    (d / "t.cpp").write_text(SOURCE)
    csrc = os.path.join(ROOT, "paper_2001_00138_amd", "csrc")
    r = subprocess.run(["g++", "-O1", "-std=c++17", "-fPIC", "-shared", "-I", os.path.join(ROOT, "tests", "host_model"), "-I", csrc,
                        "-I", os.path.join(ROOT, "include"), str(d / "t.cpp"), "-o", str(d / "t.so")], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-3000:]
    return ctypes.CDLL(str(d / "t.so"))


def test_offsets_inside_a_tile_have_32_bits(lib):
    ten = 0
    for pad in (0, 1):
        for h in range(1, 34):
            for w in range(1, 34):
                if h + 2 * pad < 3 or w + 2 * pad < 3:
                    continue
                for pool in (0, 1):
                    images = lib.images(h, w, pad, pool)
                    ten += images == 10
                    # the largest channel count whose tiles reach no further than 2^30 elements
                    most = (2 ** 30 - 1) // (images * h * w)
                    assert lib.fit(images, most + 1, 8, h, w, pad, pool) == 0, (h, w, pad, pool, images)
                    assert lib.fit(images, most // 2, 8, h, w, pad, pool) == 1, (h, w, pad, pool, images)
    assert ten                            # 8 x 3 without padding: five by two
