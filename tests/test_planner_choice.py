"""The configuration that the library chooses where none is set, against measured times: for each
layer the microseconds of the FKW walk, of the tiled kernel and of the fastest tap-product
configuration, as one MI355X took them.  The choice has to be a kernel that is not far behind the
fastest of the three.  Runs on host-only handles."""

import ctypes

import numpy as np
import pytest

from paper_2001_00138_amd import binding as B
from paper_2001_00138_amd import workloads as wl

# c_in, c_out, n, h, w, pad, patterns, kept kernels; us of walk, tiled, tap-product
MEASURED = [
    ((16, 16, 1, 32, 32, 1, 8, 117), (10, 19, 11)),
    ((48, 16, 1, 9, 7, 0, 8, 224), (10, 37, 13)),
    ((32, 104, 10, 8, 7, 1, 8, 943), (11, 27, 13)),
    ((30, 24, 25, 8, 8, 1, 24, 199), (12, 27, 13)),
    ((24, 96, 2, 12, 18, 1, 24, 627), (11, 21, 12)),
    ((24, 32, 1, 120, 120, 1, 6, 768), (21, 39, 17)),
    ((40, 344, 2, 19, 16, 1, 8, 13760), (25, 66, 19)),
    ((104, 24, 7, 25, 16, 0, 8, 1232), (26, 98, 18)),
    ((88, 32, 19, 21, 22, 0, 8, 1421), (27, 82, 20)),
    ((76, 28, 2, 107, 81, 1, 24, 1065), (49, 70, 22)),
    ((376, 112, 1, 14, 21, 0, 8, 42112), (116, 566, 39)),
    ((224, 26, 2, 93, 145, 1, 24, 5824), (334, 332, 50)),
    ((464, 40, 9, 52, 52, 1, 8, 5065), (218, 286, 65)),
    ((112, 112, 45, 20, 20, 1, 12, 12544), (334, 181, 83)),
    ((312, 208, 57, 40, 39, 0, 6, 18001), (2329, 403, 419)),
    ((200, 288, 3, 150, 156, 0, 8, 57600), (5976, 395, 562)),
    ((312, 95, 3, 211, 224, 1, 56, 29640), (7313, 629, 793)),
    ((504, 131, 14, 110, 127, 0, 6, 18279), (5361, 632, 755)),
    ((512, 512, 24, 28, 28, 1, 8, 262144), (6865, 824, 543)),
    ((512, 512, 64, 28, 28, 1, 56, 72745), (6021, 825, 739)),
    ((416, 328, 3, 217, 179, 0, 56, 37727), (9243, 992, 1213)),
    ((64, 64, 64, 224, 224, 1, 8, 1149), (7722, 624, 797)),
]


@pytest.mark.parametrize("case", MEASURED)
def test_choice_is_close_to_the_fastest(case):
    (c_in, c_out, n, h, w, pad, patterns, kept), (walk, tiled, taps) = case
    rng = np.random.default_rng(kept)
    mask = np.zeros(c_out * c_in, np.uint8)
    mask[rng.permutation(mask.size)[:kept]] = 1
    lib = wl.pattern_library(wl.PATTERN_SEED, patterns) if patterns < 56 else wl.pattern_universe()
    L = B.Layer(rng.standard_normal((c_out, c_in, 3, 3), dtype=np.float32), rng.integers(0, patterns, (c_out, c_in), dtype=np.uint8),
                mask.reshape(c_out, c_in), lib, pad=pad, host_only=True)
    choice = B.lib().patdnn_internal_choice
    choice.argtypes = [ctypes.c_void_p] + [ctypes.c_int32] * 3 + [ctypes.c_size_t, ctypes.c_void_p]
    cfg = B.Config()
    assert choice(L.handle, n, h, w, 128 << 20, ctypes.byref(cfg)) == 0
    name = B.patdnn_variant_name(cfg.variant)
    us = walk if name == "fkw" else taps if name.startswith("taps") else tiled
    # the estimates are up to 40 % off, and up to 10 us the launch is most of it
    assert us <= 1.4 * min(walk, tiled, taps), name
    L.close()
