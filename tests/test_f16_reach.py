"""Binary16 layers with outputs that a 32-bit byte offset does not reach keep the matrix kernel: 2^30 elements are its bound
for the images that one tile touches, beyond which stores go through 64-bit addresses.  Runs on host-only handles."""

import ctypes

import numpy as np
import pytest

from paper_2001_00138_amd import binding as B
from paper_2001_00138_amd import workloads as wl

# c_in, c_out, n, h, w, stride
CASES = [
    (3, 64, 1, 3000, 3000, 1),         # 0.54 * 2^30 elements
    (3, 64, 2, 2160, 3840, 1),         # two images, 0.99
    (16, 64, 2, 2160, 3840, 1),
    (64, 128, 1, 2048, 2048, 1),       # 0.5
    (16, 512, 1, 1100, 1100, 1),
    (64, 256, 1, 2048, 2048, 1),       # 2^30
    (3, 64, 1, 4200, 4200, 1),         # 1.05
    (3, 64, 2, 3000, 3000, 1),         # two images, 1.07
    (3, 40, 1, 5200, 5201, 1),
    (3, 96, 1, 6800, 6801, 2),
    (3, 64, 3, 5700, 5700, 1),         # 1.94 each
]


@pytest.mark.parametrize("case", CASES)
def test_large_outputs_keep_the_matrix_kernel(case):
    c_in, c_out, n, h, w, stride = case
    L = B.Layer(np.ones((c_out, c_in, 3, 3), np.float32), np.zeros((c_out, c_in), np.uint8), np.ones((c_out, c_in), np.uint8),
                wl.pattern_library(wl.PATTERN_SEED), stride=stride, host_only=True)
    choice = B.lib().patdnn_internal_f16_choice
    choice.argtypes = [ctypes.c_void_p] * 2 + [ctypes.c_int32] * 3
    choice.restype = ctypes.c_int32
    got = choice(L.handle, 4096, n, h, w)
    L.close()
    assert 0 <= got < 6                # a shape that does not split the channels: those have the 64-bit stores
