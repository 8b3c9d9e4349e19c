"""Large launches of the binary16 matrix-core kernel (launch shape 0), checked as tests/test_gpu_f16_matrix.py checks
the others: even and odd rows, a filter block that is nearly empty, one and several channel steps, infinite and
NaN inputs - and that larger workgroups, which shared their weights in LDS, are not back."""

import numpy as np
import pytest

import test_gpu_f16_matrix as matrix
from test_gpu_f16_matrix import torch                  # noqa: F401 (a fixture)

pytestmark = pytest.mark.gpu

# c_out, c_in, n, h, w, stride, pad, keep, elements the input starts after an aligned address, what is launched
CASES = [
    (130, 17, 1, 256, 256, 1, 1, 0.3, 0, 1),
    (66, 37, 1, 365, 361, 1, 0, 0.3, 0, 0),
    (128, 16, 43, 56, 56, 1, 1, 0.3, 1, 0),            # one channel step; even rows at an odd address; tiles over images
]
NON_FINITE = [(130, 17, 1, 256, 256, 1, 1), (70, 20, 1, 365, 361, 1, 0)]


@pytest.mark.parametrize("case", CASES)
def test_large_launches(torch, case):
    matrix.test_matrix_kernel(torch, case)


@pytest.mark.parametrize("shape", NON_FINITE)
def test_large_launches_not_finite_inputs(torch, shape):
    matrix.test_infinite_and_nan_inputs(torch, shape)


def test_where_it_is_taken(torch):
    """Some 256 workgroups of 128 filters x 512 pixels and more are twice as many of 256 pixels."""
    rng = np.random.default_rng(1)
    for c_out, side, launches in ((128, 56, 1), (64, 56, 5), (128, 54, 1)):
        _, L = matrix._layer(rng, c_out, 16, 0.3, 1, 1)
        assert matrix._launches(L, None, 42, side, side) == launches, (c_out, side)
        L.close()
