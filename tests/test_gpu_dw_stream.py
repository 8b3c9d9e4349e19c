"""Depthwise layers of large tensors (csrc/kernel_dw.hip) give the values of smaller calls, bit for bit: whole rows and
others, both strides, and the stores that leave nothing in the L2s, which inputs of more than 128 MB take at stride 1."""

import ctypes

import numpy as np
import pytest

from paper_2001_00138_amd import binding as B
from paper_2001_00138_amd import workloads as wl

pytestmark = pytest.mark.gpu


# images, channels, h, w, stride; outputs of 16 to 98 MB, none with another kind of store
@pytest.mark.parametrize("n,c,h,w,stride", [(12, 144, 56, 56, 1), (12, 144, 57, 60, 1), (12, 144, 112, 112, 2), (12, 144, 112, 119, 2),
                                            (32, 144, 56, 56, 1), (50, 144, 57, 60, 1), (26, 144, 112, 112, 2), (26, 144, 112, 119, 2)])
def test_large_outputs(n, c, h, w, stride):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    rng = np.random.default_rng(w)
    wt = rng.standard_normal((c, 1, 3, 3)).astype(np.float32)
    ids = rng.integers(0, 8, (c, 1), dtype=np.uint8)
    L = B.Layer(wt, ids, np.ones((c, 1), np.uint8), wl.pattern_library(wl.PATTERN_SEED), stride=stride, pad=1, depthwise=True)
    x = torch.randn((n, c, h, w), device="cuda", generator=torch.Generator("cuda").manual_seed(1))
    bias = torch.randn(c, device="cuda")
    whole = L.conv2d(x, bias, relu=True)
    assert whole.numel() * 4 > 1 << 24
    for i in range(n):
        assert torch.equal(whole[i:i + 1], L.conv2d(x[i:i + 1].contiguous(), bias, relu=True))
    L.close()


def _choice(L, x, out):
    choice = B.lib().patdnn_internal_dw_choice
    choice.argtypes = [ctypes.c_void_p] * 3 + [ctypes.c_int32] * 4
    return choice(L.handle, x.data_ptr(), out.data_ptr(), x.shape[0], x.shape[2], x.shape[3], int(x.element_size() == 2))


# binary16, images, h, w, elements the output starts after an aligned address, what is launched but for the stores (see dw_choice in
# csrc/kernels.hpp); 96 channels, 129 to 135 MB of input
STREAMED = [
    (False, 28, 112, 112, 0, 3),
    (False, 27, 113, 116, 0, 3),     # an odd number of rows
    (True, 56, 112, 112, 0, 5),
    (True, 53, 113, 120, 0, 5),
    (True, 54, 112, 116, 0, 3),      # four outputs a lane: rows of whole 8-byte vectors
    (True, 56, 112, 112, 4, 3),      # ... and an output that is aligned to those only
]


@pytest.mark.parametrize("case", STREAMED)
def test_stores_that_leave_nothing_in_the_l2s(case):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    half, n, h, w, shift, kind = case
    c, guard = 96, 1024
    rng = np.random.default_rng(w + h)
    wt = rng.standard_normal((c, 1, 3, 3)).astype(np.float32)
    ids = rng.integers(0, 8, (c, 1), dtype=np.uint8)
    L = B.Layer(wt, ids, (rng.random((c, 1)) < 0.9).astype(np.uint8), wl.pattern_library(wl.PATTERN_SEED), pad=1, depthwise=True)
    x = torch.randn((n, c, h, w), device="cuda", generator=torch.Generator("cuda").manual_seed(1)).to(torch.float16 if half else torch.float32)
    x.view(-1)[::100_003] = float("inf")
    bias = torch.randn(c, device="cuda")
    run = L.conv2d_f16 if half else L.conv2d
    buf = torch.full((x.numel() + 2 * guard + 8,), 7.0, dtype=x.dtype, device="cuda")
    out = buf[guard + shift:guard + shift + x.numel()].view(x.shape)
    assert x.numel() * x.element_size() > 128 << 20 and _choice(L, x, out) == kind + 4
    run(x, bias, out, relu=True)
    assert bool((buf[:guard + shift] == 7).all()) and bool((buf[guard + shift + x.numel():] == 7).all())
    for i in range(n):
        one = x[i:i + 1].contiguous()
        want = run(one, bias, relu=True)
        assert _choice(L, one, want) < 6
        assert torch.equal(out[i:i + 1].nan_to_num(-1.0), want.nan_to_num(-1.0))
    L.close()
