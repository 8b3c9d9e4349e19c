"""The depthwise kernel for narrow planes whose rows are no whole vectors (csrc/kernel_dw.hip,
dw_planes_kernel) against the kernels that an input or output that is not 16-byte aligned takes:
the sums are the same term by term, so every bit is the same, also where inputs
are infinite or NaN.  The kernel that reads element by element has its own comparison with the oracle."""

import ctypes

import numpy as np
import pytest

from paper_2001_00138_amd import binding as B
from paper_2001_00138_amd import workloads as wl

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    B.lib()
    return torch


# c, n, h, w, stride, pad, keep
CASES = [
    (960, 3, 7, 7, 1, 1, 1.0),       # several planes a thread, several workgroups an image
    (419, 5, 7, 7, 1, 1, 0.6),       # workgroups over images, a run that ends inside a vector
    (307, 7, 14, 14, 1, 1, 0.8),
    (307, 7, 14, 14, 2, 1, 1.0),
    (299, 7, 17, 9, 2, 1, 1.0),
    (301, 7, 3, 3, 1, 0, 1.0),       # one output a plane
    (300, 35, 1, 1, 1, 1, 1.0),      # one pixel a plane
    (299, 7, 15, 17, 1, 1, 1.0),     # 255 outputs,
    (299, 7, 17, 18, 1, 0, 0.7),     # 240,
    (299, 7, 15, 18, 1, 1, 1.0),     # ... more than a workgroup has threads
    (419, 10, 37, 35, 1, 1, 1.0),
    (419, 10, 35, 37, 2, 0, 0.8),
    (103, 40, 2, 501, 1, 1, 1.0),    # long rows
    (103, 40, 501, 2, 1, 1, 1.0),    # short rows
    (5, 1, 7, 7, 1, 1, 1.0),         # too few planes: the row kernel on both sides
    (4, 2, 67, 67, 1, 1, 1.0),       # too large ones
]
# Rows of more than twelve elements are dw_rows_kernel's; these are not, by what a call is said to launch
PLANES = [
    (960, 3, 7, 7, 1, 1, 1.0),
    (307, 9, 24, 10, 1, 1, 0.7),     # 240 outputs,
    (299, 9, 51, 5, 1, 1, 1.0),      # 255,
    (299, 9, 27, 10, 1, 1, 1.0),     # 270: more than a workgroup has threads
    (419, 5, 40, 11, 1, 1, 1.0),     # 440
    (299, 18, 46, 11, 1, 1, 0.9),    # more than 16 KB of LDS
    (419, 18, 41, 11, 2, 0, 0.8),    # stride 2 without padding
    (307, 40, 13, 9, 2, 1, 1.0),
    (299, 40, 8, 7, 2, 0, 1.0),      # rows of less than eight elements at stride 2
    (103, 40, 501, 2, 1, 1, 1.0),    # and of less than four, 40 KB of LDS
]


def _choice(torch, L, x, out, half):
    choice = B.lib().patdnn_internal_dw_choice
    choice.argtypes = [ctypes.c_void_p] * 3 + [ctypes.c_int32] * 4
    return choice(L.handle, x.data_ptr(), out.data_ptr(), x.shape[0], x.shape[2], x.shape[3], int(half))


def test_tall_narrow_planes_go_to_the_row_kernel(torch):
    rng = np.random.default_rng(1)
    L = B.Layer(rng.standard_normal((419, 1, 3, 3)).astype(np.float32), rng.integers(0, 8, (419, 1), dtype=np.uint8), np.ones((419, 1), np.uint8),
                wl.pattern_library(wl.PATTERN_SEED), depthwise=True)
    for h, w, want in ((40, 11, 1), (61, 11, 2), (120, 11, 2), (13, 13, 2)):
        x = torch.zeros((18, 419, h, w), device="cuda")
        assert _choice(torch, L, x, x, False) == _choice(torch, L, x, x, True) == want, (h, w)
    L.close()


@pytest.mark.parametrize("half", [False, True])
@pytest.mark.parametrize("case", PLANES)
def test_planes_kernel_is_taken_and_gives_the_same_bits(torch, case, half):
    test_same_bits_as_the_row_kernel(torch, case, half, planes=True)


@pytest.mark.parametrize("half", [False, True])
@pytest.mark.parametrize("case", CASES)
def test_same_bits_as_the_row_kernel(torch, case, half, planes=False):
    c, n, h, w, stride, pad, keep = case
    rng = np.random.default_rng(c * 1000 + h * 40 + w)
    L = B.Layer((rng.standard_normal((c, 1, 3, 3)) * 0.3).astype(np.float32), rng.integers(0, 8, (c, 1), dtype=np.uint8),
                (rng.random((c, 1)) < keep).astype(np.uint8), wl.pattern_library(wl.PATTERN_SEED), stride=stride,
                pad=pad, depthwise=True)
    dtype = torch.float16 if half else torch.float32
    x = torch.from_numpy(rng.standard_normal((n, c, h, w)).astype(np.float32)).cuda().to(dtype)
    x.view(-1)[::131] = float("inf")
    x.view(-1)[5::173] = float("nan")
    bias = torch.from_numpy(rng.standard_normal(c).astype(np.float32)).cuda()
    shape = L.output_shape(n, h, w)
    size, guard = int(np.prod(shape)), 64

    def conv(shift_in, shift_out, b, relu):
        xs = torch.empty(x.numel() + 8, dtype=dtype, device="cuda")[shift_in:shift_in + x.numel()].view(x.shape)
        xs.copy_(x)
        buf = torch.full((size + 2 * guard + 8,), 7.0, dtype=dtype, device="cuda")
        out = buf[guard + shift_out:guard + shift_out + size].view(shape)
        if planes:
            assert (_choice(torch, L, xs, out, half) == 1) == (shift_in == shift_out == 0)
        if half:
            L.conv2d_f16(xs, b, out, relu=relu)
        else:
            L.conv2d_ws(xs, b, out, relu=relu)
        torch.cuda.synchronize()
        assert bool((buf[:guard + shift_out] == 7).all()) and bool((buf[guard + shift_out + size:] == 7).all())
        return out.cpu().numpy().view(np.uint16 if half else np.uint32), out

    for b, relu in ((bias, True), (None, False)):
        want, plain = conv(1, 1, b, relu)
        for shifts in ((0, 0), (0, 1), (1, 0)):
            got, out = conv(*shifts, b, relu)
            nan = plain.isnan().cpu().numpy()
            assert np.array_equal(nan, out.isnan().cpu().numpy())
            assert np.array_equal(got[~nan], want[~nan])
    L.close()
