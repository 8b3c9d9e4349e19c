"""The depthwise kernel of two output rows a lane (csrc/kernel_dw.hip, dw_rows_kernel) against the one that reads element by
element, which layers with a weight that is not finite take: the sums are the same term by term, so every bit is the
same, also where inputs are infinite or NaN.  The latter has its own comparison with the oracle."""

import numpy as np
import pytest

from paper_2001_00138_amd import binding as B
from paper_2001_00138_amd import workloads as wl

pytestmark = pytest.mark.gpu

# c, n, h, w, stride, pad
CASES = [
    (5, 3, 13, 16, 1, 1),        # whole rows, an odd number of them
    (9, 2, 28, 28, 1, 1),        # binary16 rows of whole 8-byte vectors
    (7, 2, 9, 61, 1, 1),         # one, two and three elements over a vector
    (7, 2, 9, 62, 1, 1),
    (7, 2, 10, 63, 1, 1),
    (3, 2, 30, 223, 1, 0),       # rows longer than the columns of a wavefront, without padding
    (33, 4, 17, 14, 1, 0),       # wavefronts that end inside a row
    (4, 2, 3, 300, 1, 1),
    (65, 1, 5, 4, 1, 1),         # one vector a row
    (130, 1, 1, 72, 1, 1),       # one row
    (16, 2, 8, 24, 2, 1),
    (6, 2, 7, 8, 2, 1),
    (9, 3, 15, 37, 2, 1),        # columns of four outputs that reach one to seven past the row
    (9, 3, 16, 38, 2, 1),
    (9, 3, 15, 39, 2, 1),
    (11, 2, 14, 50, 2, 0),
    (11, 2, 13, 51, 2, 0),
    (5, 1, 11, 530, 2, 0),
]


@pytest.mark.parametrize("half", [False, True])
@pytest.mark.parametrize("case", CASES)
def test_same_bits_as_element_by_element(case, half):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    c, n, h, w, stride, pad = case
    rng = np.random.default_rng(c * 1000 + h * 40 + w)
    wt = (rng.standard_normal((c + 1, 1, 3, 3)) * 0.3).astype(np.float32)
    ids = rng.integers(0, 8, (c + 1, 1), dtype=np.uint8)
    keep = (rng.random((c + 1, 1)) < 0.9).astype(np.uint8)
    keep[c] = 1
    lib = wl.pattern_library(wl.PATTERN_SEED)
    layers = []
    for value in (1.0, np.inf):                       # of the last channel
        wt[c] = value
        layers.append(B.Layer(wt, ids, keep, lib, stride=stride, pad=pad, depthwise=True))
    dtype = torch.float16 if half else torch.float32
    x = torch.from_numpy(rng.standard_normal((n, c + 1, h, w)).astype(np.float32)).cuda().to(dtype)
    x.view(-1)[::131] = float("inf")
    x.view(-1)[5::173] = float("nan")
    bias = torch.from_numpy(rng.standard_normal(c + 1).astype(np.float32)).cuda()
    shape = layers[0].output_shape(n, h, w)
    size, guard = int(np.prod(shape)), 64
    for shift_in, shift_out, relu in ((0, 0, True), (1, 0, False), (0, 1, False), (2, 2, True)):
        xs = torch.empty(x.numel() + 8, dtype=dtype, device="cuda")[shift_in:shift_in + x.numel()].view(x.shape)
        xs.copy_(x)
        outs = []
        for L in layers:
            buf = torch.full((size + 2 * guard + 8,), 7.0, dtype=dtype, device="cuda")
            out = buf[guard + shift_out:guard + shift_out + size].view(shape)
            (L.conv2d_f16 if half else L.conv2d)(xs, bias, out, relu=relu)
            assert bool((buf[:guard + shift_out] == 7).all()) and bool((buf[guard + shift_out + size:] == 7).all())
            outs.append(out[:, :c])
        got, want = outs
        assert torch.equal(got.isnan(), want.isnan())
        bits = torch.int16 if half else torch.int32
        ok = ~want.isnan()
        assert torch.equal(got.contiguous().view(bits)[ok], want.contiguous().view(bits)[ok])
    for L in layers:
        L.close()
