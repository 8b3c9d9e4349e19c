"""GPU parity of the binary16 matrix-core kernel (csrc/kernel_f16.hip) where it can go wrong: odd and
even rows (one and two pixels per load and store), strips, tiles that span images, channel and
filter counts around its blocks, both strides, every launch shape (asserted) - and inputs that are
infinite or NaN, which must reach only the outputs whose kept weights meet them, in every launch
shape; subnormal values; and layers that keep the walk over the kept weights."""

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


def _layer(rng, c_out, c_in, keep, stride, pad, dense=False):
    ids = rng.integers(0, 8, (c_out, c_in), dtype=np.uint8)
    mask = (rng.random((c_out, c_in)) < keep).astype(np.uint8)
    wt = (rng.standard_normal((c_out, c_in, 3, 3)) * 0.3).astype(np.float32)
    lib = wl.pattern_library(wl.PATTERN_SEED)
    return (wt, ids, mask, lib), B.Layer(wt, ids, mask, lib, stride=stride, pad=pad, dense=dense)


# What a case launches (see f16_choice in csrc/kernels.hpp): twice the launch shape - 0 blocks of 64 filters
# x 128 pixels a wavefront, 1 64 x 64 (stride 2), 2 32 x 64, 3 four wavefronts on 32 x 64, 4 eight and 5 four
# on 32 x 32 - plus one where rows are staged in pairs.
def _launches(layer, pointer, n, h, w):
    choice = B.lib().patdnn_internal_f16_choice
    choice.argtypes = [ctypes.c_void_p] * 2 + [ctypes.c_int32] * 3
    choice.restype = ctypes.c_int32
    return choice(layer.handle, pointer, n, h, w)


# c_out, c_in, n, h, w, stride, pad, keep, elements the input starts after an aligned address, what is launched
CASES = [
    (130, 17, 2, 130, 128, 1, 1, 0.3, 0, 1),   # last filter block nearly empty
    (130, 17, 2, 130, 129, 1, 1, 0.3, 0, 0),   # ... odd rows
    (70, 20, 10, 107, 106, 2, 1, 0.3, 0, 3),   # stride 2, 53 output columns: pairs in, single values out
    (70, 20, 10, 107, 105, 2, 1, 0.3, 0, 2),
    (128, 33, 1, 182, 181, 1, 1, 0.3, 0, 4),
    (64, 64, 8, 112, 112, 1, 1, 0.3, 0, 5),
    (70, 20, 3, 107, 106, 2, 1, 0.3, 0, 7),
    (96, 31, 6, 66, 67, 2, 0, 0.4, 0, 10),
    (40, 16, 5, 120, 99, 1, 0, 0.3, 0, 4),
    (33, 5, 3, 161, 160, 1, 1, 0.5, 1, 4),     # even rows at an odd address
    (64, 64, 70, 14, 15, 1, 1, 0.3, 0, 6),     # channels split over wavefronts, tiles over images
    (200, 70, 9, 20, 30, 1, 1, 0.3, 0, 7),
    (33, 130, 2, 11, 7, 1, 1, 0.3, 0, 8),
    (16, 64, 1, 32, 34, 1, 1, 0.5, 0, 11),
    (31, 48, 40, 1, 1, 1, 1, 1.0, 0, 10),      # one pixel an image
    (48, 80, 33, 4, 4, 2, 0, 0.6, 0, 9),       # a strip of one column, rounded up to a pair
    (8, 100, 2, 40, 130, 2, 1, 0.4, 0, 9),     # stride 2, three strips of 22 columns, the last one not full
]


def test_cases_launch_every_shape():
    assert {c[-1] for c in CASES} == set(range(12)) == {c[-1] for c in NON_FINITE}


@pytest.mark.parametrize("case", CASES)
def test_matrix_kernel(torch, case):
    from oracle import fp16
    c_out, c_in, n, h, w, stride, pad, keep, shift, launches = case
    rng = np.random.default_rng(c_out * 1000 + h * 40 + w)
    (wt, ids, mask, lib), L = _layer(rng, c_out, c_in, keep, stride, pad)
    bias = rng.standard_normal(c_out).astype(np.float32)
    x16 = fp16.to_f16(rng.standard_normal((n, c_in, h, w)))
    x16.reshape(-1)[::37] = fp16.to_f16(np.float64(3e-7))          # subnormal
    want16, exact = fp16.conv2d_f16(wt, ids, mask, lib, x16, bias, stride=stride, pad=pad, relu=True, skip_removed=True)
    xt = torch.zeros(x16.size + shift, dtype=torch.float16, device="cuda")[shift:].view(x16.shape)
    xt.copy_(torch.from_numpy(x16))
    guard, numel = 2048, int(np.prod(want16.shape))
    buf = torch.full((numel + 2 * guard,), 7.0, dtype=torch.float16, device="cuda")
    out = buf[guard:guard + numel].view(want16.shape)
    print(f"  {case}", flush=True)
    assert _launches(L, xt.data_ptr(), n, h, w) == launches
    L.conv2d_f16(xt, torch.from_numpy(bias).cuda(), out, relu=True)
    torch.cuda.synchronize()
    assert bool((buf[:guard] == 7.0).all()) and bool((buf[guard + numel:] == 7.0).all())
    # half a binary16 spacing for the rounding, 1e-5 of the largest output for the fp32 sum
    got, scale = out.cpu().numpy().astype(np.float64), float(np.abs(exact).max())
    bound = 2.0 ** -11 * np.maximum(np.abs(exact), 2.0 ** -14) + 1e-5 * scale
    assert float((np.abs(got - exact) / bound).max()) <= 1.0
    L.close()


# c_out, c_in, n, h, w, stride, what is launched
NON_FINITE = [(130, 17, 2, 130, 128, 1, 1), (130, 17, 2, 130, 129, 1, 0), (70, 20, 10, 107, 106, 2, 3), (70, 20, 10, 107, 105, 2, 2),
              (40, 24, 5, 97, 96, 1, 5), (40, 24, 5, 97, 95, 1, 4), (40, 24, 2, 97, 96, 1, 7), (40, 24, 2, 97, 95, 1, 6),
              (33, 130, 2, 11, 8, 2, 9), (33, 130, 2, 11, 9, 2, 8), (64, 64, 70, 7, 8, 1, 11), (64, 64, 70, 7, 7, 1, 10)]


@pytest.mark.parametrize("shape", NON_FINITE)
def test_infinite_and_nan_inputs(torch, shape):
    from oracle import fp16
    c_out, c_in, n, h, w, stride, launches = shape
    rng = np.random.default_rng(sum(shape[:-1]))
    (wt, ids, mask, lib), L = _layer(rng, c_out, c_in, 0.3, stride, 1)
    # kept weights of zero, which an infinite input turns into NaN, and of either sign
    L.close()
    zero = rng.random(wt.shape) < 0.1
    wt[zero] = np.where(rng.random(zero.sum()) < 0.5, 0.0, -0.0)
    L = B.Layer(wt, ids, mask, lib, stride=stride)
    x16 = fp16.to_f16(rng.standard_normal((n, c_in, h, w)))
    for v in (np.inf, -np.inf, np.nan) * 3:
        x16[rng.integers(n), rng.integers(c_in), rng.integers(h), rng.integers(w)] = v
    x16[0, 0, 2, 2], x16[0, 1, 2, 3], x16[0, 2, 3, 2] = np.inf, -np.inf, np.inf       # that meet in one output
    bias = rng.standard_normal(c_out).astype(np.float32)
    # the walk over the kept weights, on the same values in fp32
    W = B.Layer(fp16.to_f16(wt).astype(np.float32), ids, mask, lib, stride=stride)
    W.set_config(0)
    bt = torch.from_numpy(bias).cuda()
    want16 = fp16.to_f16(W.conv2d(torch.from_numpy(x16.astype(np.float32)).cuda(), bt).cpu().numpy())
    W.close()
    print(f"  {shape}", flush=True)
    xt = torch.from_numpy(x16).cuda()
    assert _launches(L, xt.data_ptr(), n, h, w) == launches
    got = L.conv2d_f16(xt, bt).cpu().numpy()
    assert np.isnan(want16).any() and np.isposinf(want16).any() and np.isneginf(want16).any()
    np.testing.assert_array_equal(np.isnan(got), np.isnan(want16))
    np.testing.assert_array_equal(got[np.isinf(want16)], want16[np.isinf(want16)])
    ok = np.isfinite(want16)
    assert np.isfinite(got[ok]).all()
    # one binary16 spacing, and 1e-5 of the largest sum
    err = np.abs(got[ok].astype(np.float64) - want16[ok])
    assert float((err - 2.0 ** -10 * np.abs(want16[ok])).max()) <= 1e-5 * float(np.abs(want16[ok]).max()) + 2.0 ** -24
    L.close()


def test_infinite_inputs_cost_no_more_than_the_walk(torch):
    """One input in ten thousand infinite, which touches nearly every tile.  The walk over the kept
    weights takes 20 times what the finite layer takes on the matrix cores."""
    rng = np.random.default_rng(3)
    _, L = _layer(rng, 128, 128, 1 / 3.6, 1, 1)
    x = torch.randn(64, 128, 56, 56, device="cuda").half()
    out = torch.empty_like(x)

    def ms():
        best = []
        for _ in range(5):
            e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            e0.record()
            L.conv2d_f16(x, None, out)
            e1.record()
            torch.cuda.synchronize()
            best.append(e0.elapsed_time(e1))
        return min(best)

    finite = ms()
    x.view(-1)[torch.randperm(x.numel(), device="cuda")[:x.numel() // 10000]] = float("inf")
    some = ms()
    print(f"  finite {finite:.3f} ms, with infinities {some:.3f} ms", flush=True)
    assert some <= 20 * finite
    L.close()


@pytest.mark.parametrize("case", [(24, 20, 3, 13, 13, 1, False), (32, 16, 2, 21, 20, 2, False), (48, 5, 2, 18, 33, 1, True)])
def test_weights_beyond_binary16(torch, case):
    """A weight that is infinite in binary16 meets zero padding and zero inputs as a NaN, so such layers
    keep the walk over the kept weights; the other filters are as ever."""
    from oracle import fp16
    c_out, c_in, n, h, w, stride, dense = case
    rng = np.random.default_rng(sum(case))
    ids = rng.integers(0, 8, (c_out, c_in), dtype=np.uint8)
    mask = (rng.random((c_out, c_in)) < (1.0 if dense else 0.3)).astype(np.uint8)
    wt = (rng.standard_normal((c_out, c_in, 3, 3)) * 0.3).astype(np.float32)
    lib = wl.pattern_library(wl.PATTERN_SEED)
    mask[7, 3] = 1
    wt[7, 3] = 1e6
    bias = rng.standard_normal(c_out).astype(np.float32)
    x16 = fp16.to_f16(np.maximum(rng.standard_normal((n, c_in, h, w)), 0.0))
    L = B.Layer(wt, ids, mask, lib, stride=stride, dense=dense)
    got = L.conv2d_f16(torch.from_numpy(x16).cuda(), torch.from_numpy(bias).cuda()).cpu().numpy()
    L.close()
    others = np.arange(c_out) != 7
    # the oracle, without the infinite weight
    wt[7, 3] = 0.0
    _, exact = fp16.conv2d_f16(wt, ids, mask, lib, x16, bias, stride=stride, pad=1, dense=dense, skip_removed=True)
    bound = 2.0 ** -11 * np.maximum(np.abs(exact), 2.0 ** -14) + 1e-5 * float(np.abs(exact).max())
    assert float((np.abs(got.astype(np.float64) - exact) / bound)[:, others].max()) <= 1.0
    assert not np.isfinite(got[:, 7]).any()


@pytest.mark.parametrize("inputs,weights", [(3e-7, 0.3), (1.0, 3e-7), (3e-7, 30.0)])
def test_subnormal_values(torch, inputs, weights):
    """Binary16 inputs, weights and results below 2^-14: none of them is flushed to zero."""
    from oracle import fp16
    rng = np.random.default_rng(8)
    c_out, c_in, n, h, w = 40, 70, 2, 20, 21
    ids = rng.integers(0, 8, (c_out, c_in), dtype=np.uint8)
    mask = (rng.random((c_out, c_in)) < 0.5).astype(np.uint8)
    wt = (rng.standard_normal((c_out, c_in, 3, 3)) * weights).astype(np.float32)
    lib = wl.pattern_library(wl.PATTERN_SEED)
    x16 = fp16.to_f16(rng.standard_normal((n, c_in, h, w)) * inputs)
    _, exact = fp16.conv2d_f16(wt, ids, mask, lib, x16, None, stride=1, pad=1, skip_removed=True)
    L = B.Layer(wt, ids, mask, lib)
    got = L.conv2d_f16(torch.from_numpy(x16).cuda(), None).cpu().numpy().astype(np.float64)
    L.close()
    # half a binary16 spacing, and the fp32 sum's 1e-5 of the largest output
    bound = 2.0 ** -11 * np.maximum(np.abs(exact), 2.0 ** -14) + 1e-5 * float(np.abs(exact).max())
    assert float(np.abs(exact).max()) > 32 * 2.0 ** -24
    assert float((np.abs(got - exact) / bound).max()) <= 1.0
