"""GPU parity of dense layers of few input channels on the fp32 matrix cores (csrc/kernel_dense.hip) where it can go
wrong: every channel count, both strides, blocks of pixels that span images and are not full, filters around
its sets, pooled windows (and their time), inputs that are not finite or subnormal - and where the library chooses it."""

import ctypes

import numpy as np
import pytest

from paper_2001_00138_amd import binding as B
from paper_2001_00138_amd import workloads as wl

pytestmark = pytest.mark.gpu
# at most 37 products added in fp32: below 37 * 2^-24 of the sum of the terms' magnitudes
TOL = 1e-5


@pytest.fixture(scope="module")
def torch():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    B.lib()
    return torch


def _variant(name):
    return {B.patdnn_variant_name(v): v for v in range(B.patdnn_num_variants())}[name]


def _layer(rng, c_in, c_out, stride, pad, scale=1.0):
    lib = wl.pattern_library(wl.PATTERN_SEED)
    ids = np.zeros((c_out, c_in), np.uint8)
    mask = np.ones((c_out, c_in), np.uint8)
    wt = (rng.standard_normal((c_out, c_in, 3, 3)) * scale).astype(np.float32)
    dense_lib = np.array([0x1FF], dtype=lib.dtype)
    return (wt, ids, mask, dense_lib), B.Layer(wt, ids, mask, lib, stride=stride, pad=pad, dense=True)


def _choice(L, n, h, w):
    cfg = B.Config()
    choice = B.lib().patdnn_internal_choice
    choice.argtypes = [ctypes.c_void_p] + [ctypes.c_int32] * 3 + [ctypes.c_size_t, ctypes.c_void_p]
    assert choice(L.handle, n, h, w, 0, ctypes.byref(cfg)) == 0
    return B.patdnn_variant_name(cfg.variant)


# c_in, c_out, n, h, w, stride, pad
CASES = [
    (3, 64, 2, 33, 31, 1, 1),
    (3, 64, 3, 224, 224, 1, 1),        # several blocks a wavefront, a share for every XCD
    (1, 16, 5, 7, 7, 1, 1),            # blocks over two images
    (1, 1, 70, 3, 3, 1, 0),            # 32 images in a block
    (2, 33, 4, 9, 200, 2, 1),
    (4, 65, 3, 17, 12, 2, 0),
    (4, 130, 2, 40, 23, 1, 0),
    (3, 31, 1, 1, 50, 1, 1),
    (4, 96, 9, 112, 97, 1, 1),
    (2, 5, 41, 3, 3, 1, 1),            # one window an image, eight images in a block
    (3, 40, 30, 4, 5, 1, 1),
    (1, 70, 11, 5, 9, 2, 1),
]


@pytest.mark.parametrize("case", CASES)
@pytest.mark.parametrize("with_bias", [True, False])
def test_dense_kernel(torch, case, with_bias):
    c_in, c_out, n, h, w, stride, pad = case
    rng = np.random.default_rng(c_in * 1000 + w)
    data, L = _layer(rng, c_in, c_out, stride, pad)
    assert _choice(L, n, h, w) == "dense_mfma"
    bias = rng.standard_normal(c_out).astype(np.float32) if with_bias else None
    x = rng.standard_normal((n, c_in, h, w)).astype(np.float32)
    ref = torch.nn.functional.conv2d(torch.from_numpy(x).double(), torch.from_numpy(data[0]).double(),
                                     None if bias is None else torch.from_numpy(bias).double(), stride, pad)
    bt, guard = None if bias is None else torch.from_numpy(bias).cuda(), 1024
    for relu, pool in ((False, False), (True, False), (True, True)):
        want = torch.relu(ref) if relu else ref
        if pool:
            if min(ref.shape[2:]) < 2:
                continue
            want = torch.nn.functional.max_pool2d(want, 2)
        print(f"  {case} relu={relu} pool={pool}", flush=True)
        buf = torch.full((want.numel() + 2 * guard,), 777.0, device="cuda")
        out = buf[guard:guard + want.numel()].view(want.shape)
        L.conv2d_ws(torch.from_numpy(x).cuda(), bt, out, relu=relu, pool=pool)
        assert bool((buf[:guard] == 777.0).all()) and bool((buf[guard + want.numel():] == 777.0).all())
        assert float((out.cpu().double() - want).abs().max() / ref.abs().max()) <= TOL
    L.close()


@pytest.mark.parametrize("stride", [1, 2])
def test_not_finite_inputs_and_subnormal_results(torch, stride):
    """Infinite and NaN inputs give what the walk over the kept weights gives, and tiny numbers are not lost."""
    rng = np.random.default_rng(5)
    for scale, spread in ((1.0, True), (1e-20, False)):
        data, L = _layer(rng, 3, 40, stride, 1, scale)
        x = rng.standard_normal((2, 3, 40, 37)).astype(np.float32)
        if spread:
            kind = rng.random(x.shape)
            x[kind < 0.01] = np.nan
            x[kind < 0.006] = -np.inf
            x[kind < 0.004] = np.inf
        else:
            x *= np.float32(1e-20)
        got = {}
        for name in ("fkw", "dense_mfma"):
            L.set_config(_variant(name))
            got[name] = L.conv2d(torch.from_numpy(x).cuda(), None, relu=False).cpu().numpy()
        L.close()
        a, b = got["fkw"], got["dense_mfma"]
        assert np.array_equal(np.isnan(a), np.isnan(b)) and np.array_equal(a[np.isinf(a)], b[np.isinf(a)])
        ok = np.isfinite(a)
        # half a subnormal spacing for each of the 28 additions
        assert np.abs(a[ok] - b[ok]).max() <= TOL * np.abs(a[ok]).max() + 28 * 2.0 ** -149


def test_other_layers_keep_their_kernels(torch):
    rng = np.random.default_rng(6)
    data, L = _layer(rng, 5, 16, 1, 1)
    assert _choice(L, 1, 20, 20) != "dense_mfma"
    L.close()
    lib = wl.pattern_library(wl.PATTERN_SEED)
    wt = data[0][:, :3].copy()
    wt[3, 1, 1, 1] = np.inf
    L = B.Layer(wt, data[1][:, :3], data[2][:, :3], lib, dense=True)
    assert _choice(L, 1, 20, 20) != "dense_mfma"
    with pytest.raises(B.PatdnnError):
        L.set_config(_variant("dense_mfma"))
    L.close()


@pytest.mark.parametrize("c_in,c_out,n,h,w,stride", [(3, 64, 3, 57, 41, 1), (4, 40, 2, 64, 64, 2), (1, 3, 9, 5, 7, 1)])
def test_pooled_output_is_the_pooling_of_the_plain_one(torch, c_in, c_out, n, h, w, stride):
    """Bit for bit, and windows with NaN and infinities as the maximum after a ReLU has them."""
    rng = np.random.default_rng(w)
    _, L = _layer(rng, c_in, c_out, stride, 1)
    x = rng.standard_normal((n, c_in, h, w)).astype(np.float32)
    kind = rng.random(x.shape)
    x[kind < 0.01] = np.nan
    x[kind < 0.005] = np.inf
    xt, bias = torch.from_numpy(x).cuda(), torch.from_numpy(rng.standard_normal(c_out).astype(np.float32)).cuda()
    plain, pooled = L.conv2d_ws(xt, bias, relu=True), L.conv2d_ws(xt, bias, relu=True, pool=True)
    L.close()
    assert not bool(torch.isnan(plain).any())         # a ReLU makes a zero of a NaN
    assert bool((pooled == torch.nn.functional.max_pool2d(plain, 2)).all())


@pytest.mark.parametrize("c_in,c_out,n,side", [(3, 64, 8, 224), (4, 88, 32, 100)])
def test_pooled_is_no_slower_than_the_tiled_kernel(torch, c_in, c_out, n, side):
    rng = np.random.default_rng(9)
    _, L = _layer(rng, c_in, c_out, 1, 1)
    x = torch.randn((n, c_in, side, side), device="cuda", generator=torch.Generator("cuda").manual_seed(1))
    out = torch.empty((n, c_out, side // 2, side // 2), device="cuda")
    us = {}
    for _ in range(5):
        for name in ("dense_mfma", "d_g16_p7x1_s1_x16"):
            L.set_config(_variant(name))
            L.conv2d_ws(x, None, out, relu=True, pool=True)
            e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            e0.record()
            for _ in range(10):
                L.conv2d_ws(x, None, out, relu=True, pool=True)
            e1.record()
            torch.cuda.synchronize()
            us.setdefault(name, []).append(e0.elapsed_time(e1) * 100)
    L.close()
    print(us, flush=True)
    assert min(us["dense_mfma"]) <= 1.1 * min(us["d_g16_p7x1_s1_x16"])


def test_choice_is_no_less_exact(torch):
    rng = np.random.default_rng(7)
    data, L = _layer(rng, 3, 64, 1, 1)
    x = torch.randn((2, 3, 224, 224), device="cuda", generator=torch.Generator("cuda").manual_seed(1))
    ref = torch.nn.functional.conv2d(x.cpu().double(), torch.from_numpy(data[0]).double(), padding=1)
    err = {}
    for name in ("fkw", "d_g16_p7x1_s1_x16", "dense_mfma"):
        L.set_config(_variant(name))
        err[name] = float((L.conv2d(x, None, relu=False).cpu().double() - ref).norm() / ref.norm())
    print(err, flush=True)
    # 2 % for the draw of the numbers
    assert err["dense_mfma"] <= 1.02 * err["d_g16_p7x1_s1_x16"], err
    L.close()


def test_outputs_beyond_the_caches(torch):
    """Large outputs take another kind of store; the values are those of smaller calls."""
    rng = np.random.default_rng(8)
    _, L = _layer(rng, 3, 64, 1, 1)
    x = torch.randn((24, 3, 224, 224), device="cuda", generator=torch.Generator("cuda").manual_seed(2))
    whole = L.conv2d(x, None, relu=True)
    for i in range(0, 24, 8):
        assert torch.equal(whole[i:i + 8], L.conv2d(x[i:i + 8].contiguous(), None, relu=True))
    L.close()
