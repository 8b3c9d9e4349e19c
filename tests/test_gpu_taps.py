"""GPU parity of the tap-product kernel (csrc/kernel_taps.hip) where it can go wrong: tile edges
(images of 14 to 17 and 29 to 31 rows and columns), several images in one tile, filter counts
around its groups, channel counts around its chunks, empty filters, every pattern, split launches
with and without a workspace, fused pooling - against the oracle, element by element."""

import ctypes

import numpy as np
import pytest

from paper_2001_00138_amd import binding as B
from paper_2001_00138_amd import workloads as wl

pytestmark = pytest.mark.gpu
# fp32 sums in any order against fp64: at most K * 2^-24 of the sum of the terms' magnitudes with
# K <= 4 * 160, and in practice sqrt(K) * 2^-24; 1e-5 of the largest output is far above both
TOL = 1e-5


@pytest.fixture(scope="module")
def torch():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    B.lib()
    return torch


# c_out, c_in, n, h, w, pad, keep, patterns, (filters, ck, waves, ksplit)
CASES = [
    (8, 16, 1, 14, 14, 1, 0.5, 8, (8, 0, 1, 1)),          # one tile, one group
    (9, 7, 2, 15, 16, 1, 0.5, 8, (16, 3, 2, 2)),          # 15: the last size of a single tile; 16: the first of two
    (24, 33, 2, 17, 15, 1, 0.3, 12, (8, 33, 3, 1)),
    (40, 20, 2, 29, 31, 1, 0.3, 8, (16, 8, 16, 3)),       # last tile of 15 outputs, and of 3
    (17, 20, 3, 30, 29, 0, 0.4, 8, (8, 20, 2, 1)),
    (16, 12, 3, 16, 17, 0, 0.4, 6, (8, 5, 4, 2)),         # no padding: 16 columns are one tile of 14 outputs
    (130, 129, 5, 7, 7, 1, 0.25, 8, (16, 65, 8, 2)),      # four images in a tile, the last tile not full
    (12, 10, 70, 3, 3, 1, 1.0, 8, (8, 10, 2, 1)),         # sixteen images in a tile
    (11, 9, 9, 5, 8, 0, 0.6, 8, (8, 4, 1, 2)),
    (8, 160, 1, 20, 15, 1, 0.02, 8, (8, 160, 1, 1)),      # the largest chunk; filters without kernels
    (56, 56, 2, 15, 18, 1, 1.0, 56, (16, 56, 4, 1)),      # every pattern
    (1, 1, 1, 3, 40, 1, 1.0, 8, (8, 1, 1, 1)),
]


@pytest.mark.parametrize("case", CASES)
def test_tap_product_kernel(torch, oracle, case):
    from oracle import stack as ostack
    c_out, c_in, n, h, w, pad, keep, patterns, (filters, ck, waves, ksplit) = case
    rng = np.random.default_rng(c_out * 1000 + h * 40 + w)
    lib = wl.pattern_library(wl.PATTERN_SEED, patterns) if patterns < 56 else wl.pattern_universe()
    ids = rng.integers(0, patterns, (c_out, c_in), dtype=np.uint8)
    mask = (rng.random((c_out, c_in)) < keep).astype(np.uint8)
    wt = rng.standard_normal((c_out, c_in, 3, 3)).astype(np.float32)
    bias = rng.standard_normal(c_out).astype(np.float32)
    x = rng.standard_normal((n, c_in, h, w)).astype(np.float32)
    full = oracle.conv2d(wt, ids, mask, lib, x, bias, pad=pad, relu=True, skip_removed=True)
    names = {B.patdnn_variant_name(v): v for v in range(B.patdnn_num_variants())}
    L = B.Layer(wt, ids, mask, lib, pad=pad)
    L.set_config(names[f"taps_f{filters}"], ck, waves, ksplit)
    xt, bt = torch.from_numpy(x).cuda(), torch.from_numpy(bias).cuda()
    need, guard = L.workspace_floats(n, h, w), 1024
    for pool in (False, True):
        ref = ostack.maxpool2x2(full) if pool else full
        if 0 in ref.shape:
            continue
        # no room: the slices add up in the output, or the library chooses; one buffer: a pooled layer's
        # slices add up there
        for room in {need, 0, full.size if pool and ksplit > 1 else 0}:
            print(f"  {case} pool={pool} workspace={room}", flush=True)
            numel = int(np.prod(ref.shape))
            buf = torch.full((numel + 2 * guard,), 777.0, device="cuda")
            wbuf = torch.full((room + 2 * guard,), float("nan"), device="cuda")
            wbuf[:guard] = wbuf[guard + room:] = 555.0
            out = buf[guard:guard + numel].view(ref.shape)
            L.conv2d_ws(xt, bt, out, workspace=wbuf[guard:guard + room] if room else None, relu=True, pool=pool)
            torch.cuda.synchronize()
            for b, k, v in ((buf, numel, 777.0), (wbuf, room, 555.0)):
                assert bool((b[:guard] == v).all()) and bool((b[guard + k:] == v).all())
            err = float(np.abs(out.cpu().numpy().astype(np.float64) - ref).max() / np.abs(ref).max())
            assert err <= TOL, (pool, room, err)
    L.close()


# n, c_in, c_out, side; the family chosen with a workspace, whether it splits the channels, and without one
CHOICES = [((1, 16, 16, 32), "fkw", False, "fkw"), ((1, 64, 512, 14), "fkw", False, "fkw"), ((64, 96, 200, 7), "taps_f8", True, "taps_f8"),
           ((3, 200, 72, 45), "taps_f8", True, "taps_f8"), ((40, 40, 24, 60), "taps_f8", False, "taps_f8"),
           ((6, 20, 48, 150), "t_g8_p7x2_s1_x8_thw1b", False, "t_g8_p7x2_s1_x8_thw1b"), ((32, 64, 512, 28), "taps_f16", False, "taps_f16")]


@pytest.mark.parametrize("shape,with_room,split,without", CHOICES)
def test_chosen_configuration(torch, oracle, shape, with_room, split, without):
    """The library's own choice over the sizes at which it changes (walk, tiled kernel, split and unsplit
    launches, one and two groups per wavefront), with the workspace it asks for and without."""
    n, c_in, c_out, side = shape
    rng = np.random.default_rng(sum(shape))
    lib = wl.pattern_library(wl.PATTERN_SEED)
    ids = rng.integers(0, 8, (c_out, c_in), dtype=np.uint8)
    mask = (rng.random((c_out, c_in)) < 1 / 3.6).astype(np.uint8)
    wt = rng.standard_normal((c_out, c_in, 3, 3)).astype(np.float32)
    x = rng.standard_normal((n, c_in, side, side)).astype(np.float32)
    k = min(n, 2)
    ref = oracle.conv2d(wt, ids, mask, lib, x[-k:], None, skip_removed=True)
    L = B.Layer(wt, ids, mask, lib)
    need = L.workspace_floats(n, side, side)
    assert (need > 0) == split
    choice = B.lib().patdnn_internal_choice
    choice.argtypes = [ctypes.c_void_p] + [ctypes.c_int32] * 3 + [ctypes.c_size_t, ctypes.c_void_p]
    xt = torch.from_numpy(x).cuda()
    for room in {need, 0}:
        cfg = B.Config()
        assert choice(L.handle, n, side, side, room, ctypes.byref(cfg)) == 0
        assert B.patdnn_variant_name(cfg.variant) == (with_room if room else without)
        assert (cfg.ksplit > 1) == (room > 0)
        ws = torch.full((room,), float("nan"), device="cuda") if room else None
        got = L.conv2d_ws(xt, None, workspace=ws)[-k:].cpu().numpy()
        assert float(np.abs(got.astype(np.float64) - ref).max() / np.abs(ref).max()) <= TOL, room
    assert L.get_config()["variant"] == -1
    L.close()


@pytest.mark.parametrize("filters,ksplit", [(8, 1), (16, 1), (8, 2)])
def test_infinite_input_reaches_kept_kernels_only(torch, filters, ksplit):
    """A filter without a kernel in a chunk of channels keeps its bias and its other chunks' sum where
    that chunk's input is infinite or NaN."""
    rng = np.random.default_rng(5)
    c_out, c_in, h = 16, 16, 12
    lib = wl.pattern_library(wl.PATTERN_SEED, 8)
    ids = rng.integers(0, 8, (c_out, c_in), dtype=np.uint8)
    mask = np.ones((c_out, c_in), np.uint8)
    mask[::2, :8] = 0                          # even filters: nothing in the first chunk
    mask[3] = 0                                # no kernel at all
    wt = rng.standard_normal((c_out, c_in, 3, 3)).astype(np.float32)
    bias = rng.standard_normal(c_out).astype(np.float32)
    x = rng.standard_normal((1, c_in, h, h)).astype(np.float32)
    x[0, 0, 3, 3], x[0, 0, 8, 8] = np.inf, np.nan          # the first channel of the first chunk
    names = {B.patdnn_variant_name(v): v for v in range(B.patdnn_num_variants())}
    got = {}
    for name, cfg in (("fkw", (0, 0, 0, 1)), ("taps", (names[f"taps_f{filters}"], 8, 1, ksplit))):
        L = B.Layer(wt, ids, mask, lib)
        L.set_config(*cfg)
        xt, bt = torch.from_numpy(x).cuda(), torch.from_numpy(bias).cuda()
        got[name] = L.conv2d(xt, bt, relu=False).cpu().numpy()
        L.close()
    assert np.array_equal(np.isfinite(got["taps"]), np.isfinite(got["fkw"]))
    assert np.isfinite(got["taps"][0, ::2]).all() and (got["taps"][0, 3] == bias[3]).all()
    ok = np.isfinite(got["fkw"])
    assert np.abs(got["taps"][ok] - got["fkw"][ok]).max() <= TOL * np.abs(got["fkw"][ok]).max()


@pytest.mark.parametrize("shape", [(70, 3, 3, 1), (9, 5, 8, 0), (5, 7, 7, 1)])
@pytest.mark.parametrize("filters,ksplit", [(8, 1), (16, 2)])
def test_infinite_input_stays_in_its_image(torch, shape, filters, ksplit):
    """Images that share a tile lie next to each other in registers and lanes: an infinite or NaN pixel
    reaches the outputs that the walk over the kept weights gives it, and no other image."""
    n, h, w, pad = shape
    rng = np.random.default_rng(n)
    c_out, c_in = 16, 16
    lib = wl.pattern_library(wl.PATTERN_SEED, 8)
    ids = rng.integers(0, 8, (c_out, c_in), dtype=np.uint8)
    mask = (rng.random((c_out, c_in)) < 0.4).astype(np.uint8)
    wt = rng.standard_normal((c_out, c_in, 3, 3)).astype(np.float32)
    x = rng.standard_normal((n, c_in, h, w)).astype(np.float32)
    for img, v in ((1, np.inf), (n - 2, np.nan)):            # corners, whose taps reach past the image
        for y, z in ((0, 0), (0, w - 1), (h - 1, 0), (h - 1, w - 1)):
            x[img, rng.integers(c_in), y, z] = v
    names = {B.patdnn_variant_name(v): v for v in range(B.patdnn_num_variants())}
    got = {}
    for name, cfg in (("fkw", (0, 0, 0, 1)), ("taps", (names[f"taps_f{filters}"], 8, 1, ksplit))):
        L = B.Layer(wt, ids, mask, lib, pad=pad)
        L.set_config(*cfg)
        got[name] = L.conv2d(torch.from_numpy(x).cuda(), None).cpu().numpy()
        L.close()
    assert not np.isfinite(got["fkw"]).all()
    assert np.array_equal(np.isnan(got["taps"]), np.isnan(got["fkw"]))
    assert np.array_equal(got["taps"][np.isinf(got["fkw"])], got["fkw"][np.isinf(got["fkw"])])
    ok = np.isfinite(got["fkw"])
    assert ok[[i for i in range(n) if i not in (1, n - 2)]].all()
    assert np.abs(got["taps"][ok] - got["fkw"][ok]).max() <= TOL * np.abs(got["fkw"][ok]).max()


@pytest.mark.parametrize("inputs,weights", [(1e-40, 0.3), (1e-20, 1e-20), (1.0, 1e-40)])
def test_subnormal_values(torch, oracle, inputs, weights):
    """The matrix unit keeps subnormal inputs, weights and sums."""
    rng = np.random.default_rng(4)
    c_out, c_in, h = 24, 40, 17
    lib = wl.pattern_library(wl.PATTERN_SEED)
    ids = rng.integers(0, 8, (c_out, c_in), dtype=np.uint8)
    mask = (rng.random((c_out, c_in)) < 0.5).astype(np.uint8)
    wt = (rng.standard_normal((c_out, c_in, 3, 3)) * weights).astype(np.float32)
    x = (rng.standard_normal((1, c_in, h, h)) * inputs).astype(np.float32)
    ref = oracle.conv2d(wt, ids, mask, lib, x, None, skip_removed=True)
    names = {B.patdnn_variant_name(v): v for v in range(B.patdnn_num_variants())}
    for variant in ("taps_f8", "taps_f16"):
        L = B.Layer(wt, ids, mask, lib)
        L.set_config(names[variant])
        got = L.conv2d(torch.from_numpy(x).cuda(), None).cpu().numpy().astype(np.float64)
        L.close()
        # half a subnormal spacing per term
        assert 0 < np.abs(ref).max() < 2.0 ** -125
        assert np.abs(got - ref).max() <= 4 * c_in / 2 * 2.0 ** -149 + TOL * np.abs(ref).max()


# c_out, c_in, images of the launch that fills the chip, (ck, waves, ksplit), wavefronts for a group in the small launch
PARTS = [(9, 20, 2100, (20, 1, 1), 4), (24, 33, 1400, (33, 3, 1), 4), (61, 40, 520, (13, 8, 1), 2), (16, 70, 1100, (18, 2, 2), 4),
         (40, 12, 820, (5, 5, 1), 2), (8, 160, 4100, (160, 1, 1), 4)]


@pytest.mark.parametrize("case", PARTS)
def test_a_group_on_several_wavefronts(torch, case):
    """One image, whose launch gives the eight filters of a group to two or four wavefronts, against the same image in
    a launch with a wavefront for each group: the same bits.  Filters without kernels, last groups that are not full."""
    c_out, c_in, many, (ck, waves, ksplit), parts = case
    rng = np.random.default_rng(c_out)
    lib = wl.pattern_library(wl.PATTERN_SEED, 8)
    mask = (rng.random((c_out, c_in)) < 0.3).astype(np.uint8)
    mask[::5] = 0
    L = B.Layer(rng.standard_normal((c_out, c_in, 3, 3)).astype(np.float32), rng.integers(0, 8, (c_out, c_in), dtype=np.uint8), mask, lib)
    L.set_config({B.patdnn_variant_name(v): v for v in range(B.patdnn_num_variants())}["taps_f8"], ck, waves, ksplit)
    got = B.lib().patdnn_internal_taps_parts
    got.argtypes = [ctypes.c_void_p] + [ctypes.c_int32] * 3
    assert (got(L.handle, 1, 14, 14), got(L.handle, many, 14, 14)) == (parts, 1)
    x = torch.from_numpy(rng.standard_normal((many, c_in, 14, 14), dtype=np.float32)).cuda()
    bias = torch.from_numpy(rng.standard_normal(c_out).astype(np.float32)).cuda()
    outs = []
    for k in (1, many):
        out = torch.full((k, c_out, 14, 14), float("nan"), device="cuda")
        ws = torch.empty(L.workspace_floats(k, 14, 14), device="cuda") if ksplit > 1 else None
        L.conv2d_ws(x[:k], bias, out, workspace=ws, relu=True)
        outs.append(out[0])
    assert not bool(torch.isnan(outs[0]).any()) and torch.equal(outs[0], outs[1])
    L.close()
