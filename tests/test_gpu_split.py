"""GPU parity of fp32 layers on the binary16 matrix cores (csrc/kernel_split.hip) where it can go wrong: odd and
even rows, strips, tiles over several images, remainders of channels and filters, every launch shape (asserted),
workgroups with several units of work, both strides, pooled windows, inputs of all magnitudes, sums that are not
finite - and where the library chooses it."""

import ctypes

import numpy as np
import pytest

from paper_2001_00138_amd import binding as B
from paper_2001_00138_amd import workloads as wl

pytestmark = pytest.mark.gpu
# 22 bits of each factor and fp32 sums: an error of about 2^-23 of each product, and sqrt(K) 2^-24 of the sum of
# the terms' magnitudes; 1e-5 of the largest output is far above both
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


def _layer(rng, c_in, c_out, keep, stride=1, pad=1, scale=1.0):
    lib = wl.pattern_library(wl.PATTERN_SEED)
    ids = rng.integers(0, 8, (c_out, c_in), dtype=np.uint8)
    mask = (rng.random((c_out, c_in)) < keep).astype(np.uint8)
    wt = (rng.standard_normal((c_out, c_in, 3, 3)) * scale).astype(np.float32)
    return (wt, ids, mask, lib), B.Layer(wt, ids, mask, lib, stride=stride, pad=pad)


# c_in, c_out, n, h, w, stride, pad, keep, floats in front of the tensor
CASES = [
    (128, 64, 2, 14, 14, 1, 1, 0.9, 0),         # one block of 64 filters
    (31, 65, 3, 17, 33, 1, 1, 1.0, 0),          # one more filter than a block, one channel short of a step, two strips
    (33, 130, 2, 12, 34, 1, 0, 1.0, 0),         # two steps; pairs of pixels; a strip that is not full
    (33, 130, 2, 12, 34, 1, 0, 1.0, 1),         # the same rows off their pairs
    (160, 40, 5, 7, 7, 2, 1, 0.5, 0),           # tiles over several images
    (128, 200, 1, 57, 41, 2, 1, 0.3, 0),
    (96, 70, 2, 64, 64, 2, 0, 0.8, 0),
    (64, 24, 2, 39, 13, 2, 1, 1.0, 0),          # narrow rows: the smallest tiles, for one block of filters
    (40, 12, 9, 3, 3, 1, 1, 1.0, 0),
    (48, 100, 7, 3, 3, 2, 0, 1.0, 0),           # one output pixel an image
]


@pytest.mark.parametrize("case", CASES)
def test_split_kernel(torch, oracle, case):
    from oracle import stack as ostack
    c_in, c_out, n, h, w, stride, pad, keep, shift = case
    rng = np.random.default_rng(c_in * 1000 + w)
    data, L = _layer(rng, c_in, c_out, keep, stride, pad)
    bias = rng.standard_normal(c_out).astype(np.float32)
    x = rng.standard_normal((n, c_in, h, w)).astype(np.float32)
    full = oracle.conv2d(*data, x, bias, stride=stride, pad=pad, relu=True, skip_removed=True)
    L.set_config(_variant("split_f16"))
    xt = torch.empty(x.size + shift, device="cuda")[shift:].view(x.shape)
    xt.copy_(torch.from_numpy(x))
    bt, guard = torch.from_numpy(bias).cuda(), 1024
    for pool in (False, True):
        ref = ostack.maxpool2x2(full) if pool else full
        if 0 in ref.shape:
            continue
        print(f"  {case} pool={pool}", flush=True)
        numel = int(np.prod(ref.shape))
        buf = torch.full((numel + 2 * guard,), 777.0, device="cuda")
        out = buf[guard:guard + numel].view(ref.shape)
        L.conv2d_ws(xt, bt, out, relu=True, pool=pool)
        assert bool((buf[:guard] == 777.0).all()) and bool((buf[guard + numel:] == 777.0).all())
        assert float(np.abs(out.cpu().numpy().astype(np.float64) - ref).max() / np.abs(ref).max()) <= TOL
    L.close()


# c_in, c_out, n, h, w, stride, twice the number of the launch shape (plus one: pairs of pixels) and units of work, plain
# and pooled.  256 workgroups: some take a second or a third unit.
PERSISTENT = [
    (32, 64, 22, 56, 56, 1, (1, 270), (1, 270)),       # one channel step: a unit an iteration
    (32, 40, 23, 56, 57, 1, (0, 292), (0, 282)),
    (70, 130, 7, 50, 50, 1, (3, 288), (3, 288)),       # three steps, two filter sets
    (70, 130, 7, 50, 51, 1, (2, 288), (2, 288)),
    (33, 64, 2100, 5, 4, 1, (5, 329), (5, 263)),           # two steps, tiles over several images
    (40, 64, 5200, 3, 3, 1, (4, 366), (6, 325)),
    (33, 100, 90, 28, 28, 2, (7, 276), (6, 276)),
    (96, 130, 45, 37, 35, 2, (6, 482), (6, 508)),
    (128, 70, 60, 37, 38, 2, (7, 357), (6, 338)),      # four steps
]


def _plan(L, x, n, h, w, pool):
    plan, units = B.lib().patdnn_internal_split_choice, ctypes.c_int32()
    plan.argtypes = [ctypes.c_void_p] * 2 + [ctypes.c_int32] * 4 + [ctypes.c_void_p]
    plan.restype = ctypes.c_int32
    return plan(L.handle, x, n, h, w, int(pool), ctypes.byref(units)), units.value


@pytest.mark.parametrize("case", PERSISTENT)
def test_workgroups_that_go_on(torch, case):
    """Units after the first: scales, marks and sums start anew, whatever magnitudes the one before had and while the
    next one's inputs come in; values that are not finite in some of them only."""
    c_in, c_out, n, h, w, stride, *launches = case
    rng = np.random.default_rng(c_in * 1000 + w)
    _, L = _layer(rng, c_in, c_out, 0.9, stride)
    magnitude = np.array([1.0, 1e4, 1e-6, 1e12, 1e-14], np.float32)[np.arange(n) % 5][:, None, None, None]
    x = rng.standard_normal((n, c_in, h, w)).astype(np.float32) * magnitude
    for k, value in enumerate((np.nan, np.inf, -np.inf)):
        x[k + 1::37, 3, k % h, 1] = value
    xt, bias = torch.from_numpy(x).cuda(), torch.from_numpy(rng.standard_normal(c_out).astype(np.float32) * 1e-15).cuda()
    for pool, launch in zip((False, True), launches):
        assert _plan(L, xt.data_ptr(), n, h, w, pool) == launch
        assert launch[1] > 256 and launch[1] % 256
        print(f"  {case} pool={pool}", flush=True)
        got = {}
        for name in ("fkw", "split_f16"):
            L.set_config(_variant(name))
            got[name] = L.conv2d_ws(xt, bias, None, relu=pool, pool=pool).flatten(1)
        a, b = got["fkw"], got["split_f16"]
        assert torch.equal(torch.isnan(a), torch.isnan(b)) and torch.equal(a[torch.isinf(a)], b[torch.isinf(a)])
        ok = torch.isfinite(a)
        assert torch.equal(ok, torch.isfinite(b))
        zero = torch.zeros_like(a)
        worst = torch.where(ok, (a - b).abs(), zero).amax(1) / torch.where(ok, a.abs(), zero).amax(1).clamp(min=1e-30)
        assert float(worst.max()) <= TOL, int(worst.argmax())
    L.close()


@pytest.mark.parametrize("inputs,weights", [(1e-40, 1.0), (1e-30, 1e-6), (1e30, 1e-20), (1.0, 1e30)])
def test_magnitudes(torch, oracle, inputs, weights):
    """Scales far from one, and inputs whose later channels are 10^4 times the first ones'."""
    rng = np.random.default_rng(8)
    data, L = _layer(rng, 96, 40, 0.6, 2, scale=weights)
    x = (rng.standard_normal((2, 96, 19, 22)) * inputs).astype(np.float32)
    x[:, 32:] *= np.float32(1e4) if inputs < 1e20 else np.float32(1)
    ref = oracle.conv2d(*data, x, None, stride=2, skip_removed=True)
    L.set_config(_variant("split_f16"))
    got = L.conv2d(torch.from_numpy(x).cuda(), None, relu=False).cpu().numpy().astype(np.float64)
    L.close()
    assert 0 < np.abs(ref).max() < 3e38
    # half a subnormal spacing for the result, and as much for each input
    assert np.abs(got - ref).max() <= TOL * np.abs(ref).max() + 2.0 ** -149


def test_small_values_beside_large_ones(torch, oracle):
    """Images share tiles: one of inputs 10^5 times the others' costs these no more than their last bits."""
    rng = np.random.default_rng(9)
    data, L = _layer(rng, 64, 40, 1.0, 2)
    x = rng.standard_normal((6, 64, 6, 6)).astype(np.float32)
    x[2] *= np.float32(1e5)
    ref = oracle.conv2d(*data, x, None, stride=2, skip_removed=True)
    L.set_config(_variant("split_f16"))
    got = L.conv2d(torch.from_numpy(x).cuda(), None, relu=False).cpu().numpy().astype(np.float64)
    L.close()
    for i in range(6):
        assert np.abs(got[i] - ref[i]).max() <= TOL * np.abs(ref[i]).max(), i


def _reference(torch, data, x, stride, pad=1):
    """The layer in 64 bits, and for each output the sum of its terms' magnitudes."""
    wt, ids, mask, lib = data
    bits = (lib.astype(np.int64)[ids][..., None] >> np.arange(9)) & 1
    w = torch.from_numpy((wt.reshape(*ids.shape, 9) * bits * mask[..., None]).reshape(*ids.shape, 3, 3).astype(np.float64))
    xd = torch.from_numpy(x).double()
    conv = torch.nn.functional.conv2d
    return conv(xd, w, None, stride, pad), conv(xd.abs(), w.abs(), None, stride, pad)


# Each factor keeps 22 bits or more and its product 2^-21; the sums' roundings, 2^-24 of a partial sum each, are
# some hundred of random signs: an output is within 1e-6 of the sum of its terms' magnitudes
OF_TERMS = 1e-6


@pytest.mark.parametrize("large", [1e10, 1e20, -3.4028234663852886e38])
@pytest.mark.parametrize("where", ["kept channel", "removed channel", "other image", "later channels"])
@pytest.mark.parametrize("c_in,c_out,side,stride", [(160, 70, 14, 2), (96, 40, 20, 1)])
def test_ordinary_values_beside_a_large_one(torch, c_in, c_out, side, stride, where, large):
    """One large finite value costs the outputs whose kept weights do not meet it nothing: neighbours in its
    image and tile, filters that removed its channel, images beside its own."""
    rng = np.random.default_rng(11)
    (wt, ids, mask, lib), L = _layer(rng, c_in, c_out, 0.9, stride)
    L.close()
    mask[:, 5] = 0
    L = B.Layer(wt, ids, mask, lib, stride=stride)
    x = np.maximum(rng.standard_normal((4, c_in, side, side)), 0).astype(np.float32)
    x[:, 40] = 0
    x[0, 40 if where == "later channels" else 5 if where == "removed channel" else 7, side // 2 - 1, 3] = large
    if where == "later channels":
        x[:, :32] *= np.float32(1e-20)
    ref, terms = _reference(torch, (wt, ids, mask, lib), x, stride)
    keep = slice(1, None) if where == "other image" else slice(None)
    out = {}
    for name in ("fkw", "split_f16"):
        L.set_config(_variant(name))
        out[name] = L.conv2d(torch.from_numpy(x).cuda(), None, relu=False).cpu().double()
    L.close()
    fits = terms < 1e38                              # beyond, the order of the sum decides what overflows
    err = {name: float(((got - ref).abs() / terms.clamp(min=1e-300))[keep][fits[keep]].max()) for name, got in out.items()}
    print(f"  {where} {large}: {err}", flush=True)
    assert err["fkw"] <= OF_TERMS and err["split_f16"] <= OF_TERMS, err


def test_inputs_of_many_magnitudes(torch):
    """Magnitudes over sixty powers of ten, each output by the sum of its own terms."""
    rng = np.random.default_rng(12)
    data, L = _layer(rng, 100, 70, 1.0, 2)
    x = (rng.standard_normal((3, 100, 17, 22)) * 10.0 ** rng.uniform(-30, 30, (3, 100, 17, 22))).astype(np.float32)
    x[rng.random(x.shape) < 0.5] = 0
    x[1, :, :9] = 0
    x[1, rng.integers(0, 100, 40), rng.integers(0, 9, 40), rng.integers(0, 22, 40)] = np.float32(1e-15)
    ref, terms = _reference(torch, data, x, 2)
    L.set_config(_variant("split_f16"))
    got = L.conv2d(torch.from_numpy(x).cuda(), None, relu=False).cpu().double()
    L.close()
    assert float(((got - ref).abs() / terms.clamp(min=1e-300))[terms > 0].max()) <= OF_TERMS


@pytest.mark.parametrize("c_out,h,stride,pool", [(70, 21, 2, False), (33, 20, 1, True), (130, 34, 1, False)])
@pytest.mark.parametrize("share", [1e-4, 1e-2, 1.0])
def test_not_finite_inputs(torch, c_out, h, stride, pool, share):
    """Infinite and NaN inputs reach the outputs that the walk over the kept weights gives them, kept zeros
    among the weights, and the others stay as they are."""
    rng = np.random.default_rng(c_out)
    data, _ = _layer(rng, 48, c_out, 0.6, stride)
    data[0][:, 3] = 0
    L = B.Layer(*data, stride=stride)
    x = rng.standard_normal((3, 48, h, h + 2)).astype(np.float32)
    kind = rng.random(x.shape)
    x[kind < share] = np.nan
    x[kind < 0.6 * share] = -np.inf
    x[kind < 0.4 * share] = np.inf
    got = {}
    for name in ("fkw", "split_f16"):
        L.set_config(_variant(name))
        got[name] = L.conv2d_ws(torch.from_numpy(x).cuda(), None, relu=False, pool=pool).cpu().numpy()
    L.close()
    a, b = got["fkw"], got["split_f16"]
    assert np.array_equal(np.isnan(a), np.isnan(b)) and np.array_equal(a[np.isinf(a)], b[np.isinf(a)])
    ok = np.isfinite(a)
    assert np.array_equal(ok, np.isfinite(b))
    assert not ok.any() or np.abs(a[ok] - b[ok]).max() <= TOL * max(np.abs(a[ok]).max(), 1e-30)


@pytest.mark.parametrize("c_in,c_out,n,h,w", [(128, 64, 2, 54, 57), (64, 128, 8, 8, 55), (64, 64, 8, 37, 197), (128, 128, 2, 56, 56)])
def test_pooled_output_is_the_pooling_of_the_plain_one(torch, c_in, c_out, n, h, w):
    """The library's choice for a plain call and for a pooled one, whose tiles are cut differently."""
    rng = np.random.default_rng(w)
    _, L = _layer(rng, c_in, c_out, 1.0, 2)
    x = torch.randn((n, c_in, h, w), device="cuda", generator=torch.Generator("cuda").manual_seed(1))
    plain = L.conv2d_ws(x, None, relu=True)
    pooled = L.conv2d_ws(x, None, relu=True, pool=True)
    assert bool((pooled == torch.nn.functional.max_pool2d(plain, 2)).all())
    L.close()


@pytest.mark.parametrize("c,side,n,stride", [(64, 112, 32, 1), (128, 56, 8, 2)])
def test_the_tuner_knows_the_kernel(torch, c, side, n, stride):
    """Tuning finds nothing slower than what the library takes by itself (1.2 to 1.7 times as fast as the rest here)."""
    rng = np.random.default_rng(side)
    _, L = _layer(rng, c, c, 1.0, stride)
    x = torch.randn((n, c, side, side), device="cuda", generator=torch.Generator("cuda").manual_seed(1))
    out = torch.empty(L.output_shape(n, side, side), device="cuda")
    L.tune(x, None, out)
    assert B.patdnn_variant_name(L.get_config()["variant"]) == "split_f16"
    L.close()


# c_in, c_out, side, n, stride, keep; what is chosen
CHOICES = [((128, 128, 56, 8, 2, 1 / 3.6), "split_f16"), ((64, 64, 56, 8, 2, 1 / 3.6), "t_g16_p4x1_s2_x16_th"),
           ((64, 64, 56, 2, 2, 0.6), "split_f16"), ((328, 125, 72, 47, 1, 0.5), "split_f16"), ((64, 64, 112, 32, 1, 1.0), "split_f16"),
           ((512, 512, 28, 24, 1, 1.0), "taps_f16")]


@pytest.mark.parametrize("shape,name", CHOICES)
def test_choice_is_no_less_exact(torch, shape, name):
    """The library takes the kernel where its error against 64 bits is no larger than that of the kernels it stands
    in for (2 % for the draw of the numbers), for the layer and for its filters of fewest kernels (5 %: a tenth of
    the outputs), and not where the tap-product kernel is chosen."""
    c_in, c_out, side, n, stride, keep = shape
    rng = np.random.default_rng(side)
    (wt, ids, mask, lib), L = _layer(rng, c_in, c_out, keep, stride)
    cfg = B.Config()
    choice = B.lib().patdnn_internal_choice
    choice.argtypes = [ctypes.c_void_p] + [ctypes.c_int32] * 3 + [ctypes.c_size_t, ctypes.c_void_p]
    assert choice(L.handle, n, side, side, 0, ctypes.byref(cfg)) == 0
    chosen = B.patdnn_variant_name(cfg.variant)
    assert chosen == name
    if name == "taps_f16":
        L.set_config(_variant("split_f16"))          # could run it
    if chosen == "split_f16":
        x = torch.randn((4, c_in, side, side), device="cuda", generator=torch.Generator("cuda").manual_seed(1)).clamp_(min=0)
        bits = (lib.astype(np.int64)[ids][..., None] >> np.arange(9)) & 1
        dense = torch.from_numpy((wt.reshape(c_out, c_in, 9) * bits * mask[..., None]).reshape(c_out, -1).astype(np.float64)).cuda()
        ref = torch.stack([dense @ torch.nn.functional.unfold(x[i:i + 1].double(), 3, padding=1, stride=stride)[0] for i in range(4)])
        ref = ref.reshape(L.output_shape(4, side, side))
        fewest = torch.from_numpy(np.argsort(mask.sum(1), kind="stable")[:c_out // 10]).cuda()
        err = {}
        for v in ("split_f16", "fkw", "t_g16_p4x1_s2_x16_th" if stride == 2 else "t_g8_p7x2_s1_x8_thw1b"):
            L.set_config(_variant(v))
            d = L.conv2d(x, None, relu=False).double() - ref
            err[v] = float(d.norm() / ref.norm()), float(d[:, fewest].norm() / ref[:, fewest].norm())
        print(f"  {shape}: {err}", flush=True)
        mine = err.pop("split_f16")
        for other in err.values():
            assert mine[0] <= 1.02 * other[0] and mine[1] <= 1.05 * other[1], (mine, err)
    L.close()


def test_filters_of_few_kernels_and_small_weights_keep_the_other_kernels(torch):
    """One filter of fewer than 18 kernels, for which the others are more exact, or one weight that binary16 would
    not hold whole beside its filter's largest; filters without kernels do not count."""
    rng = np.random.default_rng(13)
    wt = rng.standard_normal((40, 64, 3, 3)).astype(np.float32)
    ids = rng.integers(0, 8, (40, 64), dtype=np.uint8)
    lib = wl.pattern_library(wl.PATTERN_SEED)
    for few, small, fits in ((64, 1, True), (18, 1, True), (17, 1, False), (1, 1, False), (0, 1, True),
                             (64, 2.0 ** -26, True), (64, 2.0 ** -30, False)):
        mask = np.ones((40, 64), np.uint8)
        mask[7, few:] = 0
        w = wt.copy()
        w[9] = np.where(rng.random(w[9].shape) < 0.5, 1.0, -1.0)
        w[9, 11] *= np.float32(small)
        L = B.Layer(w, ids, mask, lib, stride=2)
        if fits:
            L.set_config(_variant("split_f16"))
        else:
            with pytest.raises(B.PatdnnError):
                L.set_config(_variant("split_f16"))
        L.close()
