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


# Layers that the split kernel can run: c_in, c_out, n, h, w, stride, pad, kept kernels; us of the walk, the tiled kernel
# (at stride 2 the one that the library would take), the tap-product kernel (0: none) and the split kernel.
MEASURED_SPLIT = [
    ((128, 128, 64, 56, 56, 2, 1, 4560), (900, 104, 0, 86)),
    ((256, 256, 64, 28, 28, 2, 1, 18204), (662, 196, 0, 81)),
    ((512, 512, 64, 14, 14, 2, 1, 72817), (1216, 403, 0, 77)),
    ((128, 256, 16, 56, 56, 2, 1, 9102), (460, 89, 0, 48)),
    ((256, 256, 1, 28, 28, 2, 1, 18204), (34, 161, 0, 39)),
    ((64, 64, 8, 56, 56, 2, 1, 2048), (68, 63, 0, 18)),
    ((96, 96, 32, 112, 112, 2, 1, 4608), (1192, 212, 0, 120)),
    ((200, 400, 20, 30, 30, 2, 0, 40000), (471, 226, 0, 41)),
    ((64, 32, 40, 100, 120, 2, 1, 2048), (642, 235, 0, 95)),
    ((300, 40, 2, 33, 41, 2, 1, 6000), (65, 227, 0, 51)),
    ((40, 24, 30, 60, 60, 2, 1, 960), (91, 50, 0, 30)),
    ((120, 500, 1, 20, 20, 2, 1, 30000), (28, 114, 0, 32)),
    ((64, 64, 32, 112, 112, 1, 1, 4096), (2154, 200, 213, 124)),
    ((328, 125, 47, 72, 72, 1, 1, 20500), (7275, 725, 951, 519)),
    ((120, 300, 10, 70, 55, 1, 1, 18000), (764, 123, 138, 112)),
    ((150, 150, 8, 150, 150, 1, 1, 13500), (3001, 328, 400, 352)),
    ((32, 64, 30, 112, 112, 1, 0, 2048), (942, 111, 124, 77)),
    ((40, 400, 10, 100, 100, 1, 1, 16000), (1758, 207, 282, 196)),
]


@pytest.mark.parametrize("case", MEASURED_SPLIT)
def test_split_choice_is_no_slower_than_what_it_stands_in_for(case):
    (c_in, c_out, n, h, w, stride, pad, kept), (walk, tiled, taps, split) = case
    rng = np.random.default_rng(kept)
    mask = np.zeros(c_out * c_in, np.uint8)
    mask[rng.permutation(mask.size)[:kept]] = 1
    L = B.Layer(rng.standard_normal((c_out, c_in, 3, 3), dtype=np.float32), rng.integers(0, 8, (c_out, c_in), dtype=np.uint8),
                mask.reshape(c_out, c_in), wl.pattern_library(wl.PATTERN_SEED), stride=stride, pad=pad, host_only=True)
    L.set_config({B.patdnn_variant_name(v): v for v in range(B.patdnn_num_variants())}["split_f16"])       # can run it
    L.set_config(-1)
    choice = B.lib().patdnn_internal_choice
    choice.argtypes = [ctypes.c_void_p] + [ctypes.c_int32] * 3 + [ctypes.c_size_t, ctypes.c_void_p]
    cfg = B.Config()
    assert choice(L.handle, n, h, w, 0, ctypes.byref(cfg)) == 0
    name = B.patdnn_variant_name(cfg.variant)
    us = split if name == "split_f16" else walk if name == "fkw" else taps if name.startswith("taps") else tiled
    # the estimates are fitted to 10 %, and two runs differ by some per cent
    assert us <= 1.15 * (tiled if stride == 2 else min(walk, tiled, taps)), name
    L.close()


# Dense layers of few channels: c_in, c_out, n, h, w, stride, pad; us of the walk, the tiled kernel (0: none at stride 2)
# and the dense kernel.
MEASURED_DENSE = [
    ((3, 64, 64, 224, 224, 1, 1), (1699, 255, 180)),
    ((3, 64, 1, 224, 224, 1, 1), (34, 17, 12)),
    ((1, 1, 64, 224, 224, 1, 1), (27, 37, 41)),
    ((3, 2, 64, 224, 224, 1, 1), (71, 73, 78)),
    ((3, 4, 64, 224, 224, 1, 1), (130, 75, 82)),
    ((3, 8, 64, 224, 224, 1, 1), (236, 79, 82)),
    ((1, 16, 64, 224, 224, 1, 1), (325, 53, 51)),
    ((4, 16, 7, 97, 131, 1, 0), (20, 18, 11)),
    ((4, 88, 32, 100, 100, 1, 1), (287, 70, 47)),
    ((3, 1, 64, 224, 224, 2, 1), (18, 0, 24)),
    ((1, 2, 64, 224, 224, 2, 1), (17, 0, 14)),
    ((3, 32, 64, 112, 112, 2, 1), (114, 0, 15)),
    ((4, 130, 2, 40, 23, 1, 0), (11, 17, 11)),
    ((1, 1, 16, 112, 112, 1, 1), (11, 11, 11)),
    ((2, 512, 8, 56, 56, 1, 1), (106, 21, 17)),
]


@pytest.mark.parametrize("case", MEASURED_DENSE)
def test_dense_choice_is_no_slower_than_what_it_stands_in_for(case):
    (c_in, c_out, n, h, w, stride, pad), (walk, tiled, dense) = case
    L = B.Layer(np.ones((c_out, c_in, 3, 3), np.float32), np.zeros((c_out, c_in), np.uint8), np.ones((c_out, c_in), np.uint8),
                wl.pattern_library(wl.PATTERN_SEED), stride=stride, pad=pad, dense=True, host_only=True)
    choice = B.lib().patdnn_internal_choice
    choice.argtypes = [ctypes.c_void_p] + [ctypes.c_int32] * 3 + [ctypes.c_size_t, ctypes.c_void_p]
    cfg = B.Config()
    assert choice(L.handle, n, h, w, 0, ctypes.byref(cfg)) == 0
    name = B.patdnn_variant_name(cfg.variant)
    us = dense if name == "dense_mfma" else walk if name == "fkw" else tiled
    assert us <= 1.05 * (tiled if stride == 1 else walk), name
    L.close()


# c_in, c_out, n, h, w, stride, pad, patterns, kept kernels, dense; us of the walk over the kept weights and
# of the matrix kernel
MEASURED_F16 = [
    ((157, 6, 11, 173, 160, 2, 1, 8, 12, 0), (9, 92)),
    ((101, 6, 61, 98, 98, 2, 0, 12, 6, 0), (10, 96)),
    ((362, 2, 8, 137, 137, 2, 1, 56, 13, 0), (14, 104)),
    ((136, 2, 15, 96, 96, 2, 1, 8, 2, 0), (9, 53)),
    ((161, 4, 4, 209, 224, 1, 0, 8, 6, 0), (9, 46)),
    ((390, 16, 31, 29, 29, 1, 1, 8, 21, 0), (10, 32)),
    ((151, 17, 19, 68, 68, 1, 1, 8, 6, 0), (11, 34)),
    ((308, 1, 10, 59, 59, 2, 1, 8, 3, 0), (9, 30)),
    ((507, 23, 27, 26, 26, 1, 1, 8, 37, 0), (9, 29)),
    ((448, 11, 36, 26, 24, 1, 1, 8, 15, 0), (9, 28)),
    ((64, 70, 18, 91, 94, 1, 1, 6, 4480, 1), (2121, 55)),
    ((64, 324, 36, 26, 28, 1, 1, 12, 20736, 1), (1450, 30)),
    ((52, 19, 1, 3, 3, 1, 0, 8, 279, 0), (12, 9)),
    ((18, 108, 21, 3, 3, 1, 0, 6, 558, 0), (13, 9)),
    ((59, 23, 1, 5, 5, 1, 1, 8, 427, 0), (14, 10)),
    ((16, 20, 1, 4, 6, 1, 1, 12, 320, 1), (15, 9)),
    ((1, 5, 61, 176, 176, 1, 1, 12, 5, 1), (72, 62)),
    ((128, 128, 64, 56, 56, 1, 1, 8, 4551, 0), (1990, 100)),
    ((256, 256, 1, 28, 28, 1, 1, 8, 18204, 0), (57, 9)),
]


@pytest.mark.parametrize("case", MEASURED_F16)
def test_binary16_choice_is_close_to_the_fastest(case):
    (c_in, c_out, n, h, w, stride, pad, patterns, kept, dense), (walk, matrix) = case
    rng = np.random.default_rng(kept)
    mask = np.zeros(c_out * c_in, np.uint8)
    mask[rng.permutation(mask.size)[:kept]] = 1
    lib = wl.pattern_library(wl.PATTERN_SEED, patterns) if patterns < 56 else wl.pattern_universe()
    L = B.Layer(np.ones((c_out, c_in, 3, 3), np.float32), rng.integers(0, patterns, (c_out, c_in), dtype=np.uint8),
                mask.reshape(c_out, c_in), lib, stride=stride, pad=pad, dense=bool(dense), host_only=True)
    choice = B.lib().patdnn_internal_f16_choice
    choice.argtypes = [ctypes.c_void_p] * 2 + [ctypes.c_int32] * 3
    choice.restype = ctypes.c_int32
    got = choice(L.handle, 4096, n, h, w)
    L.close()
    assert got >= -1
    assert (walk if got < 0 else matrix) <= 1.4 * min(walk, matrix), got


# c_in, c_out, n, h, w, stride; us of the first three launch shapes of the binary16 matrix kernel (none where the library has
# no use for one: the second at stride 1, the first for few filters) and of the first that splits the channels
NONE = float("inf")
MEASURED_F16_SHAPES = [
    ((128, 128, 64, 56, 56, 1), (68, NONE, 89, 146)),
    ((256, 256, 64, 28, 28, 1), (61, NONE, 90, 132)),
    ((40, 88, 50, 54, 55, 1), (31.1, NONE, 30.5, 52)),
    ((40, 192, 16, 82, 82, 1), (37.1, NONE, 37.7, 71)),
    ((208, 272, 24, 32, 32, 1), (50, NONE, 42.5, 74)),
    ((126, 248, 15, 127, 127, 1), (135, NONE, 208, 334)),
    ((328, 256, 5, 32, 47, 1), (51, NONE, 30, 38)),
    ((89, 62, 2, 120, 120, 1), (NONE, NONE, 12, 16)),
    ((32, 264, 4, 40, 40, 1), (12, NONE, 7.3, 10)),
    ((447, 424, 9, 106, 95, 2), (237, 141, 484, 724)),
    ((39, 421, 24, 79, 121, 2), (75, 61, 150, 290)),
    ((32, 108, 17, 58, 58, 2), (12.9, 9.4, 8.5, 18.8)),
    # filters that fill sets of 128 badly
    ((48, 200, 4, 224, 208, 1), (56, NONE, 78, NONE)),
    ((159, 272, 60, 66, 66, 1), (248, NONE, 409, 784)),
    ((96, 295, 11, 172, 170, 1), (201, NONE, 302, 591)),
    ((126, 88, 20, 195, 195, 1), (224, NONE, 295, 483)),
    ((44, 280, 16, 80, 79, 1), (54, NONE, 66, NONE)),
    ((48, 133, 16, 65, 64, 1), (31, NONE, 24, NONE)),
]


@pytest.mark.parametrize("case", MEASURED_F16_SHAPES)
def test_binary16_launch_shape_is_close_to_the_fastest(case):
    (c_in, c_out, n, h, w, stride), us = case
    L = B.Layer(np.ones((c_out, c_in, 3, 3), np.float32), np.zeros((c_out, c_in), np.uint8), np.ones((c_out, c_in), np.uint8),
                wl.pattern_library(wl.PATTERN_SEED), stride=stride, host_only=True)
    choice = B.lib().patdnn_internal_f16_choice
    choice.argtypes = [ctypes.c_void_p] * 2 + [ctypes.c_int32] * 3
    choice.restype = ctypes.c_int32
    shape = choice(L.handle, 4096, n, h, w) >> 1
    L.close()
    assert 0 <= shape < 4 and us[shape] <= 1.05 * min(us), shape


# c_in, c_out, n, h, w, pad, patterns, kept kernels; us of the walk and of the tap-product kernel: layers that take little
# more than a launch, where a group on several wavefronts is faster than the walk.  One tile of at most 64 groups keeps the walk.
SMALL = [
    ((40, 155, 21, 10, 10, 1, 8, 1722), (22.9, 9.1)),
    ((24, 240, 2, 18, 18, 1, 12, 2880), (13.6, 8.3)),
    ((36, 16, 8, 39, 39, 1, 12, 160), (12.6, 7.8)),
    ((114, 24, 1, 19, 19, 1, 6, 760), (15.9, 11.3)),
    ((64, 512, 1, 14, 14, 1, 8, 9102), (13.3, 10.8)),
]


@pytest.mark.parametrize("case", SMALL)
def test_walk_of_small_layers_only_where_one_tile_has_few_groups(case):
    (c_in, c_out, n, h, w, pad, patterns, kept), _ = case
    rng = np.random.default_rng(3)
    mask = np.zeros(c_in * c_out, np.uint8)
    mask[rng.permutation(mask.size)[:kept]] = 1
    layer = B.Layer(rng.standard_normal((c_out, c_in, 3, 3), dtype=np.float32),
                    rng.integers(0, patterns, (c_out, c_in), dtype=np.uint8), mask.reshape(c_out, c_in),
                    wl.pattern_library(wl.PATTERN_SEED, patterns), pad=pad, host_only=True)
    choice = B.lib().patdnn_internal_choice
    choice.argtypes = [ctypes.c_void_p] + [ctypes.c_int32] * 3 + [ctypes.c_size_t, ctypes.c_void_p]
    for room in (1 << 27, 0):
        chosen = B.Config()
        choice(layer.handle, n, h, w, room, ctypes.byref(chosen))
        one_tile = n == 1 and (h, w) == (14, 14)
        assert B.patdnn_variant_name(chosen.variant) == ("fkw" if one_tile else "taps_f8")


# layers of few groups with room for partial sums; us in channel slices and with groups on several wavefronts
FEW_GROUPS = [
    ((34, 276, 1, 24, 15, 1, 8, 4692), (15.4, 9.8)),
    ((32, 24, 8, 20, 20, 1, 8, 768), (12.4, 8.4)),
    ((48, 80, 1, 23, 28, 1, 8, 1067), (12.1, 9.4)),
]


@pytest.mark.parametrize("case", FEW_GROUPS)
def test_few_groups_are_not_cut_into_slices_where_wavefronts_share_them(case):
    (c_in, c_out, n, h, w, pad, patterns, kept), _ = case
    rng = np.random.default_rng(4)
    mask = np.zeros(c_in * c_out, np.uint8)
    mask[rng.permutation(mask.size)[:kept]] = 1
    layer = B.Layer(rng.standard_normal((c_out, c_in, 3, 3), dtype=np.float32),
                    rng.integers(0, patterns, (c_out, c_in), dtype=np.uint8), mask.reshape(c_out, c_in),
                    wl.pattern_library(wl.PATTERN_SEED, patterns), pad=pad, host_only=True)
    choice = B.lib().patdnn_internal_choice
    choice.argtypes = [ctypes.c_void_p] + [ctypes.c_int32] * 3 + [ctypes.c_size_t, ctypes.c_void_p]
    chosen = B.Config()
    choice(layer.handle, n, h, w, 1 << 27, ctypes.byref(chosen))
    assert B.patdnn_variant_name(chosen.variant) == "taps_f8" and chosen.ksplit == 1


# Layers that stay with the tap-product kernel, the most exact one: c_in, c_out, n, h, w, pad, patterns, kept kernels; us of
# that kernel and of the one that an estimate of its launches put ahead, the tiled or (all kept) the split kernel.  The
# last one is its own only with room for slices.
MOST_EXACT = [
    ((136, 48, 9, 141, 141, 1, 8, 979), (69.6, 85.9)),
    ((384, 56, 5, 170, 170, 1, 8, 3226), (180, 198)),
    ((288, 51, 9, 134, 134, 1, 6, 4080), (188, 200)),
    ((140, 40, 22, 85, 100, 0, 8, 1556), (88, 100)),
    ((312, 24, 6, 219, 219, 1, 6, 2080), (203, 228)),
    ((80, 292, 37, 52, 52, 1, 8, 23360), (375, 228)),
    ((72, 232, 1, 190, 206, 1, 24, 16704), (150, 75)),
    ((504, 128, 5, 144, 128, 1, 8, 9677), (313, 275)),
]


@pytest.mark.parametrize("case", MOST_EXACT)
def test_layers_of_the_most_exact_kernel_stay_with_it(case):
    (c_in, c_out, n, h, w, pad, patterns, kept), _ = case
    rng = np.random.default_rng(5)
    mask = np.zeros(c_in * c_out, np.uint8)
    mask[rng.permutation(mask.size)[:kept]] = 1
    lib = wl.pattern_library(wl.PATTERN_SEED, patterns) if patterns < 56 else wl.pattern_universe()
    layer = B.Layer(rng.standard_normal((c_out, c_in, 3, 3), dtype=np.float32), rng.integers(0, patterns, (c_out, c_in), dtype=np.uint8),
                    mask.reshape(c_out, c_in), lib, pad=pad, host_only=True)
    choice = B.lib().patdnn_internal_choice
    choice.argtypes = [ctypes.c_void_p] + [ctypes.c_int32] * 3 + [ctypes.c_size_t, ctypes.c_void_p]
    chosen = B.Config()
    for room in (1 << 27,) if case is MOST_EXACT[-1] else (1 << 27, 0):
        choice(layer.handle, n, h, w, room, ctypes.byref(chosen))
        assert B.patdnn_variant_name(chosen.variant).startswith("taps")
    layer.close()


# layers for which a workspace made the library choose the walk, or slices that take longer: c_in, c_out, n, h, w, pad, patterns,
# kept kernels; us of the choice with one and without
SLOWER_WITH_ROOM = [
    ((68, 360, 1, 31, 5, 1, 8, 6800), (12.5, 8.9)),
    ((70, 295, 1, 17, 17, 1, 8, 5736), (11.3, 9.2)),
    ((39, 164, 1, 43, 43, 1, 12, 6396), (13.9, 10.5)),
    ((31, 16, 4, 60, 60, 1, 24, 248), (12.6, 8.9)),
    ((88, 24, 5, 35, 51, 1, 8, 1056), (14.3, 10.9)),
    ((81, 16, 10, 44, 44, 0, 8, 360), (13.1, 9.7)),
]


@pytest.mark.parametrize("case", SLOWER_WITH_ROOM)
def test_room_does_not_make_a_choice_slower(case):
    (c_in, c_out, n, h, w, pad, patterns, kept), _ = case
    rng = np.random.default_rng(6)
    mask = np.zeros(c_in * c_out, np.uint8)
    mask[rng.permutation(mask.size)[:kept]] = 1
    layer = B.Layer(rng.standard_normal((c_out, c_in, 3, 3), dtype=np.float32), rng.integers(0, patterns, (c_out, c_in), dtype=np.uint8),
                    mask.reshape(c_out, c_in), wl.pattern_library(wl.PATTERN_SEED, patterns), pad=pad, host_only=True)
    assert _choices(layer, n, h, w)[0] == _choices(layer, n, h, w)[1]
    layer.close()


def _choices(layer, n, h, w):
    choice = B.lib().patdnn_internal_choice
    choice.argtypes = [ctypes.c_void_p] + [ctypes.c_int32] * 3 + [ctypes.c_size_t, ctypes.c_void_p]
    chosen = []
    for room in (1 << 27, 0):
        c = B.Config()
        choice(layer.handle, n, h, w, room, ctypes.byref(c))
        chosen.append((B.patdnn_variant_name(c.variant), c.ck, c.waves, c.ksplit))
    return chosen


@pytest.mark.parametrize("seed", range(4))
def test_a_choice_that_needs_no_room_is_the_one_without(seed):
    """... and with the room that a choice asks for, no more, it is that choice."""
    rng = np.random.default_rng(seed)
    for _ in range(60):
        c_in, c_out, n = (int(v) for v in np.exp(rng.uniform(np.log([16, 16, 1]), np.log([300, 300, 64]))))
        h, w = (int(v) for v in np.exp(rng.uniform(np.log(7), np.log(60), 2)))
        mask = (rng.random((c_out, c_in)) < rng.choice([0.15, 1 / 3.6, 0.5, 1.0])).astype(np.uint8)
        layer = B.Layer(np.ones((c_out, c_in, 3, 3), np.float32), rng.integers(0, 8, (c_out, c_in), dtype=np.uint8), mask,
                        wl.pattern_library(wl.PATTERN_SEED), host_only=True)
        with_room, without = _choices(layer, n, h, w)
        if with_room[3] == 1:
            assert with_room == without, (c_in, c_out, n, h, w)
        else:
            stride = -(-n * c_out * h * w // 64) * 64
            c = B.Config()
            B.lib().patdnn_internal_choice(layer.handle, n, h, w, with_room[3] * stride, ctypes.byref(c))
            assert (B.patdnn_variant_name(c.variant), c.ck, c.waves, c.ksplit) == with_room, (c_in, c_out, n, h, w)
        layer.close()


# Launches of the tap-product kernel, us by (ck, waves) without slices: how many workgroups share a CU decides, four wavefronts a SIMD
# and four chunks of 32 channels in LDS.
MEASURED_LAUNCHES = [
    ((384, 270, 5, 33, 33, 1, 12, 28800), {(128, 8): 86.6, (128, 2): 100.4, (128, 7): 71.4}),
    ((110, 288, 2, 86, 86, 1, 8, 8800), {(55, 8): 44.1, (110, 6): 59.6, (110, 8): 45.0}),
    ((56, 392, 51, 10, 9, 1, 56, 3293), {(56, 8): 22.4, (28, 2): 24.9, (56, 10): 18.9}),
    ((104, 29, 4, 172, 167, 1, 12, 452), {(52, 4): 30.1, (26, 2): 39.1}),
    ((40, 36, 6, 117, 117, 0, 56, 720), {(40, 4): 34.9, (10, 1): 41.5, (20, 1): 32.1, (40, 3): 30.3}),
    ((53, 40, 6, 88, 137, 1, 6, 589), {(53, 8): 22.7, (27, 2): 26.8, (53, 5): 21.9}),
    ((251, 312, 10, 31, 31, 1, 12, 21753), {(63, 8): 100.9, (126, 4): 115.5, (126, 8): 96.4}),
    ((75, 288, 43, 16, 10, 1, 56, 10800), {(75, 8): 53.9, (75, 2): 62.2}),
    ((32, 127, 24, 29, 39, 1, 24, 610), {(32, 4): 15.5, (32, 2): 17.6}),
    ((24, 93, 1, 221, 224, 1, 56, 620), {(24, 4): 18.4, (24, 2): 21.3, (24, 3): 18.7}),
    ((128, 256, 1, 56, 56, 1, 8, 9102), {(128, 2): 13.5, (128, 3): 14.7, (64, 2): 15.6}),
    ((256, 256, 1, 56, 56, 1, 8, 18204), {(128, 2): 22.6, (128, 3): 25.0, (64, 2): 26.1}),
    ((512, 512, 1, 28, 28, 1, 8, 72818), {(128, 1): 36.2, (128, 2): 39.8, (64, 1): 44.5}),
]


@pytest.mark.parametrize("case", MEASURED_LAUNCHES)
def test_launch_of_the_tap_product_kernel_is_close_to_the_fastest(case):
    (c_in, c_out, n, h, w, pad, patterns, kept), us = case
    rng = np.random.default_rng(7)
    mask = np.zeros(c_in * c_out, np.uint8)
    mask[rng.permutation(mask.size)[:kept]] = 1
    lib = wl.pattern_library(wl.PATTERN_SEED, patterns) if patterns < 56 else wl.pattern_universe()
    layer = B.Layer(rng.standard_normal((c_out, c_in, 3, 3), dtype=np.float32), rng.integers(0, patterns, (c_out, c_in), dtype=np.uint8),
                    mask.reshape(c_out, c_in), lib, pad=pad, host_only=True)
    name, ck, waves, ksplit = _choices(layer, n, h, w)[1]
    layer.close()
    assert name.startswith("taps") and ksplit == 1
    assert us[ck, waves] <= 1.08 * min(us.values()), (ck, waves)


def test_a_layer_of_the_split_kernel_is_not_left_for_a_slower_launch():
    """176 -> 90 at 97 x 97, 15 images, all kept: 190 us, the tap-product kernel 302, which is estimated ahead of the tiled one, 326."""
    c_in, c_out = 176, 90
    rng = np.random.default_rng(8)
    layer = B.Layer(rng.standard_normal((c_out, c_in, 3, 3), dtype=np.float32), rng.integers(0, 8, (c_out, c_in), dtype=np.uint8),
                    np.ones((c_out, c_in), np.uint8), wl.pattern_library(wl.PATTERN_SEED), host_only=True)
    assert [c[0] for c in _choices(layer, 15, 97, 97)] == ["split_f16"] * 2
    layer.close()
