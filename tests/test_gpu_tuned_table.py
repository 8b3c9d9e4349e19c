"""The committed launch configurations (tuned_configs.json, which bench.py and the README's way of running
use) against the library's own choice: a tuned layer is not left behind by kernels that came after it
was tuned.  Timed in turns on one stream; the faster runs of each side are compared, with room for noise."""

import os

import numpy as np
import pytest

from paper_2001_00138_amd import binding as B
from paper_2001_00138_amd import workloads as wl

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("c,side,n", [(512, 7, 64), (512, 14, 64), (256, 14, 64), (128, 28, 64), (512, 14, 1), (512, 28, 1)])
def test_tuned_is_no_slower_than_chosen(c, side, n):
    compare(c, c, side, n)


@pytest.mark.parametrize("c,side,n", [(512, 14, 64), (256, 28, 64), (128, 56, 64), (512, 14, 1)])
def test_tuned_stride2_is_no_slower_than_chosen(c, side, n):
    compare(c, c, side, n, stride=2)


@pytest.mark.parametrize("n", [1, 64])
def test_tuned_first_layer_is_no_slower_than_chosen(n):
    compare(3, 64, 224, n, dense=True)


def compare(c, c_out, side, n, stride=1, dense=False):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    table = os.path.join(os.path.dirname(B.LIB_PATH), "tuned_configs.json")
    saved = wl.load_tuned_configs(table)[f"{'dense' if dense else 'sparse'}:{c}->{c_out}@{side}x{side}:s{stride}p1:n{n}"]
    names = {B.patdnn_variant_name(v): v for v in range(B.patdnn_num_variants())}
    rng = np.random.default_rng(c + side)
    layers = []
    for cfg in (None, saved):
        L = B.Layer(rng.standard_normal((c_out, c, 3, 3), dtype=np.float32), rng.integers(0, 8, (c_out, c), dtype=np.uint8),
                    (rng.random((c_out, c)) < (1.0 if dense else 1 / 3.6)).astype(np.uint8), wl.pattern_library(wl.PATTERN_SEED),
                    stride=stride, dense=dense)
        if cfg:
            L.set_config(names[cfg["variant"]], cfg["ck"], cfg["waves"], cfg["ksplit"])
        layers.append(L)
    x = torch.randn(n, c, side, side, device="cuda")
    out, ws = torch.empty(layers[0].output_shape(n, side, side), device="cuda"), torch.empty(64 << 20, device="cuda")
    us = [[], []]
    for _ in range(9):
        for k, L in enumerate(layers):
            e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            L.conv2d_ws(x, None, out, workspace=ws, relu=True)
            e0.record()
            for _ in range(10):
                L.conv2d_ws(x, None, out, workspace=ws, relu=True)
            e1.record()
            torch.cuda.synchronize()
            us[k].append(e0.elapsed_time(e1) * 100)
    chosen, tuned = (sorted(v)[2] for v in us)
    print(f"  {c}@{side} / {stride} n={n}: chosen {chosen:.1f} us, tuned {tuned:.1f} us", flush=True)
    assert tuned <= 1.25 * chosen
    for L in layers:
        L.close()
