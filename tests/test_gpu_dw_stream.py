"""Depthwise fp32 layers whose outputs take another kind of store for their size (csrc/kernel_dw.hip) give the values of
smaller calls, bit for bit: eight and four outputs per lane, whole and unaligned input vectors, both strides."""

import numpy as np
import pytest

from paper_2001_00138_amd import binding as B
from paper_2001_00138_amd import workloads as wl

pytestmark = pytest.mark.gpu


# images, channels, h, w, stride; outputs above and, image by image, below 16 MB: both tensors of up to 64 MB, of more, and
# too large for the last-level cache
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
