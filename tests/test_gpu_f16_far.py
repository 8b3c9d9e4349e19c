"""The binary16 matrix kernel where its outputs need 64-bit addresses (a tile's images have 2^30 elements and more), in every
launch shape that has them, against the same layer on bands of the input, whose outputs do not: each sum is of the
same products in the same order, so every bit is the same, infinities and NaN among the inputs included."""

import pytest

import test_gpu_f16_matrix as matrix
from test_gpu_f16_matrix import torch                  # noqa: F401 (a fixture)

pytestmark = pytest.mark.gpu

# c_out, c_in, n, h, w, stride, what is launched
CASES = [
    (128, 3, 1, 2900, 2902, 1, 1),
    (128, 3, 1, 2901, 2901, 1, 0),
    (64, 3, 2, 2900, 2902, 1, 5),      # tiles of one image only would not need them
    (40, 3, 1, 5200, 5201, 1, 4),      # a filter block that is nearly empty
    (96, 3, 1, 6800, 6800, 2, 3),
    (96, 3, 1, 6800, 6801, 2, 2),
]


@pytest.mark.parametrize("case", CASES)
def test_far_outputs_are_those_of_bands(torch, case):
    import numpy as np
    c_out, c_in, n, h, w, stride, launches = case
    rng = np.random.default_rng(c_out + h)
    _, L = matrix._layer(rng, c_out, c_in, 0.6, stride, 1)
    gen = torch.Generator(device="cuda").manual_seed(h)
    x = torch.randn((n, c_in, h, w), generator=gen, device="cuda").half()
    x[-1, -1, -3, -2] = float("inf")
    x[0, 0, h // 2, 7] = float("nan")
    bias = torch.randn(c_out, generator=gen, device="cuda")
    shape = L.output_shape(n, h, w)
    ho, wo = shape[2:]
    size, guard = n * c_out * ho * wo, 4096
    assert size >= 1 << 30 and matrix._launches(L, x.data_ptr(), n, h, w) == launches
    print(f"  {case}", flush=True)
    buf = torch.full((size + 2 * guard,), 7.0, dtype=torch.float16, device="cuda")
    out = buf[guard:guard + size].view(shape)
    L.conv2d_f16(x, bias, out, relu=False)
    assert bool((buf[:guard] == 7).all()) and bool((buf[guard + size:] == 7).all())
    rows = 400
    for img in range(n):
        for a in range(0, ho, rows):
            # output rows a .. b - 1; the band has a row more at each end that is not the image's
            b = min(a + rows, ho)
            first, end = max(a - 1, 0) * stride, min((b + 1) * stride + 1, h)
            band = x[img:img + 1, :, first:end].contiguous()
            want = L.conv2d_f16(band, bias, relu=False)[0, :, a - first // stride:][:, :b - a]
            got = out[img, :, a:b]
            assert torch.equal(got.isnan(), want.isnan()), (img, a)
            assert torch.equal(got.nan_to_num(0.0), want.nan_to_num(0.0)), (img, a)
    assert not bool(out[-1, :, -3:, -4:].isfinite().all()) and bool(out[0, :, h // (2 * stride) - 1:h // (2 * stride) + 2, :8 // stride + 2].isnan().any())
    L.close()
