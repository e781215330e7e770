"""float32 convolutions of short K whose channel count is no multiple of 4: all tile widths and K blocks, walks that end inside
a pair of row blocks, padding, strides and dilation, ragged pixels and channels, against the direct-loop oracle.  Sums are
float64 on both sides, so only the float32 roundings of the tail remain (FP32_TOL)."""

import numpy as np
import pytest
import torch

from oracle import conv as oc
from parity import FP32_TOL, rel_err, to_dev_f32, to_host_f64
from paper_1605_04711_amd import api
from test_gpu_f32 import _weights, pytestmark  # noqa: F401


@pytest.mark.parametrize("n,h,w,c,o,r,stride,pad,dil", [
    (1, 6, 6, 1, 1, 5, 1, 0, 1),             # four pixels, one channel
    (64, 28, 28, 1, 32, 5, 1, 0, 1),         # two row blocks per wave
    (65, 24, 23, 1, 64, 5, 1, 2, 1),         # 64 channels wide, padding
    (90, 31, 29, 3, 72, 3, 2, 1, 1),         # ragged channels, stride
    (33, 30, 31, 7, 33, 3, 1, 1, 2),         # K = 63: four blocks, dilation
    (70, 29, 30, 1, 16, 8, 1, 3, 1)])        # K = 64
def test_short(n, h, w, c, o, r, stride, pad, dil):
    rng = np.random.default_rng(n * h + c + o)
    tw, codes, alpha = _weights(rng, (o, c, r, r), o if c == 3 else 1)
    x = rng.uniform(-1.0, 1.0, (n, h, w, c)).astype(np.float32)
    sf = rng.uniform(-0.5, 0.5, o).astype(np.float32)
    geo = (stride,) * 2, (pad,) * 2, (dil,) * 2
    ref = oc.epilogue(oc.conv2d_fwd(x, codes, alpha, *geo), None, sf, None, relu=True)
    y = api.twn_conv2d_fwd(to_dev_f32(x), tw, *geo, y_dtype=torch.float32, shift=to_dev_f32(sf), relu=True)
    assert rel_err(to_host_f64(y), ref) <= FP32_TOL
