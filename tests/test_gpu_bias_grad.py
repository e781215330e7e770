"""Bias gradient: one and two launches, vector and single-channel loads, ragged channel groups and pixel ranges, against
float64 sums.  A channel's sum has fewer than 16 + 512 + 1024 float32 additions in a chain (pixels of a thread, rows of a
block, splits), so its error is below 1552 * 2^-24 = 9.3e-5 of the sum of magnitudes; 1e-5 is far above what random signs give."""

import numpy as np
import pytest
import torch

from paper_1605_04711_amd import api
from paper_1605_04711_amd import workloads as wl
from parity import to_dev_bf16, to_dev_f32, to_host_f64

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,h,w,o", [
    (1, 1, 1, 8), (1, 1, 1, 3),           # one pixel
    (2, 64, 64, 72), (2, 64, 64, 10),     # 8192 pixels: the last of one launch
    (3, 59, 47, 72), (3, 59, 47, 10),     # 8319: two launches, ragged ranges
    (1, 91, 91, 520), (1, 91, 91, 77),    # ragged last channel group
    (40, 33, 37, 8), (40, 33, 37, 1)])    # many ranges of few channels
@pytest.mark.parametrize("need_dw", [True, False])
def test_dbias(n, h, w, o, need_dw):
    rng = np.random.default_rng(n * h * w + o)
    x = torch.zeros((n, h, w, 8), dtype=torch.bfloat16, device="cuda")
    tw = api.twn_ternarize(to_dev_f32(rng.standard_normal((o, 8, 1, 1)).astype(np.float32)), 0.7, transposed=True)
    dy = wl.bf16_round((rng.standard_normal((n, h, w, o)) * 1e-5).astype(np.float32))
    ref = dy.astype(np.float64).sum(axis=(0, 1, 2))
    size = np.abs(dy.astype(np.float64)).sum(axis=(0, 1, 2))
    for _ in range(2):
        _, _, db = api.twn_conv2d_bwd_ste(x, to_dev_bf16(dy), tw, need_dx=False, need_dw=need_dw, need_dbias=True)
        assert np.all(np.abs(to_host_f64(db) - ref) <= 1e-5 * size)
