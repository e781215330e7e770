"""Bias gradient: one and two launches, vector and single-channel loads, ragged channel groups and pixel ranges, against
float64 sums.  A channel's sum has fewer than 32 + 8 + 512 + 80 float32 additions in a chain (pixels of a thread, the two stages over
the rows of a block, ranges), so its error is below 632 * 2^-24 = 3.8e-5 of the sum of magnitudes; 1e-5 is far above what
random signs give."""

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
    (40, 33, 37, 8), (40, 33, 37, 1),     # many ranges of few channels
    (1, 1, 3584, 72), (1, 1, 3585, 72), (1, 1, 5121, 72), (1, 1, 6143, 72),     # 512 pixels at once: seven; fours and a remainder
    (1, 1, 96, 33), (1, 1, 97, 33), (1, 1, 513, 33)])                           # 32 at once: three; eights and a remainder
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


@pytest.mark.parametrize("n,o", [(1024, 21), (1025, 21), (2047, 1025), (2049, 1025), (4096, 257), (8192, 10), (8192, 77), (8192, 72), (8281, 10001),
                                 (60025, 1201)])
def test_dbias_has_short_chains_of_additions(n, o):
    """One large value and many below half an ulp of it, which are lost one by one where they are added to it one by one: the
    error stays within what 64 ranges of every fourth pixel, their four sums and the ranges in turn would give."""
    small = 1.9921875 * 2.0 ** -25
    dy = torch.full((n, 1, 1, o), small, dtype=torch.bfloat16, device="cuda")
    dy[0] = 1.0
    tw = api.twn_ternarize(torch.ones((o, 8, 1, 1), device="cuda"), 0.7, transposed=True)
    x = torch.zeros((n, 1, 1, 8), dtype=torch.bfloat16, device="cuda")
    _, _, db = api.twn_conv2d_bwd_ste(x, dy, tw, need_dx=False, need_dw=False, need_dbias=True)
    exact = 1.0 + (n - 1) * small
    chain = -(-(-(-n // 64)) // 4) + 4 + 64
    assert float((db.double() - exact).abs().max()) <= chain * 2.0 ** -24 * exact
