"""Weight gradient over patches with halo: shapes of every patch (images, rows, columns), ragged images and channel counts,
more than nine taps, one and several pixel ranges, accumulation, against the direct-loop oracle.  float32 sums of exact
bf16 products in another order: 1e-4 under the metric of `parity`."""

import numpy as np
import pytest
import torch

from oracle import conv as oc
from paper_1605_04711_amd import api
from paper_1605_04711_amd import workloads as wl
from parity import rel_err, to_dev_bf16, to_dev_f32, to_host_f64

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,h,w,c,o,r,pad,dil", [
    (2, 16, 16, 128, 64, 3, 1, 1),        # whole tiles, 4x8 patches
    (3, 13, 21, 128, 72, 3, 1, 1),        # ragged patches, filter block of 8
    (5, 14, 14, 128, 64, 3, 1, 1),        # images no multiple of the patch's
    (33, 7, 7, 136, 64, 3, 1, 1),         # channel block of 8 in the last tile
    (2, 9, 11, 200, 48, 5, 2, 1),         # 25 taps: three groups
    (2, 12, 10, 104, 80, 3, 2, 2),        # dilation, more padding than halo
    (1, 8, 8, 1024, 512, 2, 0, 1),        # four taps, one pixel range: dW written directly
    (4, 130, 129, 64, 64, 3, 1, 1)])      # few tiles, many ranges
def test_dw(n, h, w, c, o, r, pad, dil):
    rng = np.random.default_rng(n * h + c)
    geo = (1, 1), (pad,) * 2, (dil,) * 2
    tw = api.twn_ternarize(to_dev_f32(rng.standard_normal((o, c, r, r)).astype(np.float32)), 0.7, transposed=True)
    p, q = h + 2 * pad - dil * (r - 1), w + 2 * pad - dil * (r - 1)
    x = wl.bf16_round(rng.standard_normal((n, h, w, c)).astype(np.float32))
    dy = wl.bf16_round(rng.standard_normal((n, p, q, o)).astype(np.float32))
    ref = oc.conv2d_bwd_weight(x, dy, (o, c, r, r), *geo)
    _, dw, _ = api.twn_conv2d_bwd_ste(to_dev_bf16(x), to_dev_bf16(dy), tw, *geo, need_dx=False)
    assert rel_err(to_host_f64(dw), ref) <= 1e-4
    again = torch.full_like(dw, 3.0)
    api.twn_conv2d_bwd_ste(to_dev_bf16(x), to_dev_bf16(dy), tw, *geo, need_dx=False, dW=again)
    assert torch.equal(again, dw)         # overwritten, and the same bits run to run
    api.twn_conv2d_bwd_ste(to_dev_bf16(x), to_dev_bf16(dy), tw, *geo, need_dx=False, dW=again, accumulate=True)
    assert rel_err(to_host_f64(again), 2 * ref) <= 1e-4
