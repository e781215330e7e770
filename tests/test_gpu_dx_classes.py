"""Backward-data of strided layers by residue classes in one launch of the few-tile kernel: few pixels, filter counts that are no
whole slabs (words and single fields of codes), empty classes, one and several alphas, and neighbours of the rule that stay on
one problem, against the direct-loop oracle."""

import numpy as np
import pytest

from oracle import conv as oc
from oracle import ternarize as ot
from paper_1605_04711_amd import api
from paper_1605_04711_amd import workloads as wl
from parity import BF16_TOL, rel_err, to_dev_bf16, to_dev_f32, to_host_f64

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("groups", ["one", "filters"])
@pytest.mark.parametrize("n,h,w,c,o,r,stride,pad", [
    (3, 14, 14, 64, 512, 3, 2, 1),      # few pixels, whole slabs
    (2, 13, 11, 40, 200, 5, 2, 2),      # 200 filters: words that a slab boundary cuts
    (2, 9, 12, 24, 72, 7, 2, 3),        # 72 filters: single fields
    (1, 7, 9, 16, 1000, 1, 2, 0),       # three empty classes
    (1, 8, 8, 16, 264, 2, 2, 0),        # one tap per class
    (2, 6, 5, 8, 8, 3, 2, 1)])          # too short to split
def test_dx_classes(groups, n, h, w, c, o, r, stride, pad):
    rng = np.random.default_rng(n * h + o)
    geo = (stride,) * 2, (pad,) * 2, (1, 1)
    g = o if groups == "filters" else 1
    wt = (rng.standard_normal((o, c, r, r)) * 0.05).astype(np.float32)
    tw = api.twn_ternarize(to_dev_f32(wt), 0.7, groups=g, transposed=True)
    codes, _, alpha, _ = ot.ternarize(wt, 0.7, groups=g)
    p, q = (h + 2 * pad - r) // stride + 1, (w + 2 * pad - r) // stride + 1
    x = to_dev_bf16(np.zeros((n, h, w, c), np.float32))
    dy = wl.bf16_round(rng.standard_normal((n, p, q, o)).astype(np.float32))
    dx, _, _ = api.twn_conv2d_bwd_ste(x, to_dev_bf16(dy), tw, *geo, need_dw=False)
    ref = oc.conv2d_bwd_data(dy, codes, alpha, (n, h, w, c), *geo)
    assert rel_err(to_host_f64(dx), ref) <= BF16_TOL
