"""Backward-data with one alpha per filter (or per group of filters): alpha*dY as two bf16 terms side by side, in every way
the terms and the repeated codes are prepared, against the direct-loop oracle.  With float32 output the only errors are the
2^-17 relative one of the two-term inputs and the float32 sums: against the metric's floor of 1 % of the RMS, an input
error of 2^-17 on each of K terms is at most 2^-17 * 100 = 8e-4 (random signs), bar 2e-3."""

import numpy as np
import pytest
import torch

from oracle import conv as oc
from oracle import ternarize as ot
from paper_1605_04711_amd import api
from paper_1605_04711_amd import workloads as wl
from parity import BF16_TOL, rel_err, to_dev_bf16, to_dev_f32, to_host_f64

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,h,w,c,o,r,stride,pad,groups", [
    (2, 9, 10, 64, 64, 3, 1, 1, 64),      # resident weights, terms formed on the way into LDS
    (3, 17, 8, 128, 64, 3, 1, 1, 4),      # the same, groups of 16 filters, two channel blocks
    (2, 13, 11, 24, 48, 3, 1, 1, 48),     # whole code words per tap
    (2, 13, 11, 24, 40, 3, 1, 1, 20),     # codes repeated field by field
    (2, 12, 12, 16, 10, 3, 1, 1, 10),     # filters no multiple of 8: one value per thread
    (6, 38, 36, 32, 64, 3, 2, 1, 64),     # residue classes
    (6, 38, 36, 32, 64, 1, 2, 0, 2),      # residue classes without taps: cleared pixels
    (3, 15, 15, 40, 72, 5, 2, 2, 72),     # divided taps
    (40, 1, 1, 200, 1000, 1, 1, 0, 1000)])
def test_dx(n, h, w, c, o, r, stride, pad, groups):
    rng = np.random.default_rng(n * h * c + o)
    wt = (rng.standard_normal((o, c, r, r)) * rng.uniform(0.2, 2.0, (o, 1, 1, 1))).astype(np.float32)
    tw = api.twn_ternarize(to_dev_f32(wt), 0.7, groups=groups, transposed=True)
    codes, _, alpha, _ = ot.ternarize(wt, 0.7, groups=groups)
    geo = (stride,) * 2, (pad,) * 2, (1, 1)
    p, q = (h + 2 * pad - r) // stride + 1, (w + 2 * pad - r) // stride + 1
    dy = wl.bf16_round(rng.standard_normal((n, p, q, o)).astype(np.float32))
    ref = oc.conv2d_bwd_data(dy, codes, alpha, (n, h, w, c), *geo)
    for dtype, bar in ((torch.float32, 2e-3), (torch.bfloat16, BF16_TOL)):
        dx = torch.full((n, h, w, c), 7.0, dtype=dtype, device="cuda")
        api.twn_conv2d_bwd_ste(None, to_dev_bf16(dy), tw, *geo, need_dw=False, x_shape=(n, h, w, c), dX=dx)
        got = to_host_f64(dx)
        assert rel_err(got, ref) <= bar
    # rounded to bf16 once: 2^-7 / sqrt(12) of the low end of a value's binade, 1.5e-3 of values spread over binades and
    # 1.66e-3 on these layers; rounding the sum of the high terms first makes it 2.00e-3
    assert np.linalg.norm(got - ref) <= 1.8e-3 * np.linalg.norm(ref)


def test_dx_of_the_longest_reduction():
    """2^30 - 8 filters in two groups: the two terms make a reduction within 63 of the largest int.  All codes +1 and
    dY = 1: the sum of the alphas, whose partial sums of whole steps are exact in float32."""
    o, c = (1 << 30) - 8, 8
    words = api.twn_packed_words_per_row(o)
    codes = torch.full((c, words), 0x55555555, dtype=torch.int32, device="cuda")
    tw = api.TernaryWeights(o, c, 1, 1, 2, None, codes, None, torch.tensor([1.0, 0.5], device="cuda"), None)
    dy = torch.ones((1, 1, 1, o), dtype=torch.bfloat16, device="cuda")
    dx = torch.zeros((1, 1, 1, c), dtype=torch.float32, device="cuda")
    ws = torch.empty(9 << 30, dtype=torch.uint8, device="cuda")      # what dX needs (the query covers dW too: 288 GB)
    api.twn_conv2d_bwd_ste(None, dy, tw, need_dw=False, x_shape=(1, 1, 1, c), dX=dx, workspace=ws)
    assert rel_err(to_host_f64(dx), np.full(c, (o // 2) * 1.5)) <= 1e-4
