"""Weight gradient of three-channel first layers: tiles inside the image and over its edges, one and several tiles per
workgroup, filter counts that are no multiple of 64, odd padding, both strides, accumulation, and the shapes that stay on the
general kernel (odd width, wide filters), against the direct-loop oracle.  float32 sums of exact bf16 products in another order:
1e-4 under the metric of `parity`."""

import numpy as np
import pytest
import torch

from oracle import conv as oc
from paper_1605_04711_amd import api
from paper_1605_04711_amd import workloads as wl
from parity import rel_err, to_dev_bf16, to_dev_f32, to_host_f64

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,h,w,o,r,stride,pad", [
    (2, 32, 32, 128, 3, 1, 1),        # whole tiles, two groups of filters
    (1, 62, 64, 64, 7, 2, 3),         # 7x7/2, ragged rows
    (3, 17, 18, 72, 5, 1, 2),         # ragged tiles and filters
    (2, 31, 34, 8, 3, 2, 0),          # no padding, stride 2, eight filters
    (5, 7, 8, 64, 7, 1, 3),           # an image smaller than a tile
    (1, 9, 10, 16, 2, 1, 1),          # even filter, odd padding
    (1, 8, 6, 24, 1, 1, 0),           # one tap
    (9, 97, 200, 64, 3, 1, 1),        # several tiles per workgroup
    (2, 15, 17, 64, 3, 1, 1),         # odd width: general kernel
    (1, 20, 20, 16, 9, 1, 4)])        # nine taps a row: general kernel
def test_dw_first(n, h, w, o, r, stride, pad):
    rng = np.random.default_rng(n * h + w + o)
    geo = (stride,) * 2, (pad,) * 2, (1, 1)
    tw = api.twn_ternarize(to_dev_f32(rng.standard_normal((o, 3, r, r)).astype(np.float32)), 0.7, transposed=True)
    p, q = (h + 2 * pad - r) // stride + 1, (w + 2 * pad - r) // stride + 1
    x = wl.bf16_round(rng.standard_normal((n, h, w, 3)).astype(np.float32))
    dy = wl.bf16_round(rng.standard_normal((n, p, q, o)).astype(np.float32))
    ref = oc.conv2d_bwd_weight(x, dy, (o, 3, r, r), *geo)
    _, dw, db = api.twn_conv2d_bwd_ste(to_dev_bf16(x), to_dev_bf16(dy), tw, *geo, need_dx=False, need_dbias=True)
    assert rel_err(to_host_f64(dw), ref) <= 1e-4
    assert np.allclose(to_host_f64(db), dy.astype(np.float64).sum(axis=(0, 1, 2)), rtol=0, atol=1e-5 * np.abs(dy).sum(axis=(0, 1, 2)).max())
    again = torch.full_like(dw, 3.0)
    api.twn_conv2d_bwd_ste(to_dev_bf16(x), to_dev_bf16(dy), tw, *geo, need_dx=False, dW=again)
    assert torch.equal(again, dw)         # overwritten, and the same bits run to run
    api.twn_conv2d_bwd_ste(to_dev_bf16(x), to_dev_bf16(dy), tw, *geo, need_dx=False, dW=again, accumulate=True)
    assert rel_err(to_host_f64(again), 2 * ref) <= 1e-4


@pytest.mark.parametrize("h,w,o,r,stride,pad", [
    (19, 36, 64, 3, 1, 0),            # one output row and two columns more than whole tiles, no padding
    (22, 26, 24, 5, 1, 1),
    (35, 38, 72, 7, 2, 2),
    (9, 12, 10, 3, 1, 1)])            # fewer than a tile, padded filters
def test_values_that_are_not_finite_stay_in_their_taps(h, w, o, r, stride, pad):
    """A value of X reaches the taps whose sum contains it and no other, also where a tile reaches past the output."""
    rng = np.random.default_rng(h + o)
    geo = (stride,) * 2, (pad,) * 2, (1, 1)
    tw = api.twn_ternarize(to_dev_f32(rng.standard_normal((o, 3, r, r)).astype(np.float32)), 0.7, transposed=True)
    p, q = (h + 2 * pad - r) // stride + 1, (w + 2 * pad - r) // stride + 1
    x = wl.bf16_round(rng.standard_normal((2, h, w, 3)).astype(np.float32))
    dy = wl.bf16_round(np.abs(rng.standard_normal((2, p, q, o)).astype(np.float32)) + 0.5)
    x[0, :, w - 1, 0] = np.inf
    x[1, h - 1, :, 1] = np.nan
    x[0, h - 1, 0, 2] = -np.inf
    at = np.pad(x, ((0, 0), (pad, pad + stride), (pad, pad + stride), (0, 0))).astype(np.float64)
    ref = np.zeros((o, 3, r, r))
    with np.errstate(invalid="ignore"):
        for i in range(r):
            for j in range(r):
                win = at[:, i:i + stride * (p - 1) + 1:stride, j:j + stride * (q - 1) + 1:stride]
                ref[:, :, i, j] = (win[..., None, :] * dy[..., None].astype(np.float64)).sum(axis=(0, 1, 2))
    _, dw, _ = api.twn_conv2d_bwd_ste(to_dev_bf16(x), to_dev_bf16(dy), tw, *geo, need_dx=False)
    got = to_host_f64(dw)
    fine = np.isfinite(ref)
    assert fine.any() and not fine.all()
    assert np.array_equal(np.isfinite(got), fine)
    assert rel_err(got[fine], ref[fine]) <= 1e-4
