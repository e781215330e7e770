"""Backward-data with several alphas taken with their codes: every tile of the few-tile kernel, taps of whole slabs, of single
chunks and plain products, one problem and residue classes, filters per alpha, the largest table and the first beyond it.  One
rounding to bf16 is at most 2^-9 = 1.95e-3 of a value, so the 2-norm error stays below 2.0e-3 with the terms' own 3e-6; with one
term of alpha dropped it would be 2.3e-3 (two roundings of 1.66e-3 each).  float32 outputs keep the terms of alpha * dY (2^-18 of a product)."""

import numpy as np
import pytest
import torch

from oracle import conv as oc
from oracle import ternarize as ot
from paper_1605_04711_amd import api
from paper_1605_04711_amd import workloads as wl
from parity import BF16_TOL, rel_err, to_dev_bf16, to_dev_f32, to_host_f64

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,h,w,c,o,r,stride,pad,dil,per", [
    (1, 7, 7, 64, 128, 3, 1, 1, 1, 1),        # 32x32 tiles, whole slabs
    (3, 14, 14, 128, 192, 3, 1, 1, 1, 1),     # 32x64 tiles, eight waves
    (5, 28, 27, 200, 128, 3, 1, 1, 1, 4),     # four waves, several filters per alpha
    (2, 9, 11, 40, 72, 3, 1, 1, 2, 1),        # chunks that find their taps, dilation
    (2, 13, 11, 40, 200, 5, 2, 2, 1, 1),      # residue classes, chunks
    (2, 12, 12, 64, 512, 3, 2, 1, 1, 2),      # residue classes, whole slabs
    (33, 1, 1, 72, 1000, 1, 1, 0, 1, 1),      # plain product, K = 1000
    (9, 1, 1, 16, 4096, 1, 1, 0, 1, 1),       # the largest table
    (9, 1, 1, 16, 4104, 1, 1, 0, 1, 1)])      # beyond it: terms of alpha * dY
def test_dx_alpha(n, h, w, c, o, r, stride, pad, dil, per):
    rng = np.random.default_rng(n * h + o)
    geo = (stride,) * 2, (pad,) * 2, (dil,) * 2
    groups = o // per
    wt = (rng.standard_normal((o, c, r, r)) * 0.05 * np.exp(rng.standard_normal((o, 1, 1, 1)))).astype(np.float32)
    if per == 1:
        wt[o // 2] = 0.0                      # an alpha of zero
    tw = api.twn_ternarize(to_dev_f32(wt), 0.7, groups=groups, transposed=True)
    codes, _, alpha, _ = ot.ternarize(wt, 0.7, groups=groups)
    p, q = (h + 2 * pad - dil * (r - 1) - 1) // stride + 1, (w + 2 * pad - dil * (r - 1) - 1) // stride + 1
    x = to_dev_bf16(np.zeros((n, h, w, c), np.float32))
    dy = wl.bf16_round((rng.standard_normal((n, p, q, o)) * 1e-5).astype(np.float32))
    ref = oc.conv2d_bwd_data(dy, codes, alpha, (n, h, w, c), *geo)
    for dtype, norm, worst in ((torch.bfloat16, 2.0e-3, BF16_TOL), (torch.float32, 4e-6, 2e-3)):
        dx, _, _ = api.twn_conv2d_bwd_ste(x, to_dev_bf16(dy), tw, *geo, need_dw=False, dx_dtype=dtype)
        got = to_host_f64(dx)
        assert np.linalg.norm(got - ref) <= norm * np.linalg.norm(ref)
        assert rel_err(got, ref) <= worst


LARGE_CASES = [
    (100, 9, 11, 72, 128, 3, 1, 1, 1, 1),     # two slabs per tap, ragged rows and columns
    (60, 13, 12, 136, 192, 3, 1, 1, 2, 3),    # three slabs per tap, dilation, several filters per alpha
    (170, 9, 11, 136, 128, 3, 1, 1, 1, 1),    # 528 tiles: several per workgroup
    (9, 20, 21, 264, 1024, 1, 1, 0, 1, 1),    # plain product, the largest table
    (3, 9, 11, 72, 128, 3, 1, 1, 1, 1),       # the same with K cut into ranges: terms of alpha * dY
    (2, 13, 12, 136, 192, 3, 1, 1, 2, 3),
    (5, 8, 8, 128, 64, 1, 1, 0, 1, 1),        # plain product of one slab
    (1, 20, 21, 264, 1024, 1, 1, 0, 1, 1),
    (1, 6, 7, 72, 1088, 1, 1, 0, 1, 1),       # beyond the table
    (8, 66, 66, 128, 64, 3, 1, 1, 1, 1),      # 64 filters: terms formed in the contraction
    (3, 55, 56, 64, 128, 3, 2, 1, 1, 1),      # residue classes, 64 columns
    (9, 33, 31, 136, 192, 3, 2, 1, 1, 2),     # residue classes, 136 columns
    (9, 33, 31, 72, 64, 1, 2, 0, 1, 1),       # three empty classes, one slab
    (2, 67, 65, 24, 1088, 1, 2, 0, 1, 1)]     # beyond the table: terms of alpha * dY


@pytest.mark.parametrize("n,h,w,c,o,r,stride,pad,dil,per", LARGE_CASES)
def test_dx_alpha_large_kernels(knob, n, h, w, c, o, r, stride, pad, dil, per):
    """The same in the kernels that problems of more tiles run."""
    knob("TWN_SMALL", 0)
    rng = np.random.default_rng(n * h + o)
    geo = (stride,) * 2, (pad,) * 2, (dil,) * 2
    wt = (rng.standard_normal((o, c, r, r)) * 0.05 * np.exp(rng.standard_normal((o, 1, 1, 1)))).astype(np.float32)
    tw = api.twn_ternarize(to_dev_f32(wt), 0.7, groups=o // per, transposed=True)
    codes, _, alpha, _ = ot.ternarize(wt, 0.7, groups=o // per)
    x = to_dev_bf16(np.zeros((n, h, w, c), np.float32))
    p, q = (h + 2 * pad - dil * (r - 1) - 1) // stride + 1, (w + 2 * pad - dil * (r - 1) - 1) // stride + 1
    dy = wl.bf16_round((rng.standard_normal((n, p, q, o)) * 1e-5).astype(np.float32))
    ref = oc.conv2d_bwd_data(dy, codes, alpha, (n, h, w, c), *geo)
    dx, _, _ = api.twn_conv2d_bwd_ste(x, to_dev_bf16(dy), tw, *geo, need_dw=False)
    got = to_host_f64(dx)
    assert np.linalg.norm(got - ref) <= 2.0e-3 * np.linalg.norm(ref)
    assert rel_err(got, ref) <= BF16_TOL
    again, _, _ = api.twn_conv2d_bwd_ste(x, to_dev_bf16(dy), tw, *geo, need_dw=False)
    assert torch.equal(again, dx)


# few-tile kernel, each of its tiles, taps of whole slabs, chunks, plain product, residue classes; then (second field 0) the
# persistent kernel over taps and as a plain product, and the batched residue classes of 64 and of more columns
EXACT_CASES = [
    (1, 2, 10, 10, 64, 128, 3, 1, 1), (1, 3, 21, 21, 256, 128, 3, 1, 1), (1, 5, 28, 27, 200, 128, 3, 1, 1),
    (1, 2, 9, 11, 40, 72, 3, 1, 1), (1, 33, 1, 1, 72, 200, 1, 1, 0), (1, 2, 13, 11, 40, 72, 3, 2, 1),
    (0, 100, 9, 11, 72, 128, 3, 1, 1), (0, 5, 8, 8, 128, 64, 1, 1, 0), (0, 3, 55, 56, 64, 128, 3, 2, 1), (0, 9, 33, 31, 136, 192, 3, 2, 1)]


@pytest.mark.parametrize("small,n,h,w,c,o,r,stride,pad", EXACT_CASES)
def test_dx_alpha_keeps_every_bit_of_alpha(knob, small, n, h, w, c, o, r, stride, pad):
    """dY has one value, a power of two, in a neighbourhood, so every value of dX is one product alpha * dY: a float32.  The alphas
    lie 1..3 * 2^-19 beside a tie of bf16; two bf16 terms of one would be the tie itself and round the other way."""
    knob("TWN_SMALL", small)
    rng = np.random.default_rng(n * h + o)
    step = np.arange(o) % 3 + 1
    v = np.where(np.arange(o) % 2, 1 + 2.0**-8 + step * 2.0**-19, 1 + 2.0**-7 + 2.0**-8 - step * 2.0**-19).astype(np.float32)
    wt = v[:, None, None, None] * rng.choice(np.float32([-1, 1]), (o, c, r, r))
    tw = api.twn_ternarize(to_dev_f32(wt), 0.7, groups=o, transposed=True)
    assert np.array_equal(tw.alpha.cpu().numpy(), v)
    geo = (stride,) * 2, (pad,) * 2, (1, 1)
    p, q = (h + 2 * pad - r) // stride + 1, (w + 2 * pad - r) // stride + 1
    dy = np.zeros((n, p, q, o), np.float32)
    at = dy[:, ::r, ::r]                          # r apart: no value of dX sees two of them
    which = rng.integers(0, o, at.shape[:3])
    np.put_along_axis(at, which[..., None], rng.choice(np.float32([0.5, -1, 2]), at.shape[:3])[..., None], 3)
    x = to_dev_bf16(np.zeros((n, h, w, c), np.float32))
    dx, _, _ = api.twn_conv2d_bwd_ste(x, to_dev_bf16(dy), tw, *geo, need_dw=False)
    exact = oc.conv2d_bwd_data(dy, np.sign(wt).astype(np.int8), v, (n, h, w, c), *geo)
    assert np.count_nonzero(exact) and np.array_equal(to_host_f64(dx), wl.bf16_round(exact.astype(np.float32)))
