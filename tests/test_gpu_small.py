"""The kernel for problems of few output tiles (K shared out over the waves of a workgroup) at the edges of its tiles,
of its K ranges and of its dispatch, against the direct-loop oracle.  float32 outputs: only the order of the float32
sums differs, at most K * 2^-24 of the sum of magnitudes, 1e-4 under the metric of `parity` at these sizes."""

import numpy as np
import pytest

from oracle import conv as oc
from oracle import ternarize as ot
from paper_1605_04711_amd import api
from paper_1605_04711_amd import workloads as wl
from parity import BF16_TOL, rel_err, to_dev_bf16, to_dev_f32, to_host_f64

import torch

pytestmark = pytest.mark.gpu


def _layer(rng, x_shape, w_shape, groups=1):
    x = wl.bf16_round(rng.standard_normal(x_shape).astype(np.float32))
    w = (rng.standard_normal(w_shape) * np.sqrt(2.0 / np.prod(w_shape[1:]))).astype(np.float32)
    tw = api.twn_ternarize(to_dev_f32(w), 0.7, groups=groups, transposed=True)
    codes, _, alpha, _ = ot.ternarize(w.reshape(w.shape + (1,) * (4 - w.ndim)), 0.7, groups=groups)
    return x, tw, codes, alpha


@pytest.mark.parametrize("m,n,k", [
    (1, 8, 8), (1, 1000, 512), (31, 33, 72), (33, 64, 520), (32, 32, 4608), (16, 10, 1024),      # 32x32 tiles
    (100, 40, 16384),                                                                          # deepest K of the path
    (290, 900, 136), (640, 416, 584),                                                          # 32x64, eight waves
    (1040, 500, 1048), (1000, 1000, 1024), (2100, 264, 2048)])                                 # 32x64, four waves
def test_gemm(m, n, k):
    rng = np.random.default_rng(m + n + k)
    groups = n if (m + k) % 3 == 0 else 1
    x, tw, codes, alpha = _layer(rng, (m, k), (n, k), groups)
    ref = oc.gemm_fwd(x, codes.reshape(n, k), alpha)
    assert rel_err(to_host_f64(api.twn_gemm_fwd(to_dev_bf16(x), tw, y_dtype=torch.float32)), ref) <= 1e-4
    sc, sf = rng.uniform(0.5, 1.5, n).astype(np.float32), rng.standard_normal(n).astype(np.float32)
    res = wl.bf16_round(rng.standard_normal((m, n)).astype(np.float32))
    y = api.twn_gemm_fwd(to_dev_bf16(x), tw, scale=to_dev_f32(sc), shift=to_dev_f32(sf), residual=to_dev_bf16(res), relu=True)
    assert rel_err(to_host_f64(y), oc.epilogue(ref, sc, sf, res, relu=True)) <= BF16_TOL


@pytest.mark.parametrize("n,h,w,c,o,r,stride,pad,dil", [
    (1, 7, 7, 512, 96, 3, 1, 1, 1),          # one slab per tap, 49 pixels
    (1, 14, 13, 64, 40, 3, 2, 1, 1),         # strided: dX by divided taps
    (3, 9, 11, 24, 72, 3, 1, 2, 2),          # chunks of 8 channels, dilation
    (2, 15, 15, 40, 136, 5, 2, 2, 1),
    (5, 45, 61, 40, 72, 5, 2, 2, 1),         # 32x64 tiles, four waves, divided taps
    (6, 32, 32, 64, 64, 3, 2, 1, 1),         # dX by residue classes, one launch
    (9, 32, 32, 64, 64, 1, 2, 0, 1)])        # classes without taps
def test_convolution(n, h, w, c, o, r, stride, pad, dil):
    rng = np.random.default_rng(n * h + c + o)
    groups = o if c == 64 else 1
    x, tw, codes, alpha = _layer(rng, (n, h, w, c), (o, c, r, r), groups)
    geo = (stride,) * 2, (pad,) * 2, (dil,) * 2
    ref = oc.conv2d_fwd(x, codes, alpha, *geo)
    assert rel_err(to_host_f64(api.twn_conv2d_fwd(to_dev_bf16(x), tw, *geo, y_dtype=torch.float32)), ref) <= 1e-4
    assert rel_err(to_host_f64(api.twn_conv2d_fwd(to_dev_bf16(x), tw, *geo)), ref) <= BF16_TOL
    dy = wl.bf16_round(rng.standard_normal(ref.shape).astype(np.float32))
    dx, _, _ = api.twn_conv2d_bwd_ste(None, to_dev_bf16(dy), tw, *geo, need_dw=False, x_shape=x.shape)
    assert rel_err(to_host_f64(dx), oc.conv2d_bwd_data(dy, codes, alpha, x.shape, *geo)) <= BF16_TOL


@pytest.mark.parametrize("n,h,w,c,o,r,stride,pad,groups", [
    (1, 1, 1, 64, 8, 1, 1, 0, 1), (1, 4, 4, 64, 32, 1, 1, 0, 32), (1, 4, 4, 72, 33, 3, 1, 1, 1),         # one tile of 16 rows, whole and ragged
    (1, 7, 7, 512, 512, 3, 1, 1, 1),                                    # nine slabs a wave, five in flight
    (1, 17, 1, 8, 40, 5, 1, 2, 40), (2, 9, 5, 24, 257, 3, 2, 1, 1),     # chunks of 8 channels, odd columns
    (16, 16, 16, 64, 32, 3, 1, 1, 1), (1, 16, 16, 64, 512, 1, 2, 0, 1)])        # 256 tiles, the most; one slab of K for eight waves
def test_tiles_of_sixteen_pixels(n, h, w, c, o, r, stride, pad, groups):
    rng = np.random.default_rng(h * c + o)
    x, tw, codes, alpha = _layer(rng, (n, h, w, c), (o, c, r, r), groups)
    geo = (stride,) * 2, (pad,) * 2, (1, 1)
    ref = oc.conv2d_fwd(x, codes, alpha, *geo)
    assert rel_err(to_host_f64(api.twn_conv2d_fwd(to_dev_bf16(x), tw, *geo, y_dtype=torch.float32)), ref) <= 1e-4
    sc, sf = rng.uniform(0.5, 1.5, o).astype(np.float32), rng.standard_normal(o).astype(np.float32)
    res = rng.standard_normal(ref.shape).astype(np.float32)
    y = api.twn_conv2d_fwd(to_dev_bf16(x), tw, *geo, y_dtype=torch.float32, scale=to_dev_f32(sc), shift=to_dev_f32(sf),
                           residual=to_dev_f32(res), relu=True)
    assert rel_err(to_host_f64(y), oc.epilogue(ref, sc, sf, res, relu=True)) <= 2e-4        # a sum that cancels: twice the bound of the sum
    y = api.twn_conv2d_fwd(to_dev_bf16(x), tw, *geo, scale=to_dev_f32(sc), residual=to_dev_bf16(wl.bf16_round(res)))
    assert rel_err(to_host_f64(y), oc.epilogue(ref, sc, None, wl.bf16_round(res))) <= BF16_TOL
