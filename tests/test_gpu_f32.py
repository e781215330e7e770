"""The float32 path (float64 matrix cores) at the edges of its tiles, K blocks and dispatch, against the direct-loop
oracle.  Sums are float64 on both sides, so only the float32 roundings of the tail remain (FP32_TOL)."""

import numpy as np
import pytest

from oracle import conv as oc
from oracle import ternarize as ot
from paper_1605_04711_amd import api
from paper_1605_04711_amd import workloads as wl
from parity import BF16_TOL, FP32_TOL, rel_err, to_dev_bf16, to_dev_f32, to_host_f64

import torch

pytestmark = pytest.mark.gpu


def _weights(rng, shape, groups=1):
    w = (rng.standard_normal(shape) * np.sqrt(2.0 / np.prod(shape[1:]))).astype(np.float32)
    codes, _, alpha, _ = ot.ternarize(w.reshape(shape + (1,) * (4 - len(shape))), 0.7, groups=groups)
    return api.twn_ternarize(to_dev_f32(w), 0.7, groups=groups), codes, alpha


@pytest.mark.parametrize("m,n,k", [
    (1, 1, 1), (15, 17, 15), (16, 16, 16), (17, 10, 31), (64, 10, 512), (1, 100, 999),     # one wave to sixteen
    (130, 33, 66), (600, 290, 257),                                                       # 32 channels wide
    (1030, 1020, 67), (1000, 1024, 130),                                                  # 64 channels wide
    (33, 40, 12000)])                                                                     # K over workgroups
def test_gemm(m, n, k):
    rng = np.random.default_rng(m + n + k)
    groups = n if k % 2 else 1
    tw, codes, alpha = _weights(rng, (n, k), groups)
    xpad = to_dev_f32(rng.uniform(-1.0, 1.0, (m, k + 3)).astype(np.float32))              # rows at every alignment
    ref = oc.gemm_fwd(xpad[:, :k].cpu().numpy(), codes.reshape(n, k), alpha)
    assert rel_err(to_host_f64(api.twn_gemm_fwd(xpad[:, :k], tw, y_dtype=torch.float32)), ref) <= FP32_TOL
    sc = rng.uniform(0.5, 1.5, n).astype(np.float32)
    res = wl.bf16_round(rng.standard_normal((m, n)).astype(np.float32))
    y = api.twn_gemm_fwd(xpad[:, :k], tw, y_dtype=torch.bfloat16, scale=to_dev_f32(sc), residual=to_dev_bf16(res), relu=True)
    assert rel_err(to_host_f64(y), oc.epilogue(ref, sc, None, res, relu=True)) <= BF16_TOL


@pytest.mark.parametrize("n,h,w,c,o,r,stride,pad,dil", [
    (3, 11, 9, 1, 6, 5, 1, 2, 1),            # every element finds its tap; K = 25
    (2, 13, 12, 6, 40, 3, 2, 1, 1),
    (9, 28, 28, 3, 32, 3, 1, 0, 2),          # 32 channels wide, one wave
    (2, 10, 11, 4, 20, 3, 1, 1, 1),          # four elements per tap, ragged last block
    (4, 14, 14, 20, 24, 3, 2, 2, 2),
    (40, 12, 12, 32, 64, 5, 1, 0, 1),        # 32 channels wide, four waves
    (70, 16, 16, 8, 64, 1, 1, 0, 1)])        # 64 channels wide
def test_convolution(n, h, w, c, o, r, stride, pad, dil):
    rng = np.random.default_rng(n * h + c + o)
    tw, codes, alpha = _weights(rng, (o, c, r, r), o if c == 20 else 1)
    x = rng.uniform(-1.0, 1.0, (n, h, w, c)).astype(np.float32)
    geo = (stride,) * 2, (pad,) * 2, (dil,) * 2
    ref = oc.conv2d_fwd(x, codes, alpha, *geo)
    assert rel_err(to_host_f64(api.twn_conv2d_fwd(to_dev_f32(x), tw, *geo, y_dtype=torch.float32)), ref) <= FP32_TOL
