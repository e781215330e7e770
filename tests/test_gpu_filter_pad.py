"""Backward of layers whose filter count is no multiple of 8 over dY, codes and alphas padded to the next one: one filter, codes that
cross words, several taps and strides, one and several alphas, few input channels, accumulation into dW and the
bias gradient, against the direct-loop oracle; and a workspace that leaves the padding no room."""

import numpy as np
import pytest
import torch

from oracle import conv as oc
from oracle import ternarize as ot
from paper_1605_04711_amd import api
from paper_1605_04711_amd import workloads as wl
from parity import BF16_TOL, rel_err, to_dev_bf16, to_dev_f32, to_host_f64

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("groups", ["one", "filters"])
@pytest.mark.parametrize("n,h,w,c,o,r,stride,pad", [
    (130, 1, 1, 64, 10, 1, 1, 0),       # a classifier
    (3, 9, 7, 16, 1, 3, 1, 1),          # one filter
    (2, 12, 13, 40, 21, 3, 1, 1),       # rows of codes that end in any field
    (2, 13, 11, 24, 10, 5, 2, 2),       # residue classes
    (2, 10, 12, 3, 10, 3, 1, 1),        # few input channels
    (3, 28, 28, 1, 6, 5, 1, 0)])
def test_filter_pad(groups, n, h, w, c, o, r, stride, pad):
    rng = np.random.default_rng(n * h + o)
    geo = (stride,) * 2, (pad,) * 2, (1, 1)
    g = o if groups == "filters" else 1
    wt = (rng.standard_normal((o, c, r, r)) * 0.05).astype(np.float32)
    tw = api.twn_ternarize(to_dev_f32(wt), 0.7, groups=g, transposed=True)
    codes, _, alpha, _ = ot.ternarize(wt, 0.7, groups=g)
    p, q = (h + 2 * pad - r) // stride + 1, (w + 2 * pad - r) // stride + 1
    x = wl.bf16_round(rng.standard_normal((n, h, w, c)).astype(np.float32))
    dy = wl.bf16_round(rng.standard_normal((n, p, q, o)).astype(np.float32))
    ref_dx = oc.conv2d_bwd_data(dy, codes, alpha, (n, h, w, c), *geo)
    ref_dw = oc.conv2d_bwd_weight(x, dy, (o, c, r, r), *geo)
    xd, dyd = to_dev_bf16(x), to_dev_bf16(dy)
    guard = torch.full((o + 8, c, r, r), 3.0, device="cuda")        # rows past the filters stay as they are
    dw = guard[:o]
    dx, _, db = api.twn_conv2d_bwd_ste(xd, dyd, tw, *geo, dW=dw, need_dbias=True)
    assert rel_err(to_host_f64(dx), ref_dx) <= BF16_TOL
    # products of bf16 values are exact in float32, and each of a sum's `terms` additions rounds by at most 2^-24 of the magnitudes'
    # sum; one addition more where dW is accumulated into
    terms = n * p * q + 1
    bound = terms * 2.0 ** -24 * oc.conv2d_bwd_weight(np.abs(x), np.abs(dy), (o, c, r, r), *geo)
    assert (np.abs(to_host_f64(dw) - ref_dw) <= bound).all()
    assert (np.abs(to_host_f64(db) - oc.bias_grad(dy)) <= terms * 2.0 ** -24 * oc.bias_grad(np.abs(dy))).all()
    assert torch.equal(guard[o:], torch.full_like(guard[o:], 3.0))
    api.twn_conv2d_bwd_ste(xd, dyd, tw, *geo, need_dx=False, dW=dw, accumulate=True)
    assert (np.abs(to_host_f64(dw) - 2 * ref_dw) <= 2 * bound).all()


# n, h, w, c, o, r, pad: several taps over enough filters x channels or pixels for the kernel that reads patches with halo
TAPS_CASES = [(9, 33, 29, 72, 115, 3, 1),       # several pixel ranges, a ragged filter block
              (4, 130, 129, 8, 10, 3, 1),       # many ranges of few filters
              (1, 8, 8, 512, 510, 3, 1),        # one range: dW written directly, whole tiles and one that ends inside
              (1, 8, 8, 1024, 507, 2, 0),       # four taps
              (2, 9, 11, 200, 45, 5, 2)]        # 25 taps: three groups


@pytest.mark.parametrize("n,h,w,c,o,r,pad", TAPS_CASES)
def test_filter_pad_several_taps(n, h, w, c, o, r, pad):
    """dW and dX as in test_filter_pad; nothing behind the workspace of the query and behind dW is written."""
    rng = np.random.default_rng(n * h + o)
    geo = (1, 1), (pad,) * 2, (1, 1)
    wt = (rng.standard_normal((o, c, r, r)) * 0.05).astype(np.float32)
    tw = api.twn_ternarize(to_dev_f32(wt), 0.7, transposed=True)
    codes, _, alpha, _ = ot.ternarize(wt, 0.7)
    p, q = h + 2 * pad - r + 1, w + 2 * pad - r + 1
    x = wl.bf16_round(rng.standard_normal((n, h, w, c)).astype(np.float32))
    dy = wl.bf16_round(rng.standard_normal((n, p, q, o)).astype(np.float32))
    ref_dw = oc.conv2d_bwd_weight(x, dy, (o, c, r, r), *geo)
    # see test_filter_pad
    bound = (n * p * q + 1) * 2.0 ** -24 * oc.conv2d_bwd_weight(np.abs(x), np.abs(dy), (o, c, r, r), *geo)
    xd, dyd = to_dev_bf16(x), to_dev_bf16(dy)
    need = api.twn_conv2d_bwd_ste_workspace_bytes(x.shape, tw, *geo)
    ws = torch.full((need + (1 << 20),), 0x5A, dtype=torch.uint8, device="cuda")
    rows = torch.full((o + 8, c, r, r), 3.0, device="cuda")
    dx, _, _ = api.twn_conv2d_bwd_ste(xd, dyd, tw, *geo, dW=rows[:o], workspace=ws[:need])
    assert rel_err(to_host_f64(dx), oc.conv2d_bwd_data(dy, codes, alpha, x.shape, *geo)) <= BF16_TOL
    assert (np.abs(to_host_f64(rows[:o]) - ref_dw) <= bound).all()
    api.twn_conv2d_bwd_ste(xd, dyd, tw, *geo, need_dx=False, dW=rows[:o], accumulate=True, workspace=ws[:need])
    assert (np.abs(to_host_f64(rows[:o]) - 2 * ref_dw) <= 2 * bound).all()
    assert torch.equal(rows[o:], torch.full_like(rows[o:], 3.0))
    assert bool((ws[need:] == 0x5A).all())


def test_filter_pad_no_room():
    """Too little workspace for the padded copies, enough for the partial sums: the layer runs unpadded."""
    rng = np.random.default_rng(5)
    n, h, w, c, o = 4, 9, 8, 64, 10
    wt = rng.standard_normal((o, c, 3, 3)).astype(np.float32)
    tw = api.twn_ternarize(to_dev_f32(wt), 0.7, transposed=True)
    codes, _, alpha, _ = ot.ternarize(wt, 0.7)
    x, dy = (wl.bf16_round(rng.standard_normal((n, h, w, k)).astype(np.float32)) for k in (c, o))
    ref_dx = oc.conv2d_bwd_data(dy, codes, alpha, x.shape, (1, 1), (1, 1))
    ref_dw = oc.conv2d_bwd_weight(x, dy, wt.shape, (1, 1), (1, 1))
    bound = n * h * w * 2.0 ** -24 * oc.conv2d_bwd_weight(np.abs(x), np.abs(dy), wt.shape, (1, 1), (1, 1))
    need = api.twn_conv2d_bwd_ste_workspace_bytes(x.shape, tw, (1, 1), (1, 1))
    ws = torch.full((need,), 0x5A, dtype=torch.uint8, device="cuda")
    for size in (need, need - 256):
        dx, dw, _ = api.twn_conv2d_bwd_ste(to_dev_bf16(x), to_dev_bf16(dy), tw, (1, 1), (1, 1), workspace=ws[:size])
        assert rel_err(to_host_f64(dx), ref_dx) <= BF16_TOL
        assert (np.abs(to_host_f64(dw) - ref_dw) <= bound).all()
