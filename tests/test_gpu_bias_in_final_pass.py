"""Bias gradients summed by the leading blocks of dW's final pass, in blocks of 256 and of 1024 threads, 8 channels a load and one:
bit for bit those of a call for the bias gradient alone, whose blocks of 512 threads add in the same order, and dW bit for bit
that of a call without a bias gradient."""

import re

import numpy as np
import pytest
import torch

from launches import conv, launches
from oracle import conv as oc
from paper_1605_04711_amd import api
from paper_1605_04711_amd import workloads as wl
from parity import to_dev_bf16, to_dev_f32, to_host_f64

# problem; the final pass that carries the bias gradient (its kernel, threads a block), or None
CASES = [
    ((2, 9, 9, 16, 24, 3, 1, 1, 1), ("weight_grad_reduce_kernel", 256)),             # sums scattered
    ((16, 20, 20, 24, 16, 1, 1, 0, 1), ("weight_grad_reduce_kernel", 1024)),
    ((4, 14, 14, 64, 64, 3, 1, 1, 1), ("weight_grad_reduce_rows_kernel", 256)),      # whole rows
    ((1, 64, 64, 128, 72, 3, 1, 1, 1), ("weight_grad_sum_kernel", 256)),             # several taps
    ((2, 64, 64, 64, 64, 3, 1, 1, 1), ("weight_grad_reduce_kernel", 1024)),          # 8192 pixels, the last of one launch
    ((3, 59, 47, 64, 72, 3, 1, 1, 1), None),                                         # 8319: launches of its own
    ((2, 30, 30, 3, 32, 3, 1, 1, 1), ("weight_grad_reduce_kernel", 256)),            # first layer
    ((2, 9, 11, 13, 12, 3, 1, 1, 4), ("weight_grad_reduce_kernel", 256)),            # single channels, several alphas
    ((5, 45, 61, 40, 72, 5, 2, 2, 1), ("weight_grad_reduce_kernel", 256)),
    ((1, 8, 8, 40, 72, 5, 2, 2, 1), None)]                                           # one range: no final pass


def test_cases_take_the_launches_they_name():
    """With dbias the final pass of the row is the build that sums it, without it the build that does not."""
    for parts in ("dw db", "dw"):
        answers = launches([dict(fn="bwd", parts=parts, d=conv(n, h, w, c, o, r, stride, pad, groups=groups))
                            for (n, h, w, c, o, r, stride, pad, groups), _ in CASES])
        for (_, final), a in zip(CASES, answers):
            own = [l for l in a["launches"] if l["kernel"] == "bias_grad_kernel"]
            passes = [l for l in a["launches"] if re.match("weight_grad_(reduce|sum)", l["kernel"])]
            assert bool(own) == (parts == "dw db" and final is None)
            if final is not None:
                assert [(l["kernel"], l["block"][0]) for l in passes] == [final]
            assert all(l["args"][-1] == ("true" if parts == "dw db" and final is not None else "false") for l in passes)


@pytest.mark.gpu
@pytest.mark.parametrize("n,h,w,c,o,r,stride,pad,groups", [c[0] for c in CASES])
def test_bias_in_final_pass(n, h, w, c, o, r, stride, pad, groups):
    rng = np.random.default_rng(n * h + o)
    geo = (stride,) * 2, (pad,) * 2, (1, 1)
    tw = api.twn_ternarize(to_dev_f32((rng.standard_normal((o, c, r, r)) * 0.05).astype(np.float32)), 0.7, groups=groups, transposed=True)
    p, q = (h + 2 * pad - r) // stride + 1, (w + 2 * pad - r) // stride + 1
    x = to_dev_bf16(wl.bf16_round(rng.standard_normal((n, h, w, c)).astype(np.float32)))
    dy = wl.bf16_round(rng.standard_normal((n, p, q, o)).astype(np.float32))
    d = to_dev_bf16(dy)
    _, dw, db = api.twn_conv2d_bwd_ste(x, d, tw, *geo, need_dx=False, need_dbias=True)
    _, _, alone = api.twn_conv2d_bwd_ste(x, d, tw, *geo, need_dx=False, need_dw=False, need_dbias=True)
    _, dw_alone, _ = api.twn_conv2d_bwd_ste(x, d, tw, *geo, need_dx=False)
    torch.cuda.synchronize()
    assert torch.equal(db, alone) and torch.equal(dw, dw_alone)
    # fewer than 632 float32 additions in a chain
    assert (np.abs(to_host_f64(db) - oc.bias_grad(dy)) <= 632 * 2.0 ** -24 * oc.bias_grad(np.abs(dy))).all()
