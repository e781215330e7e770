"""Large flat tensors, codes from one stream of W: whole and ragged last chunks, samples that mislead (scales that differ
between stretches, an outlier that moves Delta out of the band, all weights equal, zeros), against the oracle and, bit for bit,
against the two passes that a workspace without room for marks takes."""

import ctypes

import numpy as np
import pytest
import torch

from paper_1605_04711_amd import api
from test_gpu_ternarize import pytestmark  # noqa: F401


def both(w):
    rows, c = w.shape
    least = torch.empty(98304, dtype=torch.uint8, device="cuda")
    assert api.lib().twn_ternarize_workspace_bytes(ctypes.byref(api.WeightDesc(rows, c, 1, 1)), 1) > least.numel()
    one = api.twn_ternarize(w, 0.7)
    again = api.twn_ternarize(w, 0.7)
    two = api.twn_ternarize(w, 0.7, workspace=least)
    for t in ("packed", "delta", "nnz", "alpha"):
        assert torch.equal(getattr(one, t), getattr(again, t)), t
    for t in ("packed", "delta", "nnz"):
        assert torch.equal(getattr(one, t), getattr(two, t)), t
    assert torch.allclose(one.alpha, two.alpha, rtol=1e-7, atol=0)
    # the definition itself, in float64
    a = w.abs().double()
    delta = np.float32(np.float64(np.float32(0.7)) * float(a.sum()) / w.numel())
    assert abs(float(one.delta[0]) - delta) <= 1e-6 * abs(delta)
    on = w.abs() > one.delta[0]
    assert int(one.nnz[0]) == int(on.sum())
    if int(one.nnz[0]):
        assert abs(float(one.alpha[0]) - float(a[on].mean())) <= 1e-6 * float(one.alpha[0])
    return one


@pytest.mark.parametrize("rows,c", [(4096, 4096), (131072, 128), (4099, 4224), (24577, 896)])
def test_normal(rows, c):
    g = torch.Generator(device="cuda")
    g.manual_seed(rows)
    both(torch.randn((rows, c), generator=g, device="cuda") * 0.03)


@pytest.mark.parametrize("kind", ["scales", "outlier", "equal", "zero", "sparse", "two values"])
def test_misleading(kind):
    g = torch.Generator(device="cuda")
    g.manual_seed(5)
    w = torch.randn((4099, 4224), generator=g, device="cuda")
    if kind == "scales":
        w *= torch.logspace(-3, 3, 4099, device="cuda")[:, None]
    elif kind == "outlier":
        w.view(-1)[12345678] = 1e9
    elif kind == "equal":
        w.fill_(-0.25)
    elif kind == "zero":
        w.zero_()
    elif kind == "sparse":
        w *= (torch.rand(w.shape, generator=g, device="cuda") < 1e-5)
    else:
        w = torch.where(w > 0.5, 1.0, 0.7 * 0.30854)       # Delta next to the smaller value
    both(w.contiguous())
