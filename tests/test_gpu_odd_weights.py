"""Weight tensors that are no whole words, tiles or chunks: words of codes that cross filter taps, filters or several of both (one
to a few channels), one and several Deltas, and updates whose last chunk ends in every place of a group of four.  Codes, nnz
and the bytes are exact against the sort-based oracle; Delta and alpha within 1e-6 relative (float64 sums of the same values)."""

import numpy as np
import pytest
import torch

from oracle import sgd as osgd
from paper_1605_04711_amd import api
from paper_1605_04711_amd import workloads as wl
from parity import to_dev_f32
from test_gpu_sgd import close, f32
from test_gpu_ternarize import check_against_oracle

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("groups", [1, 3, "rows"])
@pytest.mark.parametrize("shape", [(3, 1, 1, 1), (6, 1, 5, 5), (9, 17, 1, 1), (3, 5, 1, 3), (15, 16, 3, 1), (18, 15, 3, 3), (33, 7, 2, 5),
                                   (171, 13, 3, 3), (3, 1000, 3, 3)])
def test_words_across_taps(shape, groups):
    w = wl.normal(13, shape[0] * 100 + shape[1], shape, std=0.05)
    check_against_oracle(w, 0.7, groups=shape[0] if groups == "rows" else groups)


@pytest.mark.parametrize("shape", [(1001, 63, 5, 5), (100300, 1, 4, 4)])
def test_paced_words(shape):
    """From 16 taps and 3 * 2^19 weights on the weights of a word are loaded one after the other."""
    check_against_oracle(wl.normal(13, shape[1], shape, std=0.05), 0.7)


@pytest.mark.parametrize("n", [1, 2, 3, 4, 5, 255, 1023, 1026, 4095, 4097, 8190, 12291])
def test_last_chunk_of_update(n):
    w, v, dw = (wl.normal(13, i, (1, n), std=0.05) for i in (1, 2, 3))
    guard = 64                              # elements behind the last one stay what they were
    W, V = (torch.full((n + guard,), 7.0, device="cuda") for _ in range(2))
    W[:n], V[:n] = to_dev_f32(w)[0], to_dev_f32(v)[0]
    ws = torch.empty(api.lib().twn_ternarize_workspace_bytes(api.ctypes.byref(api.WeightDesc(1, n, 1, 1)), 1), dtype=torch.uint8,
                     device="cuda")
    w_ref, v_ref = osgd.sgd_step(w, v, dw, f32(0.1), f32(0.9), f32(1e-4))
    W1, V1 = W[:n].view(1, n), V[:n].view(1, n)
    out = api.twn_ternarize(W1, 0.7)
    api.twn_sgd_update(W1, V1, to_dev_f32(dw), 0.1, 0.9, 1e-4, tern_workspace=ws)
    api.twn_ternarize_presummed(W1, out, ws, 0.7)
    torch.cuda.synchronize()
    assert close(W1.cpu().numpy(), w_ref) and close(V1.cpu().numpy(), v_ref)
    assert bool((W[n:] == 7.0).all()) and bool((V[n:] == 7.0).all())
    tw, _ = check_against_oracle(W1.cpu().numpy(), 0.7, transposed=False)
    assert torch.equal(tw.packed, out.packed) and torch.equal(tw.delta, out.delta) and torch.equal(tw.alpha, out.alpha)
