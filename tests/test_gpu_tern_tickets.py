"""The block that ends pass 2 last writes Delta, alpha and nnz: block counts around the sixteen shared tickets and at the
largest grid, several passes over one set of sums and one workspace; codes and scalars against the oracle."""

import pytest
import torch

from oracle import ternarize as ot
from paper_1605_04711_amd import api
from paper_1605_04711_amd import workloads as wl
from parity import to_dev_f32
from test_gpu_ternarize import check_against_oracle, pytestmark  # noqa: F401


@pytest.mark.parametrize("rows", [32, 15 * 32, 16 * 32, 17 * 32, 131072])      # 32 filters of 24 weights: a block of words
def test_block_counts(rows):
    check_against_oracle(wl.normal(17, rows, (rows, 24), std=0.05), 0.7, transposed=False)


@pytest.mark.parametrize("shape", [(64, 64, 3, 3), (40, 256), (33, 50)])
def test_sums_used_again(shape):
    w = wl.normal(17, shape[1], shape, std=0.05)
    dw = to_dev_f32(w)
    ws = torch.empty(98304, dtype=torch.uint8, device="cuda").fill_(0xFF)
    zero = torch.zeros_like(dw)
    api.twn_sgd_update(dw, torch.zeros_like(dw), zero, 0.0, 0.0, 0.0, tern_workspace=ws)
    tw = api.twn_ternarize(dw, 0.7)
    for f in (0.7, 0.5, 0.7):
        tw.alpha.zero_(); tw.delta.zero_(); tw.nnz.zero_(); tw.packed.zero_()
        api.twn_ternarize_presummed(dw, tw, ws, f)
        _, delta, alpha, nnz = ot.ternarize(w if w.ndim == 4 else w.reshape(*w.shape, 1, 1), f)
        assert int(tw.nnz[0]) == int(nnz[0]) and float(tw.delta[0]) == float(delta[0])
        assert abs(float(tw.alpha[0]) - float(alpha[0])) <= 1e-6 * float(alpha[0])
