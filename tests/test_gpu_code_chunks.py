"""Codes come to the persistent kernel's workgroups in chunks of two or four slabs of K, the last one of a tile shorter: inner
products whose K is one to nine slabs, over tiles that leave a workgroup one or several, must be those of a float64 product.
The sums are float32 (K * 2^-24 of the sum of magnitudes), the outputs bf16: half an ulp of the value is 2^-9."""

import numpy as np
import pytest
import torch

from oracle import packing as op
from paper_1605_04711_amd import api
from paper_1605_04711_amd import workloads as wl
from parity import BF16_TOL, rel_err, to_dev_bf16, to_host_f64

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("tile,m,n", [(14, 64 * 700 - 9, 128), (15, 128 * 600 - 3, 104), (16, 128 * 700 - 5, 64), (17, 128 * 300 - 7, 264),
                                      (18, 256 * 300 - 11, 136), (14, 50, 72), (18, 200, 72)])
@pytest.mark.parametrize("slabs", [1, 2, 3, 4, 5, 9])
def test_chunks_of_codes(knob, tile, m, n, slabs):
    knob("TWN_TILE", tile)
    knob("TWN_STREAM_PC", 4)
    k = 64 * slabs
    rng = np.random.default_rng(tile * 100 + slabs)
    x = wl.bf16_round(rng.standard_normal((m, k)).astype(np.float32))
    codes = rng.integers(-1, 2, (n, k)).astype(np.int8)
    tw = api.twn_ternarize(torch.from_numpy(codes.astype(np.float32)).cuda(), 0.1)
    assert np.array_equal(tw.packed.cpu().numpy().view(np.uint32), op.pack_weights(codes.reshape(n, k, 1, 1)))
    y = to_host_f64(api.twn_gemm_fwd(to_dev_bf16(x), tw))
    assert rel_err(y, x.astype(np.float64) @ codes.T.astype(np.float64) * float(tw.alpha.cpu()[0])) <= BF16_TOL
