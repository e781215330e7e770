"""Codes come to the persistent kernel's workgroups in chunks of two or four slabs of K, the last one of a tile shorter: inner
products whose K is one to nine slabs, over tiles that leave a workgroup one or several, must be those of a float64 product.
The sums are float32 (K * 2^-24 of the sum of magnitudes), the outputs bf16: half an ulp of the value is 2^-9."""

import numpy as np
import pytest
import torch

from launches import gemm, launches
from oracle import packing as op
from paper_1605_04711_amd import api
from paper_1605_04711_amd import workloads as wl
from parity import BF16_TOL, rel_err, to_dev_bf16, to_host_f64

CASES = [(14, 64 * 700 - 9, 128), (15, 128 * 600 - 3, 104), (16, 128 * 700 - 5, 64), (17, 128 * 300 - 7, 264), (18, 256 * 300 - 11, 136),
         (14, 50, 72), (18, 200, 72)]
SLABS = [1, 2, 3, 4, 5, 9]
BUILDS = {14: (64, 128, 4), 15: (128, 128, 2), 16: (128, 64, 4), 17: (128, 256, 4), 18: (256, 128, 4)}       # rows, columns, slabs a chunk


def test_cases_take_the_kernel_with_load_waves():
    answers = launches([dict(fn="gemm", d=gemm(m, n, 64 * slabs), env={"TWN_TILE": tile, "TWN_STREAM_PC": 4})
                        for tile, m, n in CASES for slabs in SLABS])
    walks = set()
    for (tile, m, n), a in zip([c for c in CASES for _ in SLABS], answers):
        (l,) = a["launches"]
        rows, cols, chunk = BUILDS[tile]
        assert l["kernel"] == "conv_stream_pc_kernel" and l["args"][:2] == [str(rows), str(cols)] and l["args"][7] == str(chunk)
        walks.add((tile, -(-m // rows) * -(-n // cols) > l["grid"][0]))
    assert walks == {(tile, True) for tile in BUILDS} | {(14, False), (18, False)}


@pytest.mark.gpu
@pytest.mark.parametrize("tile,m,n", CASES)
@pytest.mark.parametrize("slabs", SLABS)
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
