"""The two tiles of one workgroup per CU (128 x 256 and 256 x 128), which large problems get by how they fill the chip: ragged
row and column blocks, one tile per workgroup and (the last shape: 281 and 282 tiles on 256 CUs) a walk over two, residual and
several alphas, against the oracle."""

import numpy as np
import pytest

from oracle import conv as oc
from oracle import ternarize as ot
from paper_1605_04711_amd import api
from paper_1605_04711_amd import workloads as wl
from parity import BF16_TOL, rel_err, to_dev_bf16, to_dev_f32, to_host_f64

pytestmark = pytest.mark.gpu


CASES = [
    (1, 16, 16, 128, 128, 1),          # one tile, whole
    (1, 15, 17, 128, 136, 1),          # a row short, a column block of 8
    (3, 13, 11, 192, 264, 264),        # ragged in both, one alpha per filter
    (2, 9, 7, 128, 72, 1),             # less than a tile
    (2, 130, 138, 64, 136, 1)]         # more tiles than CUs


@pytest.mark.parametrize("tile", [17, 18])
@pytest.mark.parametrize("n,h,w,c,o,groups", CASES)
def test_wide_tiles(knob, tile, n, h, w, c, o, groups):
    knob("TWN_TILE", tile)
    rng = np.random.default_rng(n * h + o)
    x = wl.bf16_round(rng.standard_normal((n, h, w, c)).astype(np.float32))
    wt = (rng.standard_normal((o, c, 3, 3)) * 0.05).astype(np.float32)
    res = wl.bf16_round(rng.standard_normal((n, h, w, o)).astype(np.float32))
    scale, shift = (1.0 + 0.1 * rng.standard_normal(o)).astype(np.float32), (0.1 * rng.standard_normal(o)).astype(np.float32)
    tw = api.twn_ternarize(to_dev_f32(wt), 0.7, groups=groups)
    codes, _, alpha, _ = ot.ternarize(wt, 0.7, groups=groups)
    y = api.twn_conv2d_fwd(to_dev_bf16(x), tw, (1, 1), (1, 1), (1, 1), scale=to_dev_f32(scale), shift=to_dev_f32(shift),
                           residual=to_dev_bf16(res), relu=True)
    ref = oc.epilogue(oc.conv2d_fwd(x, codes, alpha, (1, 1), (1, 1), (1, 1)), scale=scale, shift=shift, residual=res, relu=True)
    assert rel_err(to_host_f64(y), ref) <= BF16_TOL
