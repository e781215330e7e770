"""Backward-data with several alphas in 128x128 tiles: ragged rows and columns, one slab per tap and several, a plain product, one
tile per workgroup and several.  The bound is that of the other kernels with alphas: one rounding to bf16 is at most 2^-9 of a
value, 2.0e-3 in the 2-norm with the float32 sums."""

import numpy as np
import pytest

from launches import conv, launches
from oracle import conv as oc
from oracle import ternarize as ot
from paper_1605_04711_amd import api
from paper_1605_04711_amd import workloads as wl
from parity import BF16_TOL, rel_err, to_dev_bf16, to_dev_f32, to_host_f64

CASES = [
    (120, 9, 11, 136, 128, 3, 1),             # two slabs per tap
    (500, 9, 11, 72, 64, 3, 1),               # one, a walk over two tiles
    (130, 9, 11, 200, 576, 1, 1)]             # plain product, several filters per alpha


def test_cases_take_tiles_of_128_rows():
    answers = launches([dict(fn="bwd", parts="dx", d=conv(n, h, w, c, o, r, groups=o // per), env={"TWN_SMALL": 0})
                        for n, h, w, c, o, r, per in CASES])
    last = [a["launches"][-1] for a in answers]
    assert [l["args"][:2] + l["args"][-1:] for l in last] == [["128", "128", "true"]] * len(CASES)
    assert [-(-n * h * w // 128) * -(-c // 128) > l["grid"][0] for (n, h, w, c, *_), l in zip(CASES, last)] == [False, True, False]


@pytest.mark.gpu
@pytest.mark.parametrize("n,h,w,c,o,r,per", CASES)
def test_dx_alpha_in_tiles_of_128_rows(knob, n, h, w, c, o, r, per):
    knob("TWN_SMALL", 0)
    rng = np.random.default_rng(n + o)
    wt = (rng.standard_normal((o, c, r, r)) * 0.05 * np.exp(rng.standard_normal((o, 1, 1, 1)))).astype(np.float32)
    tw = api.twn_ternarize(to_dev_f32(wt), 0.7, groups=o // per, transposed=True)
    codes, _, alpha, _ = ot.ternarize(wt, 0.7, groups=o // per)
    dy = wl.bf16_round((rng.standard_normal((n, h, w, o)) * 1e-5).astype(np.float32))
    geo = (1, 1), (r // 2,) * 2, (1, 1)
    dx, _, _ = api.twn_conv2d_bwd_ste(to_dev_bf16(np.zeros((n, h, w, c), np.float32)), to_dev_bf16(dy), tw, *geo, need_dw=False)
    got, ref = to_host_f64(dx), oc.conv2d_bwd_data(dy, codes, alpha, (n, h, w, c), *geo)
    assert np.linalg.norm(got - ref) <= 2.0e-3 * np.linalg.norm(ref)
    assert rel_err(got, ref) <= BF16_TOL
