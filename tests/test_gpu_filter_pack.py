"""One threshold and scale per filter in one launch: the last filter block, filters whose length is no multiple of 4, 16 or
64 values, the longest filter the launch takes and the first beyond it, taps that straddle words; codes bit for bit."""

import pytest

from paper_1605_04711_amd import workloads as wl
from test_gpu_ternarize import check_against_oracle, pytestmark  # noqa: F401


@pytest.mark.parametrize("transposed", [True, False])
@pytest.mark.parametrize("shape", [
    (512, 9216), (512, 9217), (31, 512, 3, 3), (33, 4609),     # the longest filters and the first beyond, partial blocks
    (33, 255), (31, 66), (2, 1), (47, 3),         # partial blocks of matrices, odd lengths
    (64, 3, 7, 7), (48, 5, 3, 3), (32, 1, 5, 5),  # taps whose channels are no whole dword
    (20, 16, 3, 3), (16, 6, 1, 5)])               # filters no multiple of 16: with the transposed copy the general path
def test_filter_pack(shape, transposed):
    w = wl.normal(13, shape[0] + shape[1], shape, std=0.05)
    w.reshape(-1)[:: 7] = 0.0
    check_against_oracle(w, 0.7, groups=shape[0], transposed=transposed)
