"""Which kernels the calls of the C ABI launch, on the CPU (see `launches`): dependent problems, the overrides, and the
ends of the ranges that the dispatch rules accept."""

import pytest

from launches import conv, gemm, launches


def kernels(answer):
    assert answer["rc"] == 0
    return [l["kernel"] for l in answer["launches"]]


# a block head of few tiles, one with unequal tiles, one with equal tiles of the larger kernel
HEADS = [(conv(1, 56, 56, 64, 128, 3, 2), conv(1, 56, 56, 64, 128, 1, 2)),
         (conv(1, 28, 28, 128, 64, 3, 2), conv(1, 28, 28, 128, 256, 1, 2)),
         (conv(64, 56, 56, 64, 128, 3, 2), conv(64, 56, 56, 64, 128, 1, 2))]


@pytest.mark.parametrize("first,second", HEADS)
def test_pair_shares_a_launch_only_if_independent(first, second):
    base = dict(fn="pair", d=first, d1=second)
    x, y0 = 1 << 40, 4 << 40
    independent = [base, dict(base, residual=True, residual1="residual"), dict(base, residual="X", residual1="Y1")]
    dependent = [dict(base, residual1="Y"), dict(base, residual="Y1"), dict(base, ptr={"Y1": y0}), dict(base, ptr={"Y1": y0 + 64}),
                 dict(base, ptr={"Y": x + 4096}), dict(base, ptr={"Y1": x})]
    answers = launches(independent + dependent)
    assert [len(kernels(a)) for a in answers] == [1] * len(independent) + [2] * len(dependent)


def test_an_override_has_one_value_until_it_is_reloaded():
    # set after the workspace query has asked for it: the launch, which asks at another place, still has it unset
    late = dict(fn="gemm", d=gemm(8192, 4096, 4096), env_late={"TWN_TILE": 4})
    set_, unset, late = launches([dict(late, env=late["env_late"], env_late={}), dict(late, env_late={}), late])
    assert kernels(set_) == ["gather_gemm_mfma_kernel"]
    assert kernels(late) == kernels(unset) == ["conv_stream_pc_kernel"]
