"""Which kernels the calls of the C ABI launch, on the CPU (see `launches`): dependent problems, the overrides, and the
ends of the ranges that the dispatch rules accept."""

import random

import pytest

from launches import F32, conv, gemm, launches


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


SMALL = [dict(fn="gemm", d=gemm(64, 1000, 512)), dict(fn="conv", d=conv(1, 14, 14, 256, 512, 3, 2)),
         dict(fn="bwd", d=conv(6, 38, 36, 32, 64, 3, 2), parts="dx"), dict(fn="bwd", d=conv(8, 12, 12, 128, 64, 3), parts="dw")]


@pytest.mark.parametrize("name,value,wanted", [
    ("TWN_STREAM", 0, ["gather_gemm_dma_kernel", "gather_gemm_dma_kernel", "gather_gemm_dma_batch_kernel", None]),
    ("TWN_BUFLOAD", 0, ["conv_stream_pc_kernel", "gather_gemm_dma_kernel", "gather_gemm_dma_batch_kernel", "weight_grad_patch_kernel"]),
    ("TWN_STREAM_PC", 0, ["conv_stream_kernel", "gather_gemm_dma_kernel", None, None]),
    ("TWN_STREAM_PC_STAGES", 4, ["conv_stream_pc_kernel", "gather_gemm_dma_kernel", None, None]),
    ("TWN_STREAM_KS", 2, ["conv_stream_pc_kernel", "gather_gemm_dma_kernel", None, None]),
    ("TWN_STREAM_OCC", 1, ["conv_stream_pc_kernel", "gather_gemm_dma_kernel", None, None]),
    ("TWN_WG_KS", 1, [None, None, None, "weight_grad_patch_kernel"]),
    ("TWN_WG_BLOCKS", 256, [None, None, None, "weight_grad_patch_kernel"]),
    ("TWN_WG_XCD", 0, [None, None, None, "weight_grad_patch_kernel"]),
    ("TWN_WG_ROWS_SPLITS", 4, [None, None, None, "weight_grad_patch_kernel"])])
def test_overrides_of_other_kernels_reach_small_problems(name, value, wanted):
    for kernel, a in zip(wanted, launches([dict(c, env={name: value}) for c in SMALL])):
        if kernel is not None:
            assert kernel in kernels(a)
            assert "conv_small_kernel" not in kernels(a) and "weight_grad_taps_kernel" not in kernels(a)
        if name == "TWN_BUFLOAD":           # the template argument BUF
            at = {"gather_gemm_dma_kernel": 7, "gather_gemm_dma_batch_kernel": 5, "weight_grad_patch_kernel": 1}
            assert all(l["args"][at[l["kernel"]]] == "false" for l in a["launches"] if l["kernel"] in at)


def test_pair_override_never_one_launch():
    for a in launches([dict(fn="pair", d=first, d1=second, env={"TWN_FWD_PAIR": 0}) for first, second in HEADS]):
        assert len(kernels(a)) == 2


@pytest.mark.parametrize("d", [conv(1, 1, 1, 1 << 15, 1 << 20, 1, groups=2),            # 2^32 words of repeated codes
                               conv(32, 512, 512, 4096, 64, 1, 2)])                    # 2^32 chunks of dX to clear
def test_preparation_of_dx_stays_below_the_largest_grid(d):
    (a,) = launches([dict(fn="bwd", d=d, parts="dx")])
    prep = [l for l in a["launches"] if l["kernel"] == "dx_prep_kernel"]
    assert a["rc"] == 0 and len(prep) > 1
    assert all(l["grid"][0] * l["block"][0] < 1 << 32 for l in prep)
    assert sum(l["grid"][0] for l in prep) >= 1 << 24


def _log(rng, lo, hi):
    return int(round(lo * (hi / lo) ** rng.random()))


def test_every_plan_has_a_build():
    rng = random.Random(3)
    f32 = [dict(fn="gemm", d=gemm(_log(rng, 1, 1 << 20), _log(rng, 1, 4096), _log(rng, 1, 20000), x=F32, y=F32)) for _ in range(400)]
    f32.append(dict(fn="gemm", d=gemm(1024, 1024, 1024, x=F32, y=F32)))
    dw = [dict(fn="bwd", d=conv(_log(rng, 1, 200), _log(rng, 7, 120), _log(rng, 7, 120), 8 * _log(rng, 1, 64), 8 * _log(rng, 8, 64),
                                rng.choice([2, 3, 5, 7]), dil=rng.choice([1, 1, 2])), parts="dw") for _ in range(400)]
    dw = [c for c in dw if c["d"]["H"] * c["d"]["W"] * c["d"]["N"] < 1 << 20]
    builds = set()
    for a in launches(f32 + dw):
        builds.update((k, tuple(l["args"][:2])) for k, l in zip(kernels(a), a["launches"]))
    assert {b[1] for b in builds if b[0] == "gather_gemm_f64_kernel"} == {
        ("1", "1"), ("1", "2"), ("1", "4"), ("1", "8"), ("1", "16"), ("2", "1"), ("2", "2"), ("2", "4"), ("4", "1"), ("4", "2")}
    assert {b[1] for b in builds if b[0] == "weight_grad_taps_kernel"} == {("3", "4"), ("4", "3")}
