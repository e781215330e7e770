"""Which kernels the calls of the C ABI launch, on the CPU (see `launches`): dependent problems, the overrides, the
ends of the ranges that the dispatch rules accept, and whether the GPU tests of a path have shapes that take it."""

import random
import re

import pytest

import test_gpu_conv as shapes
import test_gpu_dx_alpha as alpha_shapes
import test_gpu_filter_pad as pad_shapes
import test_gpu_wide_tiles as wide_shapes
from launches import BF16, F32, conv, gemm, launches


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
    ("TWN_STREAM_KS", 2, ["conv_stream_kernel", "gather_gemm_dma_kernel", None, None]),
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


def test_tiles_of_sixteen_pixels_fit_one_round():
    """The workgroups of a launch, empty ones of smaller problems among them, are at most 256: a CU holds one."""
    rng = random.Random(5)
    calls = [dict(fn="bwd", parts="dx", d=conv(13, 11, 9, 96, 512, 2, 2, 1))]
    calls += [dict(fn="bwd", parts="dx", d=conv(rng.randint(1, 16), rng.randint(3, 16), rng.randint(3, 16), 8 * rng.randint(1, 32),
                                                8 * rng.randint(1, 64), rng.choice([2, 3, 5]), 2)) for _ in range(300)]
    small = [l for a in launches(calls) for l in a["launches"] if l["kernel"] == "conv_small_kernel" and l["args"][6] == "true"]
    assert len(small) >= 50 and any(l["grid"][1] > 1 for l in small)
    assert all(l["grid"][0] * l["grid"][1] <= 256 for l in small)


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


def _conv_case(case, **kw):
    n, h, w, c, o, r, s, st, pd, dl = case
    return dict(conv(n, h, w, c, o, r, groups=kw.pop("groups", 1), **kw), S=s, stride_h=st[0], stride_w=st[1], pad_h=pd[0],
                pad_w=pd[1], dil_h=dl[0], dil_w=dl[1])


@pytest.mark.parametrize("y", [F32, BF16])
def test_split_k_tests_split(y):
    calls = [dict(fn="gemm", d=gemm(m, n, k, y=y), env={"TWN_SMALL": small}) for m, n, k, small in shapes.SPLITK_GEMM_CASES]
    assert all("splitk_finish_kernel" in kernels(a) for a in launches(calls))
    ds = [(conv(n, h, w, c, o, 3, groups=g, y=y), small) for n, h, w, c, o, g, small in shapes.SPLITK_CONV_CASES]
    fwd = launches([dict(fn="conv", d=d, env={"TWN_SMALL": small}) for d, small in ds])
    dx = launches([dict(fn="bwd", d=d, parts="dx", env={"TWN_SMALL": small}) for d, small in ds])
    assert ["splitk_finish_kernel" in kernels(a) for a in fwd] == [True, False, False, True, False]
    assert ["splitk_finish_kernel" in kernels(a) for a in dx] == [False, True, True, False, True]


def test_float32_split_k_tests_split():
    for split in (1, 0):
        env = {"TWN_F32_SPLITK": split}
        got = launches([dict(fn="gemm", d=gemm(m, n, k, x=F32, y=F32), env=env) for m, n, k in shapes.F32_SPLIT_CASES])
        got += launches([dict(fn="conv", d=conv(*xs, ws[0], ws[2], pad=pad, x=F32, y=F32), env=env) for xs, ws, pad in shapes.F32_CONV_CASES])
        cut = [m * n < 1 << 13 and k > 8192 for m, n, k in shapes.F32_SPLIT_CASES] + [False, True]
        assert ["fp32_splitk_finish_kernel" in kernels(a) for a in got] == [c and split == 1 for c in cut]


def test_pair_tests_run_one_launch_of_each_kernel():
    heads = [(conv(*xs, o0, 3, 2), conv(*xs, o1, 1, 2)) for xs, o0, o1 in shapes.PAIR_CASES]
    for small, one, wanted in ((1, 2, [["conv_small_kernel"]] * 4), (0, 2, [["gather_gemm_dma_batch_kernel"]] * 3 + [None]),
                               (1, 0, [["conv_small_kernel"] * 2] * 4), (0, 0, [None] * 4)):
        env = {"TWN_SMALL": small, "TWN_FWD_PAIR": one}
        for a, w in zip(launches([dict(fn="pair", d=d, d1=d1, env=env) for d, d1 in heads]), wanted):
            assert kernels(a) == w if w else len(kernels(a)) == 2 and "conv_small_kernel" not in kernels(a)


def test_residue_class_tests_run_one_launch_and_one_each():
    calls = [dict(fn="bwd", parts="dx", d=_conv_case(case + ((1, 1),), y=F32, groups=case[4] if per_filter else 1))
             for case in shapes.STRIDED_DX_CASES for per_filter in (0, 1)]
    for small, kernel in ((1, "conv_small_kernel"), (0, "gather_gemm_dma_batch_kernel")):
        env = {"TWN_DX_CLASS_MIN_PIXELS": 0, "TWN_SMALL": small}
        one = [kernels(a) for a in launches([dict(c, env=env) for c in calls])]
        each = [kernels(a) for a in launches([dict(c, env=dict(env, TWN_DX_CLASS_BATCH=0)) for c in calls])]
        assert all(k[0] == "dx_prep_kernel" and len(k) == 2 for k in one)
        several = [i for i, k in enumerate(each) if len(k) > 2]
        assert len(several) == 16 and all(one[i][1] == kernel for i in several)         # the 1x1 layer has one class


def test_weight_gradient_and_pointer_load_tests_take_the_general_kernels():
    for ks in (1, 2):
        calls = [dict(fn="bwd", parts="dw", d=_conv_case((4 * shapes.CONV_CASES[ci][0],) + shapes.CONV_CASES[ci][1:]),
                      env={"TWN_WG_KS": ks}) for ci in (1, 2, 4, 7)]
        for a in launches(calls):
            (patch,) = [l for l in a["launches"] if l["kernel"] == "weight_grad_patch_kernel"]
            assert patch["args"][3] == str(ks)
    env = {"TWN_BUFLOAD": 0}
    calls = [dict(fn="gemm", d=gemm(520, 300, 448, y=F32), env=env)]
    for ci in (1, 2):
        calls += [dict(fn="conv", d=_conv_case(shapes.CONV_CASES[ci], y=F32), env=env),
                  dict(fn="bwd", d=_conv_case(shapes.CONV_CASES[ci], y=F32), parts="dx dw", env=env)]
    buf = {"gather_gemm_dma_kernel": 7, "gather_gemm_dma_batch_kernel": 5, "weight_grad_patch_kernel": 1}
    for a in launches(calls):
        loads = [l["args"][buf[l["kernel"]]] for l in a["launches"] if l["kernel"] in buf]
        assert loads and set(loads) == {"false"}
        assert not {"conv_small_kernel", "weight_grad_taps_kernel"} & set(kernels(a))


def _up(n, to):
    return (n + to - 1) // to * to


def _partials_end(d, found):
    """Last byte of the workspace that the partial sums of a backward call reach, from the grids of its launches."""
    n, c, o, r, s = (d[f] for f in "NCORS")
    p, q = ((d[a] + 2 * d["pad_" + b] - d["dil_" + b] * (d[f] - 1) - 1) // d["stride_" + b] + 1 for a, b, f in ("HhR", "WwS"))
    by = {l["kernel"]: l["grid"] for l in found}
    end = offset = 0
    if "filter_pad_kernel" in by:
        assert o % 8 != 0
        o = _up(o, 8)
        offset = _up(n * p * q * o * 2, 256) + _up(4 * c * 8 * _up(r * s * o, 128) // 128, 256) + _up(4 * o, 256)
    (kernel,) = [k for k in by if re.fullmatch("(first_)?weight_grad(_patch|_taps)?_kernel", k)] or [None]
    x, y = by.get(kernel, (0, 0))[:2]
    if kernel is None:
        pass                                # the bias gradient alone
    elif kernel == "first_weight_grad_kernel":
        end = offset + x * o * r * _up(s, 4) * 4 * 4
    elif kernel == "weight_grad_taps_kernel":
        ranges, rest = divmod(x, _up(o, 64) // 64 * (_up(c, 32) // 32) * (_up(r * s, 9) // 9))
        assert rest == 0
        end = offset + ranges * o * c * r * s * 4 if ranges > 1 else 0
    elif "pad_c4_kernel" in by:             # the copy of X, then the partial tiles
        sp = _up(s, 2)
        offset += _up(n * (d["H"] + 2 * d["pad_h"]) * (d["W"] + 2 * d["pad_w"] + sp - s) * 8, 256)
        end = offset + y * o * r * sp * 4 * 4
    elif kernel == "weight_grad_kernel" or y > 1:
        end = offset + y * o * c * r * s * 4
    if "bias_grad_final_kernel" in by:
        where = offset if "pad_c4_kernel" in by and "filter_pad_kernel" not in by else 0
        end = max(end, where + by["bias_grad_kernel"][1] * d["O"] * 4)
    return end


def test_partial_sums_of_the_weight_gradient_fit_the_workspace():
    """The workspace query and the launch have to have the same kernel and ranges in mind, with and without padded filters."""
    rng = random.Random(7)
    calls = []
    while len(calls) < 3000:
        r, dil = rng.choice([1, 2, 3, 3, 3, 5, 7]), rng.choice([1, 1, 1, 2])
        c = rng.choice([3, 8 * _log(rng, 1, 80), 8 * _log(rng, 1, 80), _log(rng, 1, 600)])
        d = conv(_log(rng, 1, 64), _log(rng, 1, 120), _log(rng, 1, 120), c, rng.choice([_log(rng, 1, 600), 8 * _log(rng, 1, 80)]), r,
                 rng.choice([1, 1, 1, 2]), dil=dil, groups=1, pad=rng.choice([0, r // 2 * dil, dil * (r - 1)]))
        if min(d["H"], d["W"]) + 2 * d["pad_h"] > dil * (r - 1) and d["N"] * d["H"] * d["W"] < 1 << 19:
            calls.append(dict(fn="bwd", d=d, parts="dw db"))
    # around the limits of the kernel for several taps: 65536 pixels, 8192 filters x channels
    calls += [dict(fn="bwd", d=conv(64, 38, 38, 512, 84, 3), parts="dw"), dict(fn="bwd", d=conv(64, 40, 40, 16, 10, 3), parts="dw"),
              dict(fn="bwd", d=conv(36, 93, 92, 64, 250, 2), parts="dw"), dict(fn="bwd", d=conv(4, 128, 128, 24, 10, 3), parts="dw")]
    routes, over = {}, []
    for call, a in zip(calls, launches(calls)):
        ks = kernels(a)
        padded = "filter_pad_kernel" in ks
        for k in ks:
            routes[k, padded] = routes.get((k, padded), 0) + 1
        end = _partials_end(call["d"], a["launches"])
        if end > a["need"]:
            over.append((call["d"], a["need"], end))
    assert not over, (len(over), over[:4])
    wanted = ["weight_grad_patch_kernel", "weight_grad_taps_kernel", "weight_grad_kernel", "first_weight_grad_kernel", "pad_c4_kernel"]
    assert all(routes.get((k, padded), 0) >= 20 for k in wanted for padded in (False, True)), routes


def test_padded_several_tap_tests_take_the_kernel_for_several_taps():
    calls = [dict(fn="bwd", parts="dw", d=conv(n, h, w, c, o, r, pad=pad)) for n, h, w, c, o, r, pad in pad_shapes.TAPS_CASES]
    answers = launches(calls)
    assert all({"filter_pad_kernel", "weight_grad_taps_kernel"} <= set(kernels(a)) for a in answers)
    assert [kernels(a)[-1] == "weight_grad_sum_kernel" for a in answers] == [True, True, False, False, False]


def test_first_layers_run_with_the_workspace_of_the_general_kernel():
    """The kernel for three-channel layers may want more than the general one, which the call then falls back to."""
    ds = [conv(3, 3, 2, 3, 512, 3, 2), conv(15, 3, 20, 3, 88, 1), conv(40, 12, 2, 3, 136, 3), conv(22, 12, 4, 3, 384, 1)]
    calls = [dict(fn="bwd", d=d, parts=parts) for d in ds for parts in ("dw", "dw db", "db")]
    least = [a["need"] for a in launches([dict(c, env={"TWN_FIRST": 0}) for c in calls])]
    full = launches(calls)
    assert all(a["need"] > n for a, n in zip(full, least))
    for call, n, f, a in zip(calls, least, full, launches([dict(c, ws=n) for c, n in zip(calls, least)])):
        assert kernels(a) and _partials_end(call["d"], a["launches"]) <= n
        if "dw" in call["parts"]:
            assert "first_weight_grad_kernel" in kernels(f) and "weight_grad_patch_kernel" in kernels(a)


# 128 x 128 blocks: 392 and 512 (the wider tiles leave the busiest CU no more of them), 392 again with a short K
WIDE = [conv(16, 56, 56, 128, 128, 3), conv(32, 32, 32, 256, 256, 3), conv(16, 56, 56, 512, 128, 1)]


# the kernel that answers each override where the three shapes would take wide tiles; K groups are its last template argument
@pytest.mark.parametrize("name,value,kernel,groups", [
    ("TWN_STREAM_PC_STAGES", 3, "conv_stream_kernel", "1"), ("TWN_STREAM_PC_STAGES", 4, "conv_stream_pc_kernel", None),
    ("TWN_STREAM_PC", 0, "conv_stream_kernel", "1"), ("TWN_STREAM_PC", 4, "conv_stream_pc_kernel", None),
    ("TWN_STREAM_KS", 1, "conv_stream_pc_kernel", None), ("TWN_STREAM_KS", 2, "conv_stream_kernel", "2"),
    ("TWN_STREAM_OCC", 1, "conv_stream_pc_kernel", None), ("TWN_STREAM", 0, "gather_gemm_dma_kernel", None),
    ("TWN_BUFLOAD", 0, "conv_stream_pc_kernel", None)])
def test_overrides_of_the_persistent_kernels_run_where_wide_tiles_would(name, value, kernel, groups):
    plain = launches([dict(fn="conv", d=d) for d in WIDE])
    assert [kernels(a) + a["launches"][0]["args"][:2] for a in plain] == [["conv_stream_pc_kernel", m, n] for m, n in
                                                                          (("256", "128"), ("128", "256"), ("128", "128"))]
    for a in launches([dict(fn="conv", d=d, env={name: value}) for d in WIDE]):
        assert kernels(a) == [kernel]
        assert groups is None or a["launches"][0]["args"][-1] == groups


def test_load_waves_leave_taps_that_span_their_marks():
    """Their mark of a row outside the image, 2^31, stays outside while the taps span less than 2^30 rows and columns."""
    calls = [dict(fn="conv", d=dict(conv(1, 1, 1, 64, 128, 3), pad_h=d, dil_h=d), env={"TWN_SMALL": 0, "TWN_TILE": 14}) for d in (1 << 28, 1 << 29)]
    assert [kernels(a) for a in launches(calls)] == [["conv_stream_pc_kernel"], ["gather_gemm_dma_kernel"]]


def test_k_groups_that_are_asked_for():
    """TWN_STREAM_KS on every tile that has K groups, also where load waves are the rule; TWN_STREAM_PC asks for those all the same."""
    d = conv(16, 14, 14, 512, 512, 3)
    for tile, ks in ((14, 2), (14, 4), (15, 2), (16, 2)):
        (a,) = launches([dict(fn="conv", d=d, env={"TWN_TILE": tile, "TWN_STREAM_KS": ks})])
        assert kernels(a) == ["conv_stream_kernel"] and a["launches"][0]["args"][-1] == str(ks)
        (a,) = launches([dict(fn="conv", d=d, env={"TWN_TILE": tile, "TWN_STREAM_KS": ks, "TWN_STREAM_PC": 4})])
        assert kernels(a) == ["conv_stream_pc_kernel"]


def test_short_float32_kernel_leaves_paddings_that_pass_its_sentinel():
    """Elements behind K carry a row offset of -2^28, which a padding of 2^28 rows would bring back into the image."""
    d = dict(conv(1, 4, 1, 1, 1, 3, x=F32, y=F32, pad=0), S=1)
    answers = launches([dict(fn="conv", d=dict(d, pad_h=p)) for p in (1 << 16, 1 << 24, 1 << 28)])
    assert [kernels(a) for a in answers] == [["gather_gemm_f64_short_kernel"], ["gather_gemm_f64_kernel"], ["gather_gemm_f64_kernel"]]


def test_wide_tile_tests_walk_to_a_second_tile():
    for tile, rows, cols in ((17, 128, 256), (18, 256, 128)):
        answers = launches([dict(fn="conv", d=conv(n, h, w, c, o, 3, groups=g), env={"TWN_TILE": tile})
                            for n, h, w, c, o, g in wide_shapes.CASES])
        walks = []
        for (n, h, w, c, o, g), a in zip(wide_shapes.CASES, answers):
            assert kernels(a) == ["conv_stream_pc_kernel"] and a["launches"][0]["args"][:2] == [str(rows), str(cols)]
            walks.append(-(-n * h * w // rows) * -(-o // cols) > a["launches"][0]["grid"][0])
        assert walks == [False] * (len(walks) - 1) + [True]


def _dx_alpha(d, small=1):
    """Whether the alphas of backward-data stay with the codes (the ALPHA builds), per call."""
    return [[(l["kernel"], l["args"][-1]) for l in a["launches"] if l["kernel"] != "dx_prep_kernel"][0]
            for a in launches([dict(fn="bwd", parts="dx", d=x, env={"TWN_SMALL": small}) for x in d])]


def test_exact_alpha_tests_take_the_alphas_with_the_codes():
    for small, wanted in ((1, [("conv_small_kernel", "true")] * 6),
                          (0, [("conv_stream_pc_kernel", "true")] * 2 + [("gather_gemm_dma_batch_kernel", "true")] * 2)):
        cases = [c[1:] for c in alpha_shapes.EXACT_CASES if c[0] == small]
        assert _dx_alpha([conv(n, h, w, c, o, r, s, pad, groups=o) for n, h, w, c, o, r, s, pad in cases], small) == wanted

    large = _dx_alpha([conv(n, h, w, c, o, r, s, pad, dil, o // per) for n, h, w, c, o, r, s, pad, dil, per in alpha_shapes.LARGE_CASES], 0)
    assert large[:4] == [("conv_stream_pc_kernel", "true")] * 4 and large[6] == ("conv_stream_pc_kernel", "true")


def test_alphas_stay_with_the_codes_while_the_third_product_costs_less_than_scaling():
    layers = [(conv(64, 14, 14, 256, 256, 3, groups=256), True), (conv(64, 14, 14, 512, 512, 3, groups=512), False),
              (conv(64, 7, 7, 512, 512, 3, groups=512), False), (conv(64, 7, 7, 512, 256, 3, groups=256), True),
              (conv(64, 40, 40, 256, 256, 3, groups=256), False), (conv(64, 40, 40, 256, 256, 1, groups=256), True),
              (conv(64, 28, 28, 256, 512, 3, 2, groups=512), True), (conv(64, 28, 28, 512, 512, 3, 2, groups=512), False)]
    assert [a == "true" for _, a in _dx_alpha([d for d, _ in layers])] == [inside for _, inside in layers]
