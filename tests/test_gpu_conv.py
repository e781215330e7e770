"""GPU parity of the forward block (Eq. 2; Alg. 1 step 8) and of the
straight-through backward (Alg. 1 steps 9-10) against the direct-loop oracle.
Bar: max relative error <= 2e-2 on bf16-MFMA paths, <= 1e-5 on float32 paths,
with err = max |y - ref| / max(|ref|, 1e-2 rms(ref)).  Weights go through the
whole pipeline: twn_ternarize on the GPU, oracle ternarizer on the CPU."""

import os

import numpy as np
import pytest
import torch

from oracle import conv as oc
from oracle import ternarize as ot
from paper_1605_04711_amd import api
from paper_1605_04711_amd import workloads as wl
from parity import BF16_TOL, FP32_TOL, rel_err, to_dev_bf16, to_dev_f32, to_host_f64

pytestmark = pytest.mark.gpu

F = 0.7


def make_layer(seed, x_shape, w_shape, bf16=True, groups=1, transposed=False):
    g = np.random.default_rng(seed)
    x = g.standard_normal(x_shape).astype(np.float32)
    if bf16:
        x = wl.bf16_round(x)
    fan_in = int(np.prod(w_shape[1:]))
    w = (g.standard_normal(w_shape) * np.sqrt(2.0 / fan_in)).astype(np.float32)
    tw = api.twn_ternarize(to_dev_f32(w), F, groups=groups, transposed=transposed)
    w4 = w if w.ndim == 4 else w.reshape(w.shape[0], w.shape[1], 1, 1)
    codes, delta, alpha, nnz = ot.ternarize(w4, F, groups=groups)
    return x, w, tw, codes, alpha


GEMM_CASES = [(300, 200, 320), (257, 130, 64), (1, 10, 1024), (128, 1000, 512), (64, 40, 100), (513, 257, 136)]


@pytest.mark.usefixtures("both_dispatches")
@pytest.mark.parametrize("m,n,k", GEMM_CASES)
def test_gemm_fwd_bf16(m, n, k):
    x, w, tw, codes, alpha = make_layer(m + n + k, (m, k), (n, k))
    y = api.twn_gemm_fwd(to_dev_bf16(x), tw, y_dtype=torch.float32)
    yb = api.twn_gemm_fwd(to_dev_bf16(x), tw, y_dtype=torch.bfloat16)
    ref = oc.gemm_fwd(x, codes.reshape(n, k), alpha)
    assert rel_err(to_host_f64(y), ref) <= 1e-4          # fp32 accumulation of exact bf16 products
    assert rel_err(to_host_f64(yb), ref) <= BF16_TOL


@pytest.mark.parametrize("tile", [1, 2, 3, 4, 5, 6])
def test_gemm_fwd_every_tile_shape(tile, knob):
    knob("TWN_TILE", str(tile))
    m, n, k = 520, 300, 448
    x, w, tw, codes, alpha = make_layer(tile, (m, k), (n, k))
    y = api.twn_gemm_fwd(to_dev_bf16(x), tw, y_dtype=torch.float32)
    ref = oc.gemm_fwd(x, codes.reshape(n, k), alpha)
    assert rel_err(to_host_f64(y), ref) <= 1e-4


DMA_TILES = [12, 14, 15, 16, 17, 24, 30]


@pytest.mark.parametrize("tile", DMA_TILES)
def test_every_direct_to_lds_tile_shape(tile, knob):
    # every instantiated tile of the direct-to-LDS kernel: a ragged GEMM and a padded, strided convolution
    knob("TWN_TILE", str(tile))
    m, n, k = 520, 300, 448
    x, w, tw, codes, alpha = make_layer(tile, (m, k), (n, k))
    y = api.twn_gemm_fwd(to_dev_bf16(x), tw, y_dtype=torch.float32)
    assert rel_err(to_host_f64(y), oc.gemm_fwd(x, codes.reshape(n, k), alpha)) <= 1e-4
    nb, h, w_, c, o, r, s, st, pd, dl = (3, 15, 13, 24, 72, 3, 3, (2, 1), (1, 2), (1, 1))
    x, w, tw, codes, alpha = make_layer(50 + tile, (nb, h, w_, c), (o, c, r, s))
    y = api.twn_conv2d_fwd(to_dev_bf16(x), tw, st, pd, dl, y_dtype=torch.float32)
    assert rel_err(to_host_f64(y), oc.conv2d_fwd(x, codes, alpha, st, pd, dl)) <= 1e-4


@pytest.mark.parametrize("tile", [30])
def test_pinned_accumulator_tiles(tile, knob):
    # the 256x256 tiles keep their 16 accumulator tiles per wave in hand-assigned registers: both load paths
    # (K and channel counts that are / are not multiples of 64), both epilogues, and backward-data
    knob("TWN_TILE", str(tile))
    for seed, (m, n, k) in enumerate([(520, 600, 448), (300, 257, 440), (1100, 512, 1024)]):
        x, w, tw, codes, alpha = make_layer(300 + seed, (m, k), (n, k))
        ref = oc.gemm_fwd(x, codes.reshape(n, k), alpha)
        y = api.twn_gemm_fwd(to_dev_bf16(x), tw, y_dtype=torch.float32)
        assert rel_err(to_host_f64(y), ref) <= 1e-4
        yb = api.twn_gemm_fwd(to_dev_bf16(x), tw)
        assert rel_err(to_host_f64(yb), ref) <= BF16_TOL
    m, n, k = 700, 320, 256
    x, w, tw, codes, alpha = make_layer(310, (m, k), (n, k), groups=n)
    g = np.random.default_rng(4)
    scale = g.uniform(0.5, 1.5, n).astype(np.float32)
    shift = g.standard_normal(n).astype(np.float32)
    res = wl.bf16_round(g.standard_normal((m, n)).astype(np.float32))
    y = api.twn_gemm_fwd(to_dev_bf16(x), tw, scale=to_dev_f32(scale), shift=to_dev_f32(shift),
                         residual=to_dev_bf16(res), relu=True)
    ref = oc.epilogue(oc.gemm_fwd(x, codes.reshape(n, k), alpha), scale, shift, res, relu=True)
    assert rel_err(to_host_f64(y), ref) <= BF16_TOL
    for seed, (nb, h, w_, c, o, r, s, st, pd, dl) in enumerate([
            (3, 17, 17, 64, 320, 3, 3, (1, 1), (1, 1), (1, 1)),
            (3, 15, 13, 24, 72, 3, 3, (2, 1), (1, 2), (1, 1))]):
        x, w, tw, codes, alpha = make_layer(320 + seed, (nb, h, w_, c), (o, c, r, s), transposed=True)
        ref = oc.conv2d_fwd(x, codes, alpha, st, pd, dl)
        y = api.twn_conv2d_fwd(to_dev_bf16(x), tw, st, pd, dl, y_dtype=torch.float32)
        assert rel_err(to_host_f64(y), ref) <= 1e-4
        yb = api.twn_conv2d_fwd(to_dev_bf16(x), tw, st, pd, dl)
        assert rel_err(to_host_f64(yb), ref) <= BF16_TOL
        dy = wl.bf16_round(g.standard_normal(ref.shape).astype(np.float32))
        dx, _, _ = api.twn_conv2d_bwd_ste(None, to_dev_bf16(dy), tw, st, pd, dl, need_dx=True, need_dw=False,
                                          x_shape=(nb, h, w_, c), dx_dtype=torch.float32)
        assert rel_err(to_host_f64(dx), oc.conv2d_bwd_data(dy, codes, alpha, (nb, h, w_, c), st, pd, dl)) <= 1e-4


STRIDE1_CASES = [
    # N  H   W   C    O    R  S  pad     dil      (stride 1, several taps, channels in whole 64-wide slabs)
    (3, 17, 17, 64, 128, 3, 3, (1, 1), (1, 1)),
    (5, 8, 8, 128, 72, 3, 3, (1, 1), (1, 1)),
    (2, 20, 33, 64, 64, 3, 3, (0, 2), (1, 1)),
    (1, 19, 19, 64, 48, 3, 3, (2, 2), (2, 2)),
    (2, 12, 12, 192, 136, 5, 5, (2, 2), (1, 1)),
    (3, 9, 30, 64, 256, 1, 3, (0, 1), (1, 1)),
]


@pytest.mark.usefixtures("both_dispatches")
@pytest.mark.parametrize("ci", range(len(STRIDE1_CASES)))
def test_stride1_multi_tap_layers_forward_and_backward_data(ci):
    n, h, w_, c, o, r, s, pd, dl = STRIDE1_CASES[ci]
    st = (1, 1)
    x, w, tw, codes, alpha = make_layer(600 + ci, (n, h, w_, c), (o, c, r, s), transposed=True)
    g = np.random.default_rng(ci)
    scale = g.uniform(0.5, 1.5, o).astype(np.float32)
    shift = g.standard_normal(o).astype(np.float32)
    y = api.twn_conv2d_fwd(to_dev_bf16(x), tw, st, pd, dl, y_dtype=torch.float32)
    ref = oc.conv2d_fwd(x, codes, alpha, st, pd, dl)
    assert rel_err(to_host_f64(y), ref) <= 1e-4
    res = wl.bf16_round(g.standard_normal(ref.shape).astype(np.float32))
    yb = api.twn_conv2d_fwd(to_dev_bf16(x), tw, st, pd, dl, scale=to_dev_f32(scale), shift=to_dev_f32(shift),
                            residual=to_dev_bf16(res), relu=True)
    assert rel_err(to_host_f64(yb), oc.epilogue(ref, scale, shift, res, relu=True)) <= BF16_TOL
    if o % 64 == 0:
        dy = wl.bf16_round(g.standard_normal(ref.shape).astype(np.float32))
        dx, _, _ = api.twn_conv2d_bwd_ste(None, to_dev_bf16(dy), tw, st, pd, dl, need_dx=True, need_dw=False,
                                          x_shape=(n, h, w_, c), dx_dtype=torch.float32)
        assert rel_err(to_host_f64(dx), oc.conv2d_bwd_data(dy, codes, alpha, (n, h, w_, c), st, pd, dl)) <= 1e-4


@pytest.mark.usefixtures("both_dispatches")
def test_gemm_epilogue_groups_and_strides():
    m, n, k = 200, 96, 256
    x, w, tw, codes, alpha = make_layer(11, (m, k), (n, k), groups=n)
    g = np.random.default_rng(2)
    scale = g.uniform(0.5, 1.5, n).astype(np.float32)
    shift = g.standard_normal(n).astype(np.float32)
    res = wl.bf16_round(g.standard_normal((m, n)).astype(np.float32))
    xpad = torch.zeros((m, k + 8), dtype=torch.bfloat16, device="cuda")
    xpad[:, :k] = to_dev_bf16(x)
    y = api.twn_gemm_fwd(xpad[:, :k], tw, scale=to_dev_f32(scale), shift=to_dev_f32(shift),
                         residual=to_dev_bf16(res), relu=True)
    ref = oc.epilogue(oc.gemm_fwd(x, codes.reshape(n, k), alpha), scale, shift, res, relu=True)
    assert rel_err(to_host_f64(y), ref) <= BF16_TOL
    assert float(to_host_f64(y).min()) >= 0.0


CONV_CASES = [
    # N  H   W   C   O   R  S  stride  pad     dil
    (2, 13, 11, 16, 40, 3, 3, (1, 1), (1, 1), (1, 1)),
    (3, 17, 17, 64, 128, 3, 3, (1, 1), (1, 1), (1, 1)),
    (2, 14, 14, 128, 256, 3, 3, (2, 2), (1, 1), (1, 1)),
    (1, 19, 19, 32, 48, 3, 3, (1, 1), (6, 6), (6, 6)),
    (2, 12, 12, 32, 64, 5, 5, (1, 1), (0, 0), (1, 1)),
    (2, 31, 29, 3, 64, 7, 7, (2, 2), (3, 3), (1, 1)),
    (2, 16, 16, 3, 128, 3, 3, (1, 1), (1, 1), (1, 1)),
    (2, 14, 14, 64, 128, 1, 1, (2, 2), (0, 0), (1, 1)),
    (5, 9, 9, 24, 10, 1, 1, (1, 1), (0, 0), (1, 1)),
    (1, 10, 12, 8, 8, 3, 2, (2, 1), (1, 0), (1, 2)),
]


VARIANTS = [api.TWN_VAR_BF16_ALPHA_LDS, api.TWN_VAR_I8_STORED_POSTSCALE]


@pytest.mark.parametrize("variant", VARIANTS)
@pytest.mark.parametrize("m,n,k", [(300, 200, 320), (513, 257, 136), (64, 40, 104), (1, 10, 1024)])
def test_gemm_fwd_comparison_variants(variant, m, n, k):
    # alpha-at-expansion rounds alpha to bf16 (one more 2^-9 relative error); int8-stored is exact like the product path
    x, w, tw, codes, alpha = make_layer(m + n + k + variant, (m, k), (n, k), groups=(n if m == 300 else 1))
    y = api.twn_gemm_fwd(to_dev_bf16(x), tw, y_dtype=torch.float32, variant=variant)
    ref = oc.gemm_fwd(x, codes.reshape(n, k), alpha)
    assert rel_err(to_host_f64(y), ref) <= (BF16_TOL if variant == api.TWN_VAR_BF16_ALPHA_LDS else 1e-4)
    yb = api.twn_gemm_fwd(to_dev_bf16(x), tw, variant=variant)
    assert rel_err(to_host_f64(yb), ref) <= BF16_TOL


def test_int8_codes_match_oracle_codes():
    n, k = 70, 200
    x, w, tw, codes, alpha = make_layer(77, (4, k), (n, k))
    i8 = tw.weights_for(api.TWN_VAR_I8_STORED_POSTSCALE).cpu().numpy()
    assert i8.dtype == np.int8 and np.array_equal(i8, codes.reshape(n, k))


@pytest.mark.parametrize("variant", VARIANTS)
@pytest.mark.parametrize("ci", [0, 2, 3, 5, 8, 9])
def test_conv2d_fwd_comparison_variants(variant, ci):
    n, h, w_, c, o, r, s, st, pd, dl = CONV_CASES[ci]
    x, w, tw, codes, alpha = make_layer(300 + ci, (n, h, w_, c), (o, c, r, s))
    if variant == api.TWN_VAR_I8_STORED_POSTSCALE and (r * s * c) % 8:
        with pytest.raises(api.TwnError):      # int8 rows must be 8-byte multiples
            api.twn_conv2d_fwd(to_dev_bf16(x), tw, st, pd, dl, variant=variant)
        return
    g = np.random.default_rng(ci)
    scale = g.uniform(0.5, 1.5, o).astype(np.float32)
    # alpha-at-expansion carries bf16(alpha)'s 2^-9 relative error through the whole sum; a shift that cancels
    # the sum would turn that into an unbounded relative error of the result, so that variant is checked unshifted
    shift = g.standard_normal(o).astype(np.float32) if variant == api.TWN_VAR_I8_STORED_POSTSCALE else None
    y = api.twn_conv2d_fwd(to_dev_bf16(x), tw, st, pd, dl, variant=variant, scale=to_dev_f32(scale),
                           shift=None if shift is None else to_dev_f32(shift), relu=True)
    ref = oc.epilogue(oc.conv2d_fwd(x, codes, alpha, st, pd, dl), scale, shift, None, relu=True)
    assert rel_err(to_host_f64(y), ref) <= BF16_TOL


def test_conv2d_bwd_data_alpha_at_expansion_variant():
    n, h, w_, c, o, r, s, st, pd, dl = CONV_CASES[1]
    x, w, tw, codes, alpha = make_layer(401, (n, h, w_, c), (o, c, r, s), transposed=True)
    yshape = api.conv_out_shape((n, h, w_, c), tw, st, pd, dl)
    dy = wl.bf16_round(np.random.default_rng(5).standard_normal(yshape).astype(np.float32))
    dx, _, _ = api.twn_conv2d_bwd_ste(None, to_dev_bf16(dy), tw, st, pd, dl, need_dx=True, need_dw=False,
                                      x_shape=(n, h, w_, c), variant=api.TWN_VAR_BF16_ALPHA_LDS)
    ref = oc.conv2d_bwd_data(dy, codes, alpha, (n, h, w_, c), st, pd, dl)
    assert rel_err(to_host_f64(dx), ref) <= BF16_TOL


@pytest.mark.usefixtures("both_dispatches")
@pytest.mark.parametrize("ci", range(len(CONV_CASES)))
def test_conv2d_fwd_bf16(ci):
    n, h, w_, c, o, r, s, st, pd, dl = CONV_CASES[ci]
    x, w, tw, codes, alpha = make_layer(100 + ci, (n, h, w_, c), (o, c, r, s))
    y = api.twn_conv2d_fwd(to_dev_bf16(x), tw, st, pd, dl, y_dtype=torch.float32)
    ref = oc.conv2d_fwd(x, codes, alpha, st, pd, dl)
    assert tuple(y.shape) == ref.shape
    assert rel_err(to_host_f64(y), ref) <= 1e-4
    yb = api.twn_conv2d_fwd(to_dev_bf16(x), tw, st, pd, dl)
    assert rel_err(to_host_f64(yb), ref) <= BF16_TOL


@pytest.mark.usefixtures("both_dispatches")
def test_conv2d_fwd_fused_block_tail():
    n, h, w_, c, o, r, s, st, pd, dl = CONV_CASES[1]
    x, w, tw, codes, alpha = make_layer(7, (n, h, w_, c), (o, c, r, s), groups=o)
    g = np.random.default_rng(3)
    scale = g.uniform(0.5, 1.5, o).astype(np.float32)
    shift = g.standard_normal(o).astype(np.float32)
    ref0 = oc.conv2d_fwd(x, codes, alpha, st, pd, dl)
    res = wl.bf16_round(g.standard_normal(ref0.shape).astype(np.float32))
    y = api.twn_conv2d_fwd(to_dev_bf16(x), tw, st, pd, dl, scale=to_dev_f32(scale), shift=to_dev_f32(shift),
                           residual=to_dev_bf16(res), relu=True)
    assert rel_err(to_host_f64(y), oc.epilogue(ref0, scale, shift, res, relu=True)) <= BF16_TOL


PAIR_CASES = [   # x shape, O of the 3x3 / stride-2 convolution, O of the 1x1 / stride-2 shortcut (few tiles: one launch for all)
    ((4, 28, 28, 64), 128, 128),       # same tile of the large-problem kernels: one launch; 784 pixels leave a ragged last tile
    ((3, 14, 14, 128), 256, 256),
    ((2, 13, 9, 72), 136, 136),        # odd image, C % 64 != 0 (per-lane pointer loads), ragged channel tile
    ((2, 16, 16, 64), 64, 128),        # different tile shapes: one launch after the other
]


@pytest.mark.usefixtures("both_dispatches")
@pytest.mark.parametrize("one_launch", [2, 0])
@pytest.mark.parametrize("ci", range(len(PAIR_CASES)))
def test_conv2d_fwd_pair(ci, one_launch, knob):
    """A residual block's first convolution and its projection shortcut over the same input (Sec. 3.1's ResNet-18
    has three such block heads), each against the oracle and against its own twn_conv2d_fwd call."""
    knob("TWN_FWD_PAIR", str(one_launch))
    xs, o0, o1 = PAIR_CASES[ci]
    c = xs[3]
    x, _, tw0, codes0, alpha0 = make_layer(700 + ci, xs, (o0, c, 3, 3), groups=o0 if ci == 1 else 1)
    _, _, tw1, codes1, alpha1 = make_layer(720 + ci, xs, (o1, c, 1, 1))
    g = np.random.default_rng(40 + ci)
    sc0, sf0 = g.uniform(0.5, 1.5, o0).astype(np.float32), g.standard_normal(o0).astype(np.float32)
    sc1, sf1 = g.uniform(0.5, 1.5, o1).astype(np.float32), g.standard_normal(o1).astype(np.float32)
    geos = (((2, 2), (1, 1), (1, 1)), ((2, 2), (0, 0), (1, 1)))
    xd = to_dev_bf16(x)
    y0, y1 = api.twn_conv2d_fwd_pair(xd, (tw0, tw1), geos, scales=(to_dev_f32(sc0), to_dev_f32(sc1)),
                                     shifts=(to_dev_f32(sf0), to_dev_f32(sf1)), relus=(True, False))
    ref0 = oc.epilogue(oc.conv2d_fwd(x, codes0, alpha0, *geos[0]), sc0, sf0, None, relu=True)
    ref1 = oc.epilogue(oc.conv2d_fwd(x, codes1, alpha1, *geos[1]), sc1, sf1, None, relu=False)
    assert tuple(y0.shape) == ref0.shape and tuple(y1.shape) == ref1.shape
    assert rel_err(to_host_f64(y0), ref0) <= BF16_TOL
    assert rel_err(to_host_f64(y1), ref1) <= BF16_TOL
    s0 = api.twn_conv2d_fwd(xd, tw0, *geos[0], scale=to_dev_f32(sc0), shift=to_dev_f32(sf0), relu=True)
    s1 = api.twn_conv2d_fwd(xd, tw1, *geos[1], scale=to_dev_f32(sc1), shift=to_dev_f32(sf1), relu=False)
    assert rel_err(to_host_f64(y0), to_host_f64(s0)) <= 1e-2      # a bf16 ulp: the K order may differ between kernels
    assert rel_err(to_host_f64(y1), to_host_f64(s1)) <= 1e-2


@pytest.mark.parametrize("batch", [8, 64])
def test_lenet_layers_fp32(batch):
    for li, layer in enumerate(wl.lenet5(batch)):
        x = wl.uniform01(0, wl.IDX_INPUT + li, layer.x_shape)
        w = wl.kaiming_weights(0, li, layer)
        tw = api.twn_ternarize(to_dev_f32(w), F)
        codes, delta, alpha, nnz = ot.ternarize(w, F)
        y = api.twn_conv2d_fwd(to_dev_f32(x), tw, (layer.stride,) * 2, (layer.pad,) * 2, (layer.dil,) * 2,
                               y_dtype=torch.float32, relu=True)
        ref = oc.epilogue(oc.conv2d_fwd(x, codes, alpha, (layer.stride,) * 2, (layer.pad,) * 2, (layer.dil,) * 2),
                          relu=True)
        assert rel_err(to_host_f64(y), ref) <= FP32_TOL, layer.name
    # the fully-connected layers through the GEMM entry point
    layer = wl.lenet5(batch)[2]
    x = wl.uniform01(0, 77, (batch, layer.C))
    w = wl.kaiming_weights(0, 2, layer)
    tw = api.twn_ternarize(to_dev_f32(w.reshape(layer.O, layer.C)), F)
    codes, delta, alpha, nnz = ot.ternarize(w, F)
    y = api.twn_gemm_fwd(to_dev_f32(x), tw, y_dtype=torch.float32)
    assert rel_err(to_host_f64(y), oc.gemm_fwd(x, codes.reshape(layer.O, layer.C), alpha)) <= FP32_TOL


F32_SPLIT_CASES = [   # M, N, K: float32 problems with few tiles: K shared out over the waves of a tile's workgroup, and beyond
    (64, 500, 800), (64, 10, 500), (200, 100, 1000), (33, 48, 130), (96, 130, 2000), (5, 7, 4000),
    (64, 10, 16400), (5, 7, 40003), (100, 64, 9001), (33, 40, 33007),       # 8192 over workgroups too (ragged last block)
]


@pytest.mark.parametrize("split", [1, 0])
@pytest.mark.parametrize("m,n,k", F32_SPLIT_CASES)
def test_gemm_fwd_fp32_split_k(m, n, k, split, knob):
    knob("TWN_F32_SPLITK", str(split))
    g = np.random.default_rng(m + n + k)
    x = g.uniform(-1.0, 1.0, (m, k)).astype(np.float32)
    w = (g.standard_normal((n, k)) * 0.05).astype(np.float32)
    tw = api.twn_ternarize(to_dev_f32(w), F)
    codes, delta, alpha, nnz = ot.ternarize(w.reshape(n, k, 1, 1), F)
    # no shift here: a float32 addition that cancels the sum would put its own rounding above the bound of this path
    y = api.twn_gemm_fwd(to_dev_f32(x), tw, y_dtype=torch.float32, relu=True)
    ref = oc.epilogue(oc.gemm_fwd(x, codes.reshape(n, k), alpha), relu=True)
    assert rel_err(to_host_f64(y), ref) <= FP32_TOL


F32_CONV_CASES = [((16, 20, 20, 32), (64, 32, 5, 5), 0),       # 4096 pixels x K = 800: four waves share K
                  ((1, 5, 5, 404), (20, 404, 5, 5), 2)]        # 25 pixels x K = 10100: K over the waves of several workgroups


@pytest.mark.parametrize("xs,ws,pad", F32_CONV_CASES)
def test_conv2d_fwd_fp32_shared_k(xs, ws, pad):
    x = wl.uniform01(0, 91, xs)
    g = np.random.default_rng(17)
    w = (g.standard_normal(ws) * 0.05).astype(np.float32)
    tw = api.twn_ternarize(to_dev_f32(w), F)
    codes, delta, alpha, nnz = ot.ternarize(w, F)
    y = api.twn_conv2d_fwd(to_dev_f32(x), tw, (1, 1), (pad, pad), (1, 1), y_dtype=torch.float32)
    assert rel_err(to_host_f64(y), oc.conv2d_fwd(x, codes, alpha, (1, 1), (pad, pad), (1, 1))) <= FP32_TOL


SPLITK_GEMM_CASES = [   # M, N, K, TWN_SMALL: bf16 products whose K is cut into ranges with a finishing launch
    (64, 64, 32768, 1), (33, 72, 16648, 1), (130, 40, 17000, 1),                     # by the rule: K above 16384
    (64, 1000, 1024, 0), (40, 72, 1160, 0), (200, 130, 2056, 0), (1, 10, 4096, 0)]   # with the few-tile kernel off
SPLITK_CONV_CASES = [   # N, H, W, C, O, alpha groups, TWN_SMALL (3x3): forward over 9 C, data gradient over 9 O (twice with groups)
    (1, 7, 7, 2048, 40, 1, 1), (2, 5, 6, 24, 1864, 1, 1), (1, 6, 6, 16, 1024, 1024, 1), (1, 9, 8, 136, 72, 1, 0), (2, 7, 7, 24, 136, 4, 0)]
# n additions of float32 round a sum that stays within 4 RMS by 2^-24 * 4 RMS each, with random signs: sqrt(n) * 2^-24 * 4 RMS,
# n = K / 16 (an MFMA step adds 16 products), against the metric's floor of 1 % of the RMS: 1.1e-3 for K = 32768
SPLITK_BAR = 1.1e-3


@pytest.mark.parametrize("m,n,k,small", SPLITK_GEMM_CASES)
def test_gemm_fwd_split_k(m, n, k, small, knob):
    knob("TWN_SMALL", small)
    x, w, tw, codes, alpha = make_layer(m + n + k, (m, k), (n, k), groups=n if m % 2 == 0 else 1)
    ref = oc.gemm_fwd(x, codes.reshape(n, k), alpha)
    assert api.twn_gemm_fwd_workspace_bytes(m, tw) > 0                  # K is cut
    assert rel_err(to_host_f64(api.twn_gemm_fwd(to_dev_bf16(x), tw, y_dtype=torch.float32)), ref) <= SPLITK_BAR
    g = np.random.default_rng(k)
    scale, shift = g.uniform(0.5, 1.5, n).astype(np.float32), g.standard_normal(n).astype(np.float32)
    res = wl.bf16_round(g.standard_normal((m, n)).astype(np.float32))
    y = api.twn_gemm_fwd(to_dev_bf16(x), tw, scale=to_dev_f32(scale), shift=to_dev_f32(shift), residual=to_dev_bf16(res), relu=True)
    assert rel_err(to_host_f64(y), oc.epilogue(ref, scale, shift, res, relu=True)) <= BF16_TOL


@pytest.mark.parametrize("n,h,w_,c,o,groups,small", SPLITK_CONV_CASES)
def test_convolution_split_k(n, h, w_, c, o, groups, small, knob):
    knob("TWN_SMALL", small)
    geo = (1, 1), (1, 1), (1, 1)
    x, w, tw, codes, alpha = make_layer(n + c + o, (n, h, w_, c), (o, c, 3, 3), groups=groups, transposed=True)
    y = api.twn_conv2d_fwd(to_dev_bf16(x), tw, *geo, y_dtype=torch.float32)
    ref = oc.conv2d_fwd(x, codes, alpha, *geo)
    assert rel_err(to_host_f64(y), ref) <= SPLITK_BAR
    dy = wl.bf16_round(np.random.default_rng(o).standard_normal(ref.shape).astype(np.float32))
    dx, _, _ = api.twn_conv2d_bwd_ste(None, to_dev_bf16(dy), tw, *geo, need_dw=False, x_shape=x.shape, dx_dtype=torch.float32)
    # two bf16 terms per value with several alphas: 2^-17 of each, bar of the per-filter tests
    assert rel_err(to_host_f64(dx), oc.conv2d_bwd_data(dy, codes, alpha, x.shape, *geo)) <= (2e-3 if groups > 1 else SPLITK_BAR)


BWD_CASES = list(range(len(CONV_CASES)))      # includes the 7x7 / stride-2 / C = 3 stem shape (index 5)


@pytest.mark.parametrize("ks", [1, 2])
@pytest.mark.parametrize("ci", [1, 2, 4, 7])
def test_weight_grad_wave_groups(ci, ks, knob):
    # the weight-gradient kernel with one and with two groups of waves per workgroup (the second sums the groups
    # through LDS), on tiles of 128 filters (cases 1, 2, 7) and on the 64-filter arrangement (case 4), several
    # pixel ranges per tile in each
    knob("TWN_WG_KS", ks)
    n, h, w_, c, o, r, s, st, pd, dl = CONV_CASES[ci]
    n = 4 * n                                     # more pixels: more than one range per tile
    x, w, tw, codes, alpha = make_layer(260 + ci, (n, h, w_, c), (o, c, r, s), transposed=True)
    p, q = oc.out_size(h, r, st[0], pd[0], dl[0]), oc.out_size(w_, s, st[1], pd[1], dl[1])
    dy = wl.bf16_round(np.random.default_rng(360 + ci).standard_normal((n, p, q, o)).astype(np.float32))
    _, dw, _ = api.twn_conv2d_bwd_ste(to_dev_bf16(x), to_dev_bf16(dy), tw, st, pd, dl, need_dx=False)
    assert rel_err(to_host_f64(dw), oc.conv2d_bwd_weight(x, dy, codes.shape, st, pd, dl)) <= 1e-4


@pytest.mark.usefixtures("both_dispatches")
@pytest.mark.parametrize("ci", BWD_CASES)
def test_conv2d_bwd_ste(ci):
    n, h, w_, c, o, r, s, st, pd, dl = CONV_CASES[ci]
    x, w, tw, codes, alpha = make_layer(200 + ci, (n, h, w_, c), (o, c, r, s), transposed=True)
    p, q = oc.out_size(h, r, st[0], pd[0], dl[0]), oc.out_size(w_, s, st[1], pd[1], dl[1])
    dy = wl.bf16_round(np.random.default_rng(300 + ci).standard_normal((n, p, q, o)).astype(np.float32))
    dx, dw, db = api.twn_conv2d_bwd_ste(to_dev_bf16(x), to_dev_bf16(dy), tw, st, pd, dl, need_dbias=True,
                                        dx_dtype=torch.float32)
    ref_dx = oc.conv2d_bwd_data(dy, codes, alpha, x.shape, st, pd, dl)
    ref_dw = oc.conv2d_bwd_weight(x, dy, codes.shape, st, pd, dl)
    assert rel_err(to_host_f64(dx), ref_dx) <= 1e-4
    assert rel_err(to_host_f64(dw), ref_dw) <= 1e-4
    assert rel_err(to_host_f64(db), oc.bias_grad(dy)) <= 1e-4
    dxb, _, _ = api.twn_conv2d_bwd_ste(to_dev_bf16(x), to_dev_bf16(dy), tw, st, pd, dl, need_dw=False)
    assert rel_err(to_host_f64(dxb), ref_dx) <= BF16_TOL
    # accumulate into an existing gradient; dW does not depend on the codes or alpha (identity STE)
    _, dw2, _ = api.twn_conv2d_bwd_ste(to_dev_bf16(x), to_dev_bf16(dy), tw, st, pd, dl, need_dx=False,
                                       dW=dw.clone(), accumulate=True)
    assert rel_err(to_host_f64(dw2), 2 * ref_dw) <= 1e-4


@pytest.mark.usefixtures("both_dispatches")
def test_fc_backward_is_the_1x1_case():
    m, k, n = 128, 512, 1000
    x, w, tw, codes, alpha = make_layer(9, (m, 1, 1, k), (n, k, 1, 1), transposed=True)
    dy = wl.bf16_round(np.random.default_rng(10).standard_normal((m, 1, 1, n)).astype(np.float32))
    dx, dw, _ = api.twn_conv2d_bwd_ste(to_dev_bf16(x), to_dev_bf16(dy), tw, dx_dtype=torch.float32)
    assert rel_err(to_host_f64(dx), oc.conv2d_bwd_data(dy, codes, alpha, x.shape)) <= 1e-4
    assert rel_err(to_host_f64(dw), oc.conv2d_bwd_weight(x, dy, codes.shape)) <= 1e-4


def _sample(total, count, seed):
    return np.unique(np.random.default_rng(seed).integers(0, total, size=count))


def test_full_size_gemm_sampled():
    """Config: X [8192 x 4096] bf16 N(0,1), W [4096 x 4096] N(0, 0.02^2), f = 0.7; sampled outputs.
    For time, Delta comes from the oracle's threshold routine and alpha is recomputed here from the codes
    (Eq. 5 written out) instead of through the oracle's sort route; nnz is compared with the GPU's count."""
    m, n, k = 8192, 4096, 4096
    x = wl.bf16_round(wl.normal(3, wl.IDX_INPUT, (m, k)))
    w = wl.normal(3, 1, (n, k), std=0.02)
    tw = api.twn_ternarize(to_dev_f32(w), F)
    y = api.twn_gemm_fwd(to_dev_bf16(x), tw)
    torch.cuda.synchronize()
    delta = ot.threshold(w, F)
    codes = ot.codes_from_threshold(w, delta)
    nnz = int(np.count_nonzero(codes))
    alpha = np.float32(float(np.sum(np.abs(w)[codes != 0], dtype=np.float64)) / nnz)
    assert int(tw.nnz.cpu()[0]) == nnz
    idx = np.concatenate([_sample(m * n, 20000, 5), np.array([0, n - 1, (m - 1) * n, m * n - 1])])
    ref = oc.gemm_fwd_at(x, codes, alpha, idx)
    got = to_host_f64(y).ravel()[idx]
    assert rel_err(got, ref) <= BF16_TOL


@pytest.mark.parametrize("name", ["stem", "l1.0.conv1", "l2.0.conv1", "l2.0.down", "l3.1.conv2", "l4.1.conv2", "fc"])
def test_full_size_resnet18_layers_sampled(name):
    layers = {l.name: (i, l) for i, l in enumerate(wl.resnet18(64))}
    li, layer = layers[name]
    x = wl.bf16_round(wl.normal(2, wl.IDX_INPUT + li, layer.x_shape))
    w = wl.kaiming_weights(2, li, layer)
    tw = api.twn_ternarize(to_dev_f32(w), F)
    codes, delta, alpha, nnz = ot.ternarize(w, F)
    st, pd, dl = (layer.stride,) * 2, (layer.pad,) * 2, (layer.dil,) * 2
    y = api.twn_conv2d_fwd(to_dev_bf16(x), tw, st, pd, dl)
    total = int(np.prod(layer.y_shape))
    # random outputs plus the four image corners of the first and last image (border taps)
    n_, p_, q_, o_ = layer.y_shape
    corners = [((b * p_ + pp) * q_ + qq) * o_ for b in (0, n_ - 1) for pp in (0, p_ - 1) for qq in (0, q_ - 1)]
    idx = np.concatenate([_sample(total, 20000, li), np.array(corners)])
    ref = oc.conv2d_fwd_at(x, codes, alpha, idx, st, pd, dl)
    assert rel_err(to_host_f64(y).ravel()[idx], ref) <= BF16_TOL


@pytest.mark.parametrize("name", ["conv1", "conv5", "conv8", "fc6", "fc7"])
def test_full_size_detection_backbone_layers_sampled(name):
    # the 300x300 detection stand-in at batch 32: odd image sizes, the dilated 3x3 (dilation 6) and the 1x1 layer
    layers = {l.name: (i, l) for i, l in enumerate(wl.vgg16_ssd(32))}
    li, layer = layers[name]
    x = wl.bf16_round(wl.normal(4, wl.IDX_INPUT + li, layer.x_shape))
    w = wl.kaiming_weights(4, li, layer)
    tw = api.twn_ternarize(to_dev_f32(w), F)
    codes, delta, alpha, nnz = ot.ternarize(w, F)
    st, pd, dl = (layer.stride,) * 2, (layer.pad,) * 2, (layer.dil,) * 2
    y = api.twn_conv2d_fwd(to_dev_bf16(x), tw, st, pd, dl)
    total = int(np.prod(layer.y_shape))
    n_, p_, q_, o_ = layer.y_shape
    corners = [((b * p_ + pp) * q_ + qq) * o_ for b in (0, n_ - 1) for pp in (0, p_ - 1) for qq in (0, q_ - 1)]
    idx = np.concatenate([_sample(total, 20000, li), np.array(corners)])
    ref = oc.conv2d_fwd_at(x, codes, alpha, idx, st, pd, dl)
    assert rel_err(to_host_f64(y).ravel()[idx], ref) <= BF16_TOL


@pytest.mark.parametrize("name", ["c1", "c2", "c4", "c6", "fc1"])
def test_full_size_vgg7_backward_sampled(name):
    layers = {l.name: (i, l) for i, l in enumerate(wl.vgg7(128))}
    li, layer = layers[name]
    x = wl.bf16_round(wl.normal(1, wl.IDX_INPUT + li, layer.x_shape))
    dy = wl.bf16_round(wl.normal(1, wl.IDX_DY + 10 * li, layer.y_shape))
    w = wl.kaiming_weights(1, li, layer)
    tw = api.twn_ternarize(to_dev_f32(w), F, transposed=True)
    codes, delta, alpha, nnz = ot.ternarize(w, F)
    st, pd, dl = (layer.stride,) * 2, (layer.pad,) * 2, (layer.dil,) * 2
    dx, dw, _ = api.twn_conv2d_bwd_ste(to_dev_bf16(x), to_dev_bf16(dy), tw, st, pd, dl, need_dx=(name != "c1"))
    i2 = _sample(layer.n_weights, 300, li + 7)
    ref_dw = oc.conv2d_bwd_weight_at(x, dy, layer.w_shape, i2, st, pd, dl)
    assert rel_err(to_host_f64(dw).ravel()[i2], ref_dw) <= 1e-3
    if dx is not None:
        i1 = _sample(int(np.prod(layer.x_shape)), 20000, li)
        ref_dx = oc.conv2d_bwd_data_at(dy, codes, alpha, layer.x_shape, i1, st, pd, dl)
        assert rel_err(to_host_f64(dx).ravel()[i1], ref_dx) <= BF16_TOL


@pytest.mark.parametrize("name", ["c1", "c2", "c3", "c4", "c5", "c6", "fc1", "fc2"])
def test_full_size_vgg7_forward_sampled(name):
    """The timed workload's forward calls at full size, as bench.py launches them (fused scale/shift/ReLU tail,
    weights ternarized by the multi-tensor call); sampled outputs plus the image corners against the oracle."""
    all_layers = wl.vgg7(128)
    layers = {l.name: (i, l) for i, l in enumerate(all_layers)}
    li, layer = layers[name]
    x = wl.bf16_round(wl.normal(1, wl.IDX_INPUT + li, layer.x_shape))
    w = wl.kaiming_weights(1, li, layer)
    tw = api.twn_ternarize_batch([to_dev_f32(w)], F, transposed=True)[0]
    codes, delta, alpha, nnz = ot.ternarize(w if w.ndim == 4 else w.reshape(w.shape[0], w.shape[1], 1, 1), F)
    g = np.random.default_rng(900 + li)
    scale = g.uniform(0.5, 1.5, layer.O).astype(np.float32)
    shift = (0.1 * g.standard_normal(layer.O)).astype(np.float32)
    st, pd, dl = (layer.stride,) * 2, (layer.pad,) * 2, (layer.dil,) * 2
    y = api.twn_conv2d_fwd(to_dev_bf16(x), tw, st, pd, dl, scale=to_dev_f32(scale), shift=to_dev_f32(shift), relu=True)
    total = int(np.prod(layer.y_shape))
    n_, p_, q_, o_ = layer.y_shape
    corners = [((b * p_ + pp) * q_ + qq) * o_ for b in (0, n_ - 1) for pp in (0, p_ - 1) for qq in (0, q_ - 1)]
    idx = np.unique(np.concatenate([_sample(total, 20000, li), np.array(corners), np.array([total - 1])]))
    z = oc.conv2d_fwd_at(x, codes, alpha, idx, st, pd, dl)
    ch = idx % o_
    ref = np.maximum(z * scale[ch].astype(np.float64) + shift[ch].astype(np.float64), 0.0)
    got = to_host_f64(y).ravel()[idx]
    # relative to the magnitudes before the ReLU cut (a clipped output has no scale of its own)
    floor = 1e-2 * np.sqrt(np.mean(z * z))
    assert np.max(np.abs(got - ref) / np.maximum(np.abs(ref), floor)) <= BF16_TOL


def test_library_calls_capture_into_a_graph_and_replay():
    # the library only launches kernels and takes its workspaces from the caller, so a ternarize + forward +
    # two-stream backward sequence captures into a HIP graph; every replay (with eager work and
    # synchronisations between the replays) must reproduce the eager results bit for bit
    n, h, w_, c, o = 4, 12, 12, 64, 128
    st, pd, dl = (1, 1), (1, 1), (1, 1)
    g = np.random.default_rng(77)
    x = to_dev_bf16(wl.bf16_round(g.standard_normal((n, h, w_, c)).astype(np.float32)))
    dy = to_dev_bf16(wl.bf16_round(g.standard_normal((n, h, w_, o)).astype(np.float32)))
    wts = [to_dev_f32((g.standard_normal((o, c, 3, 3)) * 0.05).astype(np.float32)),
           to_dev_f32((g.standard_normal((10, 256)) * 0.05).astype(np.float32))]
    tws = api.twn_ternarize_batch(wts, F, transposed=True)
    tern_ws = torch.empty(api.lib().twn_ternarize_batch_workspace_bytes(2), dtype=torch.uint8, device="cuda")
    y = torch.empty((n, h, w_, o), dtype=torch.bfloat16, device="cuda")
    dx = torch.empty((n, h, w_, c), dtype=torch.bfloat16, device="cuda")
    dw = torch.empty((o, c, 3, 3), dtype=torch.float32, device="cuda")
    nws = max(16, api.twn_conv2d_bwd_ste_workspace_bytes((n, h, w_, c), tws[0], st, pd, dl))
    ws_a = torch.empty(nws, dtype=torch.uint8, device="cuda")
    ws_b = torch.empty(nws, dtype=torch.uint8, device="cuda")
    ws_f = torch.empty(max(16, api.twn_conv2d_fwd_workspace_bytes((n, h, w_, c), tws[0], st, pd, dl)),
                       dtype=torch.uint8, device="cuda")
    side_a, side_b = torch.cuda.Stream(), torch.cuda.Stream()

    def sequence():
        api.twn_ternarize_batch(wts, F, transposed=True, out=tws, workspace=tern_ws)
        api.twn_conv2d_fwd(x, tws[0], st, pd, dl, relu=True, out=y, workspace=ws_f)
        cur = torch.cuda.current_stream()
        fork = torch.cuda.Event()
        fork.record(cur)
        side_a.wait_event(fork)
        side_b.wait_event(fork)
        api.twn_conv2d_bwd_ste(None, dy, tws[0], st, pd, dl, need_dx=True, need_dw=False, dX=dx, x_shape=(n, h, w_, c),
                               workspace=ws_a, stream=side_a)
        api.twn_conv2d_bwd_ste(x, dy, tws[0], st, pd, dl, need_dx=False, need_dw=True, dW=dw, workspace=ws_b,
                               stream=side_b)
        ja, jb = torch.cuda.Event(), torch.cuda.Event()
        ja.record(side_a)
        jb.record(side_b)
        cur.wait_event(ja)
        cur.wait_event(jb)

    outs = (y, dx, dw, tws[0].packed, tws[0].packed_T, tws[1].packed, tws[0].alpha)
    sequence()
    torch.cuda.synchronize()
    ref = [t.clone() for t in outs]
    cap = torch.cuda.Stream()
    cap.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(cap):
        sequence()
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=cap):
        sequence()
    torch.cuda.synchronize()
    for rep in range(4):
        for t in outs:
            t.zero_()
        if rep % 2:
            # eager work of the program itself between two replays
            api.twn_conv2d_fwd(x, api.twn_ternarize(wts[0], F), st, pd, dl)
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        for a, b in zip(ref, outs):
            assert torch.equal(a, b)


def test_per_lane_pointer_load_path(knob):
    # tensors of 2 GiB and more cannot use buffer descriptors and fall back to per-lane pointers; the switch
    # that forces that path keeps it covered at test sizes: GEMM, convolution, both gradients
    knob("TWN_BUFLOAD", "0")
    m, n, k = 520, 300, 448
    x, w, tw, codes, alpha = make_layer(41, (m, k), (n, k))
    y = api.twn_gemm_fwd(to_dev_bf16(x), tw, y_dtype=torch.float32)
    assert rel_err(to_host_f64(y), oc.gemm_fwd(x, codes.reshape(n, k), alpha)) <= 1e-4
    for ci in (1, 2):
        nb, h, w_, c, o, r, s, st, pd, dl = CONV_CASES[ci]
        x, w, tw, codes, alpha = make_layer(42 + ci, (nb, h, w_, c), (o, c, r, s), transposed=True)
        ref = oc.conv2d_fwd(x, codes, alpha, st, pd, dl)
        y = api.twn_conv2d_fwd(to_dev_bf16(x), tw, st, pd, dl, y_dtype=torch.float32)
        assert rel_err(to_host_f64(y), ref) <= 1e-4
        dy = wl.bf16_round(np.random.default_rng(45 + ci).standard_normal(ref.shape).astype(np.float32))
        dx, dw, _ = api.twn_conv2d_bwd_ste(to_dev_bf16(x), to_dev_bf16(dy), tw, st, pd, dl, dx_dtype=torch.float32)
        assert rel_err(to_host_f64(dx), oc.conv2d_bwd_data(dy, codes, alpha, x.shape, st, pd, dl)) <= 1e-4
        assert rel_err(to_host_f64(dw), oc.conv2d_bwd_weight(x, dy, codes.shape, st, pd, dl)) <= 1e-4


@pytest.mark.usefixtures("both_dispatches")
@pytest.mark.parametrize("groups", ["filters", 4])
def test_conv2d_bwd_data_per_filter_alpha(groups):
    # Alg. 1 with one alpha per filter (or per group of filters): alpha_o sits inside the sum over o, so the
    # library scales dY per channel first and carries the product as two bf16 terms (16 significant bits, 2^-17
    # relative per input).  Under the metric of every other test (error against max(|ref|, 1% of the RMS)) that is
    # 2^-17 / 1e-2 = 8e-4 at the smallest outputs with float32 output (bar here 2e-3; the per-layer path, whose
    # inputs are exact, has 1e-4), and the bf16-MFMA bar of 2e-2 with bf16 output as for every other layer.
    for ci in (1, 2, 9):
        n, h, w_, c, o, r, s, st, pd, dl = CONV_CASES[ci]
        gcount = o if groups == "filters" else groups
        x, w, tw, codes, alpha = make_layer(500 + ci, (n, h, w_, c), (o, c, r, s), groups=gcount, transposed=True)
        p, q = oc.out_size(h, r, st[0], pd[0], dl[0]), oc.out_size(w_, s, st[1], pd[1], dl[1])
        dy = wl.bf16_round(np.random.default_rng(510 + ci).standard_normal((n, p, q, o)).astype(np.float32))
        ref = oc.conv2d_bwd_data(dy, codes, alpha, x.shape, st, pd, dl)
        dx, dw, _ = api.twn_conv2d_bwd_ste(to_dev_bf16(x), to_dev_bf16(dy), tw, st, pd, dl, dx_dtype=torch.float32)
        assert rel_err(to_host_f64(dx), ref) <= 2e-3
        dxb, _, _ = api.twn_conv2d_bwd_ste(None, to_dev_bf16(dy), tw, st, pd, dl, need_dw=False, x_shape=x.shape)
        assert rel_err(to_host_f64(dxb), ref) <= BF16_TOL
        assert rel_err(to_host_f64(dw), oc.conv2d_bwd_weight(x, dy, codes.shape, st, pd, dl)) <= 1e-4


STRIDED_DX_CASES = [
    # N  H   W   C   O    R  S  stride  pad
    (2, 14, 14, 128, 256, 3, 3, (2, 2), (1, 1)),
    (2, 15, 13, 16, 64, 3, 3, (2, 2), (1, 1)),      # odd extents: the classes have different numbers of pixels
    (3, 16, 16, 64, 128, 1, 1, (2, 2), (0, 0)),     # 1x1: three of the four classes have no tap (zeros)
    (2, 31, 29, 8, 64, 7, 7, (2, 2), (3, 3)),
    (2, 12, 17, 32, 64, 5, 5, (2, 2), (2, 2)),
    (2, 13, 12, 24, 128, 3, 3, (2, 1), (1, 1)),
    (2, 12, 13, 24, 64, 3, 2, (1, 2), (0, 1)),
    (1, 9, 9, 8, 64, 2, 2, (2, 2), (0, 0)),         # taps and stride coincide: one tap per class
    (2, 10, 10, 16, 64, 3, 3, (2, 2), (0, 0)),
]


@pytest.mark.usefixtures("both_dispatches")
@pytest.mark.parametrize("ci", range(len(STRIDED_DX_CASES)))
def test_strided_backward_data_by_residue_classes(ci, knob):
    # strided layers run one stride-1 contraction per residue class of the output pixels (forced here for
    # small shapes); both output types, and the generic divided gather as a cross-check
    n, h, w_, c, o, r, s, st, pd = STRIDED_DX_CASES[ci]
    dl = (1, 1)
    x, w, tw, codes, alpha = make_layer(700 + ci, (n, h, w_, c), (o, c, r, s), transposed=True)
    p, q = oc.out_size(h, r, st[0], pd[0], 1), oc.out_size(w_, s, st[1], pd[1], 1)
    dy = wl.bf16_round(np.random.default_rng(710 + ci).standard_normal((n, p, q, o)).astype(np.float32))
    ref = oc.conv2d_bwd_data(dy, codes, alpha, x.shape, st, pd, dl)
    knob("TWN_DX_CLASS_MIN_PIXELS", "0")
    dx32, _, _ = api.twn_conv2d_bwd_ste(None, to_dev_bf16(dy), tw, st, pd, dl, need_dw=False, x_shape=x.shape,
                                        dx_dtype=torch.float32)
    assert rel_err(to_host_f64(dx32), ref) <= 1e-4
    dxb, _, _ = api.twn_conv2d_bwd_ste(None, to_dev_bf16(dy), tw, st, pd, dl, need_dw=False, x_shape=x.shape)
    assert rel_err(to_host_f64(dxb), ref) <= BF16_TOL
    # one launch per class instead of all classes in one launch: the same bits
    knob("TWN_DX_CLASS_BATCH", "0")
    dxs, _, _ = api.twn_conv2d_bwd_ste(None, to_dev_bf16(dy), tw, st, pd, dl, need_dw=False, x_shape=x.shape,
                                       dx_dtype=torch.float32)
    assert torch.equal(dxs, dx32)
    knob("TWN_DX_CLASSES", "0")
    dxg, _, _ = api.twn_conv2d_bwd_ste(None, to_dev_bf16(dy), tw, st, pd, dl, need_dw=False, x_shape=x.shape,
                                       dx_dtype=torch.float32)
    assert rel_err(to_host_f64(dxg), ref) <= 1e-4


@pytest.mark.usefixtures("both_dispatches")
@pytest.mark.parametrize("ci", range(len(STRIDED_DX_CASES)))
def test_strided_backward_data_by_residue_classes_per_filter_alpha(ci, knob):
    # the residue-class path with one alpha per filter: alpha_o * dY as two bf16 terms side by side, one contraction
    # per class over both through the output-row remap (bars as in the per-filter test above)
    n, h, w_, c, o, r, s, st, pd = STRIDED_DX_CASES[ci]
    dl = (1, 1)
    x, w, tw, codes, alpha = make_layer(720 + ci, (n, h, w_, c), (o, c, r, s), groups=o, transposed=True)
    p, q = oc.out_size(h, r, st[0], pd[0], 1), oc.out_size(w_, s, st[1], pd[1], 1)
    dy = wl.bf16_round(np.random.default_rng(730 + ci).standard_normal((n, p, q, o)).astype(np.float32))
    ref = oc.conv2d_bwd_data(dy, codes, alpha, x.shape, st, pd, dl)
    knob("TWN_DX_CLASS_MIN_PIXELS", "0")
    dx32, _, _ = api.twn_conv2d_bwd_ste(None, to_dev_bf16(dy), tw, st, pd, dl, need_dw=False, x_shape=x.shape,
                                        dx_dtype=torch.float32)
    assert rel_err(to_host_f64(dx32), ref) <= 2e-3
    dxb, _, _ = api.twn_conv2d_bwd_ste(None, to_dev_bf16(dy), tw, st, pd, dl, need_dw=False, x_shape=x.shape)
    assert rel_err(to_host_f64(dxb), ref) <= BF16_TOL


def test_full_size_resnet18_strided_backward_data_sampled():
    layers = {l.name: (i, l) for i, l in enumerate(wl.resnet18(64))}
    for name in ("l2.0.conv1", "l2.0.down"):
        li, layer = layers[name]
        dy = wl.bf16_round(wl.normal(2, wl.IDX_DY + 10 * li, layer.y_shape))
        w = wl.kaiming_weights(2, li, layer)
        tw = api.twn_ternarize(to_dev_f32(w), F, transposed=True)
        codes, delta, alpha, nnz = ot.ternarize(w, F)
        st, pd, dl = (layer.stride,) * 2, (layer.pad,) * 2, (layer.dil,) * 2
        dx, _, _ = api.twn_conv2d_bwd_ste(None, to_dev_bf16(dy), tw, st, pd, dl, need_dw=False, x_shape=layer.x_shape)
        n_, h_, w_, c_ = layer.x_shape
        corners = [((b * h_ + hh) * w_ + ww) * c_ for b in (0, n_ - 1) for hh in (0, 1, h_ - 2, h_ - 1)
                   for ww in (0, 1, w_ - 2, w_ - 1)]
        idx = np.unique(np.concatenate([_sample(int(np.prod(layer.x_shape)), 20000, li), np.array(corners)]))
        ref = oc.conv2d_bwd_data_at(dy, codes, alpha, layer.x_shape, idx, st, pd, dl)
        assert rel_err(to_host_f64(dx).ravel()[idx], ref) <= BF16_TOL


@pytest.mark.parametrize("name", ["stem", "l1.0.conv1", "l2.0.conv1", "l3.0.down", "l4.1.conv2", "fc"])
def test_full_size_resnet18_backward_sampled(name):
    """The layers bench.py times in the ResNet-18 backward, at full size (batch 64): sampled dW entries
    (every tap position of some filter included) and sampled dX entries with the image corners."""
    layers = {l.name: (i, l) for i, l in enumerate(wl.resnet18(64))}
    li, layer = layers[name]
    x = wl.bf16_round(wl.normal(2, wl.IDX_INPUT + li, layer.x_shape))
    dy = wl.bf16_round(wl.normal(2, wl.IDX_DY + 10 * li, layer.y_shape))
    w = wl.kaiming_weights(2, li, layer)
    tw = api.twn_ternarize(to_dev_f32(w), F, transposed=True)
    codes, delta, alpha, nnz = ot.ternarize(w, F)
    st, pd, dl = (layer.stride,) * 2, (layer.pad,) * 2, (layer.dil,) * 2
    need_dx = name != "stem"
    dx, dw, _ = api.twn_conv2d_bwd_ste(to_dev_bf16(x), to_dev_bf16(dy), tw, st, pd, dl, need_dx=need_dx)
    per_filter = layer.C * layer.R * layer.S
    # all taps and channels of the first and the last filter (at most 600 entries each), plus random entries
    first = np.arange(min(per_filter, 600))
    last = layer.n_weights - 1 - np.arange(min(per_filter, 600))
    i2 = np.unique(np.concatenate([_sample(layer.n_weights, 300, li + 7), first, last]))
    if layer.N * layer.P * layer.Q > 300000:
        i2 = i2[:: max(1, i2.size // 400)]        # the oracle sums ~10^6 pixels per entry on the large layers
    ref_dw = oc.conv2d_bwd_weight_at(x, dy, layer.w_shape, i2, st, pd, dl)
    assert rel_err(to_host_f64(dw).ravel()[i2], ref_dw) <= 1e-3
    if need_dx:
        n_, h_, w_, c_ = layer.x_shape
        corners = [((b * h_ + hh) * w_ + ww) * c_ for b in (0, n_ - 1) for hh in (0, h_ - 1) for ww in (0, w_ - 1)]
        i1 = np.unique(np.concatenate([_sample(int(np.prod(layer.x_shape)), 20000, li), np.array(corners)]))
        ref_dx = oc.conv2d_bwd_data_at(dy, codes, alpha, layer.x_shape, i1, st, pd, dl)
        assert rel_err(to_host_f64(dx).ravel()[i1], ref_dx) <= BF16_TOL


FIRST_LAYER_CASES = [
    # N  H   W   O   R  S  stride  pad      (C = 3, even W: the persistent first-layer kernel)
    (2, 30, 28, 64, 7, 7, (2, 2), (3, 3)),
    (3, 18, 20, 72, 3, 3, (1, 1), (1, 1)),
    (2, 17, 22, 40, 5, 5, (2, 2), (2, 2)),       # even padding: the patch starts at the first tap
    (1, 9, 10, 8, 3, 3, (1, 1), (0, 0)),
    (2, 21, 26, 136, 3, 3, (1, 2), (1, 1)),      # three channel tiles, mixed strides
    (2, 40, 36, 64, 7, 5, (2, 1), (3, 2)),
    (5, 33, 34, 64, 1, 1, (1, 1), (0, 0)),
]


@pytest.mark.parametrize("ci", range(len(FIRST_LAYER_CASES)))
def test_first_layer_kernel(ci):
    n, h, w_, o, r, s, st, pd = FIRST_LAYER_CASES[ci]
    dl = (1, 1)
    groups = o if ci % 2 else 1
    x, w, tw, codes, alpha = make_layer(800 + ci, (n, h, w_, 3), (o, 3, r, s), groups=groups)
    g = np.random.default_rng(ci)
    scale = g.uniform(0.5, 1.5, o).astype(np.float32)
    shift = g.standard_normal(o).astype(np.float32)
    ref0 = oc.conv2d_fwd(x, codes, alpha, st, pd, dl)
    y = api.twn_conv2d_fwd(to_dev_bf16(x), tw, st, pd, dl)
    assert tuple(y.shape) == ref0.shape
    assert rel_err(to_host_f64(y), ref0) <= BF16_TOL
    res = wl.bf16_round(g.standard_normal(ref0.shape).astype(np.float32))
    y2 = api.twn_conv2d_fwd(to_dev_bf16(x), tw, st, pd, dl, scale=to_dev_f32(scale), shift=to_dev_f32(shift),
                            residual=to_dev_bf16(res), relu=True)
    assert rel_err(to_host_f64(y2), oc.epilogue(ref0, scale, shift, res, relu=True)) <= BF16_TOL


def test_first_layer_kernel_matches_generic_path(knob):
    # the same call through the generic small-C path (padded copy + re-ordered codes): both round once from fp32
    n, h, w_, o, r, s, st, pd = FIRST_LAYER_CASES[0]
    x, w, tw, codes, alpha = make_layer(850, (n, h, w_, 3), (o, 3, r, s))
    y1 = api.twn_conv2d_fwd(to_dev_bf16(x), tw, st, pd, (1, 1))
    knob("TWN_FIRST", "0")
    y0 = api.twn_conv2d_fwd(to_dev_bf16(x), tw, st, pd, (1, 1))
    ref = oc.conv2d_fwd(x, codes, alpha, st, pd, (1, 1))
    assert rel_err(to_host_f64(y0), ref) <= BF16_TOL and rel_err(to_host_f64(y1), ref) <= BF16_TOL
    assert rel_err(to_host_f64(y1), to_host_f64(y0)) <= BF16_TOL


C64_CASES = [
    # N  H   W   O    pad     (C = 64, 3x3, stride 1: weights resident in registers, 8x8 pixel tiles with halo in LDS)
    (3, 17, 19, 64, (1, 1)),        # ragged tiles in both directions
    (2, 16, 24, 128, (1, 1)),       # two channel tiles, whole pixel tiles
    (5, 8, 8, 64, (1, 1)),          # one tile per image
    (2, 20, 33, 64, (0, 2)),        # output smaller / larger than the input
    (1, 7, 5, 192, (2, 0)),
    (24, 40, 36, 64, (1, 1)),       # 600 tiles: more than the resident workgroups, so some walk two tiles
]


@pytest.mark.parametrize("ci", range(len(C64_CASES)))
def test_resident_weight_3x3_kernel_forward(ci):
    n, h, w_, o, pd = C64_CASES[ci]
    st = dl = (1, 1)
    groups = o if ci % 2 else 1
    x, w, tw, codes, alpha = make_layer(900 + ci, (n, h, w_, 64), (o, 64, 3, 3), groups=groups)
    g = np.random.default_rng(ci)
    scale = g.uniform(0.5, 1.5, o).astype(np.float32)
    shift = g.standard_normal(o).astype(np.float32)
    ref0 = oc.conv2d_fwd(x, codes, alpha, st, pd, dl)
    y = api.twn_conv2d_fwd(to_dev_bf16(x), tw, st, pd, dl)
    assert tuple(y.shape) == ref0.shape
    assert rel_err(to_host_f64(y), ref0) <= BF16_TOL
    res = wl.bf16_round(g.standard_normal(ref0.shape).astype(np.float32))
    y2 = api.twn_conv2d_fwd(to_dev_bf16(x), tw, st, pd, dl, scale=to_dev_f32(scale), shift=to_dev_f32(shift),
                            residual=to_dev_bf16(res), relu=True)
    assert rel_err(to_host_f64(y2), oc.epilogue(ref0, scale, shift, res, relu=True)) <= BF16_TOL


@pytest.mark.parametrize("ci", range(len(C64_CASES)))
def test_resident_weight_3x3_kernel_backward_data(ci):
    # the data gradient of a layer with 64 FILTERS is the same kind of problem over dY (mirrored taps, transposed codes)
    n, h, w_, c, pd = C64_CASES[ci]
    st = dl = (1, 1)
    x, w, tw, codes, alpha = make_layer(930 + ci, (n, h, w_, c), (64, c, 3, 3), transposed=True)
    p, q = h + 2 * pd[0] - 2, w_ + 2 * pd[1] - 2
    dy = wl.bf16_round(np.random.default_rng(ci).standard_normal((n, p, q, 64)).astype(np.float32))
    dx, _, _ = api.twn_conv2d_bwd_ste(None, to_dev_bf16(dy), tw, st, pd, dl, need_dx=True, need_dw=False,
                                      x_shape=(n, h, w_, c))
    assert rel_err(to_host_f64(dx), oc.conv2d_bwd_data(dy, codes, alpha, (n, h, w_, c), st, pd, dl)) <= BF16_TOL


@pytest.mark.parametrize("ci", [0, 3])
def test_resident_weight_3x3_kernel_backward_data_per_filter_alpha(ci):
    # one alpha per filter: the kernel forms alpha * dY as two bf16 terms on the way into LDS and multiplies both
    n, h, w_, c, pd = C64_CASES[ci]
    st = dl = (1, 1)
    x, w, tw, codes, alpha = make_layer(940 + ci, (n, h, w_, c), (64, c, 3, 3), groups=64, transposed=True)
    p, q = h + 2 * pd[0] - 2, w_ + 2 * pd[1] - 2
    dy = wl.bf16_round(np.random.default_rng(50 + ci).standard_normal((n, p, q, 64)).astype(np.float32))
    dx, _, _ = api.twn_conv2d_bwd_ste(None, to_dev_bf16(dy), tw, st, pd, dl, need_dx=True, need_dw=False,
                                      x_shape=(n, h, w_, c))
    assert rel_err(to_host_f64(dx), oc.conv2d_bwd_data(dy, codes, alpha, (n, h, w_, c), st, pd, dl)) <= BF16_TOL


def test_resident_weight_3x3_kernel_long_tile_walks(knob):
    knob("TWN_C64_OCC", "1")          # half the workgroups: two to three tiles each
    n, h, w_, o, pd = C64_CASES[5]
    x, w, tw, codes, alpha = make_layer(950, (n, h, w_, 64), (o, 64, 3, 3))
    y = api.twn_conv2d_fwd(to_dev_bf16(x), tw, (1, 1), pd, (1, 1))
    assert rel_err(to_host_f64(y), oc.conv2d_fwd(x, codes, alpha, (1, 1), pd, (1, 1))) <= BF16_TOL


def test_resident_weight_3x3_kernel_matches_generic_path(knob):
    n, h, w_, o, pd = C64_CASES[0]
    x, w, tw, codes, alpha = make_layer(960, (n, h, w_, 64), (o, 64, 3, 3))
    y1 = api.twn_conv2d_fwd(to_dev_bf16(x), tw, (1, 1), pd, (1, 1), relu=True)
    knob("TWN_C64", "0")
    y0 = api.twn_conv2d_fwd(to_dev_bf16(x), tw, (1, 1), pd, (1, 1), relu=True)
    ref = oc.epilogue(oc.conv2d_fwd(x, codes, alpha, (1, 1), pd, (1, 1)), relu=True)
    assert rel_err(to_host_f64(y0), ref) <= BF16_TOL and rel_err(to_host_f64(y1), ref) <= BF16_TOL
    assert rel_err(to_host_f64(y1), to_host_f64(y0)) <= BF16_TOL


@pytest.mark.parametrize("name", ["l1.0.conv1", "l1.0.conv2", "l2.0.conv2", "l3.0.conv2", "l4.1.conv2", "stem"])
def test_full_size_layers_are_identical_run_to_run(name):
    """Every output element is written, with the same bits, on every run (a 16-byte store whose data registers were
    overwritten one instruction later once left a few pixels per launch with an address in place of data)."""
    layers = {L.name: (li, L) for li, L in enumerate(wl.resnet18(64))}
    li, L = layers[name]
    g = torch.Generator(device="cuda").manual_seed(li)
    x = torch.randn(L.x_shape, device="cuda", generator=g).to(torch.bfloat16)
    tw = api.twn_ternarize(to_dev_f32(wl.kaiming_weights(2, li, L)), F)
    res = torch.randn(L.y_shape, device="cuda", generator=g).to(torch.bfloat16) if name.endswith("conv2") else None
    y = torch.empty(L.y_shape, dtype=torch.bfloat16, device="cuda")
    call = api.prepare_conv2d_fwd(x, tw, (L.stride,) * 2, (L.pad,) * 2, (L.dil,) * 2, out=y, residual=res, relu=True)
    y.fill_(-7.0)
    call()
    torch.cuda.synchronize()
    ref = y.clone()
    for fill in (0.0, -7.0, 3.0, 0.0, -7.0, 3.0, 0.0, -7.0):
        y.fill_(fill)
        call()
        torch.cuda.synchronize()
        assert torch.equal(y, ref)
    assert float(ref.min()) >= 0.0          # ReLU everywhere: no fill value left


@pytest.mark.parametrize("name", ["l1.0.conv1", "l2.0.conv1", "l3.1.conv2", "l4.0.down"])
def test_full_size_backward_is_identical_run_to_run(name):
    layers = {L.name: (li, L) for li, L in enumerate(wl.resnet18(64))}
    li, L = layers[name]
    g = torch.Generator(device="cuda").manual_seed(100 + li)
    x = torch.randn(L.x_shape, device="cuda", generator=g).to(torch.bfloat16)
    dy = torch.randn(L.y_shape, device="cuda", generator=g).to(torch.bfloat16)
    tw = api.twn_ternarize(to_dev_f32(wl.kaiming_weights(2, li, L)), F, transposed=True)
    geo = ((L.stride,) * 2, (L.pad,) * 2, (L.dil,) * 2)
    dx = torch.empty(L.x_shape, dtype=torch.bfloat16, device="cuda")
    dw = torch.empty((L.O, L.C, L.R, L.S), dtype=torch.float32, device="cuda")
    ref = None
    for fill in (0.0, -7.0, 3.0, 0.0, -7.0, 3.0):
        dx.fill_(fill)
        dw.fill_(fill)
        api.twn_conv2d_bwd_ste(x, dy, tw, *geo, dX=dx, dW=dw)
        torch.cuda.synchronize()
        if ref is None:
            ref = (dx.clone(), dw.clone())
        assert torch.equal(dx, ref[0]) and torch.equal(dw, ref[1])


def test_full_size_gemm_and_wide_tiles_are_identical_run_to_run():
    g = torch.Generator(device="cuda").manual_seed(5)
    cases = []
    x = torch.randn((8192, 4096), device="cuda", generator=g).to(torch.bfloat16)
    tw = api.twn_ternarize(torch.randn((4096, 4096), device="cuda", generator=g) * 0.02, F)
    y = torch.empty((8192, 4096), dtype=torch.bfloat16, device="cuda")
    cases.append((api.prepare_gemm_fwd(x, tw, out=y, relu=True), y))
    L = {l.name: l for l in wl.vgg16_ssd(32)}["conv8"]
    x2 = torch.randn(L.x_shape, device="cuda", generator=g).to(torch.bfloat16)
    tw2 = api.twn_ternarize(to_dev_f32(wl.kaiming_weights(5, 7, L)), F)
    y2 = torch.empty(L.y_shape, dtype=torch.bfloat16, device="cuda")
    cases.append((api.prepare_conv2d_fwd(x2, tw2, (L.stride,) * 2, (L.pad,) * 2, (L.dil,) * 2, out=y2, relu=True), y2))
    for call, out in cases:
        out.fill_(-7.0)
        call()
        torch.cuda.synchronize()
        ref = out.clone()
        for fill in (0.0, -7.0, 3.0, 0.0):
            out.fill_(fill)
            call()
            torch.cuda.synchronize()
            assert torch.equal(out, ref)
        assert float(ref.min()) >= 0.0
