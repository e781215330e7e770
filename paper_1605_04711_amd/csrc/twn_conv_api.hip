// C-ABI entry points of the forward block (Eq. 2; Alg. 1 step 8) and of the
// straight-through backward (Alg. 1 steps 9-10): host-side validation and the
// translation of descriptors into kernel launches.
#include "twn_kernels.h"

using namespace twn;

namespace {

int out_dim(int h, int r, int stride, int pad, int dil) {
    const int64_t eff = static_cast<int64_t>(h) + 2LL * pad - static_cast<int64_t>(dil) * (r - 1) - 1;
    if (eff < 0) return 0;
    return static_cast<int>(eff / stride + 1);
}

int32_t check_conv_desc(const twn_conv_desc* d, int* P, int* Q) {
    if (!d) return TWN_ERR_NULL;
    if (d->N <= 0 || d->H <= 0 || d->W <= 0 || d->C <= 0 || d->O <= 0 || d->R <= 0 || d->S <= 0)
        return TWN_ERR_SHAPE;
    if (d->stride_h <= 0 || d->stride_w <= 0 || d->dil_h <= 0 || d->dil_w <= 0 || d->pad_h < 0 || d->pad_w < 0)
        return TWN_ERR_SHAPE;
    if (d->alpha_groups < 1 || d->O % d->alpha_groups != 0) return TWN_ERR_SHAPE;
    *P = out_dim(d->H, d->R, d->stride_h, d->pad_h, d->dil_h);
    *Q = out_dim(d->W, d->S, d->stride_w, d->pad_w, d->dil_w);
    if (*P <= 0 || *Q <= 0) return TWN_ERR_SHAPE;
    const int64_t K = static_cast<int64_t>(d->R) * d->S * d->C;
    const int64_t KT = static_cast<int64_t>(d->R) * d->S * d->O;
    if (K >= (1LL << 30) || KT >= (1LL << 30)) return TWN_ERR_SHAPE;
    if (static_cast<int64_t>(d->N) * d->H * d->W >= (1LL << 31)) return TWN_ERR_SHAPE;
    if (static_cast<int64_t>(d->N) * (*P) * (*Q) >= (1LL << 31)) return TWN_ERR_SHAPE;
    if (d->H >= (1 << 24) || d->W >= (1 << 24)) return TWN_ERR_SHAPE;
    return TWN_OK;
}

int32_t check_dtype(int32_t t) { return (t == TWN_F32 || t == TWN_BF16) ? TWN_OK : TWN_ERR_UNSUPPORTED; }

int32_t check_variant(int32_t variant, int32_t x_dtype) {
    switch (variant) {
        case TWN_VAR_BF16_POSTSCALE: return x_dtype == TWN_BF16 ? TWN_OK : TWN_ERR_UNSUPPORTED;
        case TWN_VAR_FP32: return x_dtype == TWN_F32 ? TWN_OK : TWN_ERR_UNSUPPORTED;
        case TWN_VAR_BF16_ALPHA_LDS:
        case TWN_VAR_I8_STORED_POSTSCALE:
        case TWN_VAR_BF16_SIGN1_POSTSCALE:
        case TWN_VAR_ADDSUB_SPARSE: return x_dtype == TWN_BF16 ? TWN_OK : TWN_ERR_UNSUPPORTED;
        default: return TWN_ERR_UNSUPPORTED;
    }
}

// Output / residual alignment: rows whose channel count and leading dimension are multiples of 8 are written
// with 16-byte stores (and the residual read with 8-byte loads); other shapes are accessed element by element.
int32_t check_out_align(int32_t y_dtype, int64_t NC, int64_t ldy, const void* Y, const void* residual) {
    const size_t elem = (y_dtype == TWN_F32) ? 4 : 2;
    const bool vec = (NC % 8 == 0) && (ldy % 8 == 0);
    if (!aligned(Y, vec ? 16 : elem)) return TWN_ERR_ALIGN;
    if (residual && !aligned(residual, vec ? 16 : elem)) return TWN_ERR_ALIGN;
    return TWN_OK;
}

void set_epilogue(GatherGemm& g, const twn_epilogue* ep) {
    g.scale = ep ? ep->scale : nullptr;
    g.shift = ep ? ep->shift : nullptr;
    g.residual = ep ? ep->residual : nullptr;
    g.relu = ep ? (ep->relu != 0) : 0;
}

size_t splitk_bytes(const GatherGemm& g, int variant) {
    if (variant == TWN_VAR_FP32) {
        const int32_t splits = gather_gemm_fp32_splits(g);
        return splits > 1 ? static_cast<size_t>(splits) * static_cast<size_t>(g.M) * g.NC * sizeof(double) : 0;
    }
    if (variant != TWN_VAR_BF16_POSTSCALE) return 0;   // the other variants never split K
    const int32_t splits = gather_gemm_splits(g);
    return splits > 1 ? static_cast<size_t>(splits) * static_cast<size_t>(g.M) * g.NC * sizeof(float) : 0;
}

// Attaches the split-K workspace (if the problem uses one) and launches.
int32_t dispatch(GatherGemm& g, int variant, void* workspace, size_t workspace_bytes, hipStream_t st,
                 bool allow_split = true) {
    if (variant == TWN_VAR_FP32) {
        g.splits = allow_split ? gather_gemm_fp32_splits(g) : 1;
        g.partial = nullptr;
        if (g.splits > 1) {
            const size_t need = static_cast<size_t>(g.splits) * static_cast<size_t>(g.M) * g.NC * sizeof(double);
            if (!workspace || workspace_bytes < need || !aligned(workspace, 16)) return TWN_ERR_WORKSPACE;
            g.partial = static_cast<float*>(workspace);
        }
        return launch_gather_gemm_fp32(g, st);
    }
    if (variant == TWN_VAR_ADDSUB_SPARSE) {
        g.splits = 1;
        g.partial = nullptr;
        return launch_conv_addsub(g, st);
    }
    if (variant != TWN_VAR_BF16_POSTSCALE) {
        if (variant == TWN_VAR_I8_STORED_POSTSCALE && (g.K % 8 != 0 || !aligned(g.Wq, 8))) return TWN_ERR_UNSUPPORTED;
        if (variant == TWN_VAR_BF16_SIGN1_POSTSCALE) {
            if (!aligned(g.Wq, 16)) return TWN_ERR_ALIGN;
            g.wpr = static_cast<int32_t>(twn_packed1_words_per_row(g.K));    // 1-bit rows
        }
        g.splits = 1;
        g.partial = nullptr;
        return launch_gather_gemm_mfma(g, variant, st);
    }
    g.splits = allow_split ? gather_gemm_splits(g) : 1;
    g.partial = nullptr;
    if (g.splits > 1) {
        const size_t need = static_cast<size_t>(g.splits) * static_cast<size_t>(g.M) * g.NC * sizeof(float);
        if (!workspace || workspace_bytes < need || !aligned(workspace, 16)) return TWN_ERR_WORKSPACE;
        g.partial = static_cast<float*>(workspace);
    }
    return launch_gather_gemm_mfma(g, variant, st);
}

void fill_gemm(GatherGemm& g, const twn_gemm_desc* d) {
    g.M = d->M;
    g.xs = d->ldx ? d->ldx : d->K;
    g.ldy = d->ldy ? d->ldy : d->N;
    g.IH = g.IW = g.OH = g.OW = 1;
    g.IC = d->K;
    g.NC = d->N;
    g.R = g.S = 1;
    g.sh = g.sw = g.dh = g.dw = g.divh = g.divw = 1;
    g.ph = g.pw = 0;
    g.K = d->K;
    g.wpr = static_cast<int32_t>(twn_packed_words_per_row(d->K));
    g.rows_per_group = d->N / d->alpha_groups;
    g.y_f32 = (d->y_dtype == TWN_F32);
    g.plain_gemm = 1;
}

void fill_conv_fwd(GatherGemm& g, const twn_conv_desc* d, int P, int Q) {
    g.M = static_cast<int64_t>(d->N) * P * Q;
    g.xs = d->C;
    g.ldy = d->O;
    g.IH = d->H;
    g.IW = d->W;
    g.IC = d->C;
    g.OH = P;
    g.OW = Q;
    g.NC = d->O;
    g.R = d->R;
    g.S = d->S;
    g.sh = d->stride_h;
    g.sw = d->stride_w;
    g.ph = d->pad_h;
    g.pw = d->pad_w;
    g.dh = d->dil_h;
    g.dw = d->dil_w;
    g.divh = g.divw = 1;
    g.K = d->R * d->S * d->C;
    g.wpr = static_cast<int32_t>(twn_packed_words_per_row(g.K));
    g.rows_per_group = d->O / d->alpha_groups;
    g.y_f32 = (d->y_dtype == TWN_F32);
    g.plain_gemm = (d->R == 1 && d->S == 1 && d->stride_h == 1 && d->stride_w == 1 && d->pad_h == 0 &&
                    d->pad_w == 0);
}

// dX = gather over dY: row (n,h,w), k = (r,s,o):
//   p = (h + ph - r*dh)/sh when divisible, q likewise; weights = transposed packed copy.
void fill_conv_bwd_data(GatherGemm& g, const twn_conv_desc* d, int P, int Q) {
    g.M = static_cast<int64_t>(d->N) * d->H * d->W;
    g.xs = d->O;
    g.ldy = d->C;
    g.IH = P;
    g.IW = Q;
    g.IC = d->O;
    g.OH = d->H;
    g.OW = d->W;
    g.NC = d->C;
    g.R = d->R;
    g.S = d->S;
    g.sh = g.sw = 1;
    g.ph = -d->pad_h;
    g.pw = -d->pad_w;
    g.dh = -d->dil_h;
    g.dw = -d->dil_w;
    g.divh = d->stride_h;
    g.divw = d->stride_w;
    g.K = d->R * d->S * d->O;
    g.wpr = static_cast<int32_t>(twn_packed_words_per_row(g.K));
    g.rows_per_group = d->C;
    g.y_f32 = (d->y_dtype == TWN_F32);
    g.plain_gemm = (d->R == 1 && d->S == 1 && d->stride_h == 1 && d->stride_w == 1 && d->pad_h == 0 &&
                    d->pad_w == 0);
}

// ---- small-C forward path (C <= 4, bf16, dilation 1): geometry of the padded copy ----
struct SmallC {
    int Hp, Wp, Sp;
    size_t x_bytes, w_bytes;
};

bool small_c(const twn_conv_desc* d, SmallC* sc) {
    if (d->variant != TWN_VAR_BF16_POSTSCALE || d->x_dtype != TWN_BF16) return false;
    if (d->C > 4 || d->dil_h != 1 || d->dil_w != 1) return false;
    sc->Sp = (d->S + 1) & ~1;
    sc->Hp = d->H + 2 * d->pad_h;
    sc->Wp = d->W + 2 * d->pad_w + (sc->Sp - d->S);
    sc->x_bytes = round_up(static_cast<size_t>(d->N) * sc->Hp * sc->Wp * 4 * sizeof(uint16_t), 256);
    sc->w_bytes = round_up(twn_packed_bytes(d->O, static_cast<int64_t>(d->R) * sc->Sp * 4), 256);
    return static_cast<int64_t>(d->N) * sc->Hp * sc->Wp < (1LL << 31);
}

void fill_conv_fwd_small_c(GatherGemm& g, const twn_conv_desc* d, const SmallC& sc, int P, int Q) {
    fill_conv_fwd(g, d, P, Q);
    g.xs = 4;                    // elements per padded pixel
    g.IH = sc.Hp;
    g.IW = sc.Wp;
    g.IC = 8;                    // one 16-byte chunk = two adjacent taps x 4 channels
    g.S = sc.Sp / 2;
    g.ph = g.pw = 0;             // the border is part of the copy
    g.dw = 2;                    // chunk j of a filter row starts 2 pixels after chunk j-1
    g.K = d->R * sc.Sp * 4;
    g.wpr = static_cast<int32_t>(twn_packed_words_per_row(g.K));
    g.plain_gemm = 0;
    g.chunk_gather = 1;
}

// Backward-data over dY scaled by several alphas: two bf16 terms per value, side by side as twice the channels.  From 1 GiB of
// dY on they make a tensor that the persistent kernels and buffer loads do not take; one contraction through per-lane
// pointers is still faster than two through descriptors (dY of 1.5 GiB, 192 x 64 x 64, 1024 filters of 3x3 over 256 channels: 8.2 ->
// 7.1 ms; the same with stride 2 and 128 x 128 pixels: 9.8 -> 7.7).
void two_terms(GatherGemm& g) {
    g.xs *= 2;
    g.IC *= 2;
    g.K *= 2;
    g.wpr = static_cast<int32_t>(twn_packed_words_per_row(g.K));
}

// Strided backward-data as stride-1 problems, one per residue class (a, b) of the output pixels
// (h = a + sh*u, w = b + sw*v): the taps that reach the class are r = r0 + jr*sh with r0 = (a + pad_h) % sh, the
// coordinate read is p = u + (a + pad_h - r0)/sh - jr, i.e. an undivided gather with dilation -1.  Used for
// dilation 1, O % 8 == 0, C % 8 == 0, stride products up to 4.
struct DxClasses {
    int count;                  // classes that have taps
    bool any_empty;             // some class has none: those pixels of dX are zero
    GatherGemm g[4];
    DxClassTable tb;
    int64_t code_words;
};

bool strided_dx_classes(const twn_conv_desc* d, int P, int Q, bool two, DxClasses* out) {
    const int sh = d->stride_h, sw = d->stride_w;
    if (sh * sw <= 1 || sh * sw > 4 || d->dil_h != 1 || d->dil_w != 1 || d->O % 8 != 0 || d->C % 8 != 0 ||
        d->variant != TWN_VAR_BF16_POSTSCALE || d->x_dtype != TWN_BF16)
        return false;
    // Launches of the large kernels (whole slabs per tap) only pay when each class still has enough pixels to fill the chip;
    // below that, and for taps of no whole slabs, the classes have to fit one launch of the few-tile kernel.
    const bool enough = static_cast<int64_t>(d->N) * ((d->H + sh - 1) / sh) * ((d->W + sw - 1) / sw) >=
                        env_int(Env::DX_CLASS_MIN_PIXELS, 2048);
    if (!enough && env_set(Env::DX_CLASS_MIN_PIXELS)) return false;
    out->count = 0;
    out->any_empty = false;
    out->code_words = 0;
    for (int a = 0; a < sh; ++a)
        for (int b = 0; b < sw; ++b) {
            const int U = (d->H - a + sh - 1) / sh, V = (d->W - b + sw - 1) / sw;
            if (U <= 0 || V <= 0) continue;         // no pixel in this class
            const int r0 = (a + d->pad_h) % sh, s0 = (b + d->pad_w) % sw;
            const int nr = r0 < d->R ? (d->R - r0 + sh - 1) / sh : 0, ns = s0 < d->S ? (d->S - s0 + sw - 1) / sw : 0;
            if (nr == 0 || ns == 0) {
                out->any_empty = true;
                continue;
            }
            const int k = out->count++;
            GatherGemm& g = out->g[k];
            g = GatherGemm{};
            fill_conv_bwd_data(g, d, P, Q);
            g.M = static_cast<int64_t>(d->N) * U * V;
            g.OH = U;
            g.OW = V;
            g.R = nr;
            g.S = ns;
            g.ph = -((a + d->pad_h - r0) / sh);
            g.pw = -((b + d->pad_w - s0) / sw);
            g.dh = g.dw = -1;
            g.divh = g.divw = 1;
            g.K = nr * ns * d->O;
            g.wpr = static_cast<int32_t>(twn_packed_words_per_row(g.K));
            if (two) two_terms(g);
            g.plain_gemm = 0;
            g.orU = U; g.orV = V; g.orH = d->H; g.orW = d->W;
            g.ora = a; g.orb = b; g.orsh = sh; g.orsw = sw;
            out->tb.r0[k] = r0; out->tb.nr[k] = nr; out->tb.s0[k] = s0; out->tb.ns[k] = ns;
            out->tb.wpr[k] = g.wpr;
            out->tb.first_word[k] = out->code_words;
            out->code_words += static_cast<int64_t>(d->C) * g.wpr;
        }
    out->tb.count = out->count;
    out->tb.sh = sh;
    out->tb.sw = sw;
    for (int k = out->count; k <= 4; ++k) out->tb.first_word[k] = out->code_words;
    if (out->count == 0 || (enough && d->O % 64 == 0)) return out->count > 0;
    if (conv_small_tile(out->g, out->count) == 0) return false;
    // Against all taps in one problem, most of whose products are zeros: a slab of a tile costs 0.3 us of a CU and 0.16 us of the
    // chain of its workgroup, the launch that gathers the codes 3.5 (several alphas have it anyway).  (us, dX alone, all taps ->
    // classes: 5x45x61 pixels, 72 filters 5x5/2 over 40 channels 16.8 -> 15.1; 5x27x25, 200, 5x5/2 over 40, several alphas
    // 37.6 -> 17.3; 3x14x14, 512, 3x3/2 over 256, several alphas 28.6 -> 12.5, one alpha 14.6 -> 9.5)
    auto cost = [](const GatherGemm* g, int count) {
        double slabs = 0.0, chain = 0.0;
        for (int k = 0; k < count; ++k) {
            const int kt = k_slabs(g[k].K);
            slabs += static_cast<double>((g[k].M + 31) / 32) * ((g[k].NC + 31) / 32) * kt;
            if (0.16 * kt > chain) chain = 0.16 * kt;
        }
        const double chip = 0.3 * slabs / 256.0;
        return chip > chain ? chip : chain;
    };
    GatherGemm all{};
    fill_conv_bwd_data(all, d, P, Q);
    if (two) two_terms(all);
    return conv_small_tile(&all, 1) == 0 || cost(&all, 1) > cost(out->g, out->count) + (two ? 0.0 : 3.5);
}

// Workspace of backward-data, in this order: gathered codes (residue classes; several alphas: repeated for the second
// term), dY scaled by several alphas as two bf16 terms, one float (the unit alpha), split-K partials of the contraction.
struct DxPlan {
    bool classes;           // cl describes the problem, else `g`
    bool two;               // several alphas: two terms per value of dY
    DxClasses cl;
    GatherGemm g;           // all taps in one problem (also when classes is set: the fallback without a workspace)
    DxClassTable tb;        // its codes, all taps as one class
    size_t code_bytes, scaled_bytes, one_bytes, split_bytes;
    size_t bytes() const { return code_bytes + scaled_bytes + one_bytes + split_bytes; }
};

// `inside`: several alphas stay with the codes (alpha_in of the problems) instead of making two terms of dY.
void plan_dx(const twn_conv_desc* d, int P, int Q, DxPlan* p, bool allow_classes, bool inside = false) {
    p->two = d->alpha_groups > 1 && !inside;
    p->classes = allow_classes && strided_dx_classes(d, P, Q, p->two, &p->cl);
    p->g = GatherGemm{};
    fill_conv_bwd_data(p->g, d, P, Q);
    p->code_bytes = p->scaled_bytes = p->one_bytes = p->split_bytes = 0;
    if (p->two) {
        two_terms(p->g);
        p->tb = DxClassTable{};
        p->tb.count = p->tb.sh = p->tb.sw = 1;
        p->tb.nr[0] = d->R;
        p->tb.ns[0] = d->S;
        p->tb.wpr[0] = p->g.wpr;
        for (int k = 1; k <= 4; ++k) p->tb.first_word[k] = static_cast<int64_t>(d->C) * p->g.wpr;
        p->scaled_bytes = round_up(static_cast<size_t>(d->N) * P * Q * d->O * 2 * sizeof(uint16_t), 256);
        p->one_bytes = 256;
    }
    const int64_t words = p->classes ? p->cl.code_words : (p->two ? p->tb.first_word[1] : 0);
    p->code_bytes = round_up(static_cast<size_t>(words) * sizeof(uint32_t), 256);
    if (!p->classes) p->split_bytes = splitk_bytes(p->g, d->variant);      // classes are never split
}

WgShape taps_shape(const twn_conv_desc* d, int P, int Q) {
    return WgShape{d->N, d->H, d->W, d->C, d->O, d->R, d->S, P, Q, d->stride_h, d->stride_w, d->dil_h, d->dil_w};
}

// Three-channel first layers have a kernel of their own, unless an override shapes the general one.
FirstGradPlan first_grad_plan(const twn_conv_desc* d, int P, int Q) {
    if (env_int(Env::FIRST, 1) == 0 || env_int(Env::BUFLOAD, 1) == 0 || env_set(Env::WG_BLOCKS) || env_set(Env::WG_KS) ||
        env_set(Env::WG_ROWS_SPLITS) || env_set(Env::WG_XCD))
        return FirstGradPlan{};
    return plan_first_weight_grad(taps_shape(d, P, Q));
}
size_t first_grad_bytes(const twn_conv_desc* d, const FirstGradPlan& f) {
    return f.use ? static_cast<size_t>(f.splits) * d->O * f.J * sizeof(float) : 0;
}

// The least workspace of a weight gradient: [padded copy of X in first-layer mode] + split partials + bias partials.
size_t weight_grad_bytes(const twn_conv_desc* d, int P, int Q) {
    SmallC sc;
    if (small_c(d, &sc) && d->O % 8 == 0) {
        const int64_t Jp = static_cast<int64_t>(d->R) * sc.Sp * 4;
        const int64_t splits =
            route_weight_grad(WgShape{d->N, sc.Hp, sc.Wp, 8, d->O, d->R, sc.Sp / 2, P, Q, d->stride_h, d->stride_w, 1, 2}, true).splits;
        return sc.x_bytes + static_cast<size_t>((splits * d->O * Jp + 64LL * d->O) * sizeof(float));
    }
    const int64_t J = static_cast<int64_t>(d->R) * d->S * d->C;
    const int64_t splits = route_weight_grad(taps_shape(d, P, Q), false).splits;
    return static_cast<size_t>((splits * d->O * J + 64LL * d->O) * sizeof(float));
}

// Filter counts that are no multiple of 8 (a classifier's ten, a detection head's 84): 16-byte chunks of dY do not exist, and both
// gradients would run in the kernels that load element by element (bound by their loads, one 2-byte element each).  One launch
// pads dY, codes and alphas to the next multiple of 8 in the workspace, the layer is that of so many filters (its kernels and
// their ranges too), and dW leaves the added ones out.  (us of dX + dW, before -> with the launch: 128 pixels 1024 -> 10
// 29.4 -> 14.9; 64x40x40x16 -> 10, 3x3 135 -> 33; 5x20x22x512 -> 10, 7x7 269 -> 38; 64x38x38x512 -> 84, 3x3 1999 -> 213;
// 64x112x112x3 -> 10, 3x3, one alpha per filter 935 -> 124; 3 pixels 1024 -> 10 19.3 -> 13.0, but dX alone there 6.5 -> 7.8
// against 14.6 -> 7.6 at 128 pixels and 6.9 -> 6.5 at 64: below 64 pixels only with dW.)
struct FilterPadPlan {
    bool use;
    twn_conv_desc d;            // the padded layer
    size_t dy_bytes, code_bytes, alpha_bytes;
    size_t bytes() const { return dy_bytes + code_bytes + alpha_bytes; }
};
FilterPadPlan plan_filter_pad(const twn_conv_desc* d, int P, int Q) {
    FilterPadPlan p{};
    if (d->O % 8 == 0 || d->variant != TWN_VAR_BF16_POSTSCALE || d->x_dtype != TWN_BF16 ||
        (d->alpha_groups != 1 && d->alpha_groups != d->O))
        return p;
    p.d = *d;
    p.d.O = (d->O + 7) & ~7;
    p.d.alpha_groups = d->alpha_groups == 1 ? 1 : p.d.O;
    const int64_t pixels = static_cast<int64_t>(d->N) * P * Q, kt = static_cast<int64_t>(d->R) * d->S * p.d.O;
    const int64_t dw = static_cast<int64_t>(p.d.O) * d->R * (d->S + 1) * (d->C < 8 ? 8 : d->C);
    // well inside the limits of every kernel below, so that nothing is refused for the filters added
    if (kt >= (1LL << 29) || pixels * p.d.O >= (1LL << 30) || dw >= (1LL << 28)) return p;
    p.dy_bytes = round_up(static_cast<size_t>(pixels) * p.d.O * sizeof(uint16_t), 256);
    p.code_bytes = round_up(twn_packed_bytes(d->C, kt), 256);
    p.alpha_bytes = round_up(static_cast<size_t>(p.d.O) * sizeof(float), 256);
    p.use = true;
    return p;
}

}  // namespace

extern "C" size_t twn_gemm_fwd_workspace_bytes(const twn_gemm_desc* d) {
    if (!d || d->M <= 0 || d->N <= 0 || d->K <= 0 || d->alpha_groups < 1) return 0;
    GatherGemm g{};
    fill_gemm(g, d);
    return splitk_bytes(g, d->variant);
}

extern "C" int32_t twn_gemm_fwd(const twn_gemm_desc* d, const void* X, const void* weights,
                                const float* alpha, const twn_epilogue* ep, void* Y,
                                void* workspace, size_t workspace_bytes, void* stream) {
    if (!d || !X || !weights || !alpha || !Y) return TWN_ERR_NULL;
    if (d->M <= 0 || d->N <= 0 || d->K <= 0 || d->M >= (1LL << 31) || d->K >= (1 << 30)) return TWN_ERR_SHAPE;
    if (d->alpha_groups < 1 || d->N % d->alpha_groups != 0) return TWN_ERR_SHAPE;
    int32_t rc = check_dtype(d->x_dtype);
    if (rc == TWN_OK) rc = check_dtype(d->y_dtype);
    if (rc == TWN_OK) rc = check_variant(d->variant, d->x_dtype);
    if (rc != TWN_OK) return rc;
    const int64_t ldx = d->ldx ? d->ldx : d->K;
    const int64_t ldy = d->ldy ? d->ldy : d->N;
    if (ldx < d->K || ldy < d->N) return TWN_ERR_SHAPE;
    if (!aligned(weights, 16)) return TWN_ERR_ALIGN;
    if (d->x_dtype == TWN_BF16 && !aligned(X, 2)) return TWN_ERR_ALIGN;
    if (d->x_dtype == TWN_F32 && !aligned(X, 4)) return TWN_ERR_ALIGN;
    if (d->x_dtype == TWN_BF16 && d->K % 8 == 0 && ldx % 8 == 0 && !aligned(X, 16)) return TWN_ERR_ALIGN;
    rc = check_out_align(d->y_dtype, d->N, ldy, Y, ep ? ep->residual : nullptr);
    if (rc != TWN_OK) return rc;

    GatherGemm g{};
    g.X = X;
    g.Wq = weights;
    g.alpha = alpha;
    set_epilogue(g, ep);
    g.Y = Y;
    fill_gemm(g, d);
    return dispatch(g, d->variant, workspace, workspace_bytes, as_stream(stream));
}

extern "C" size_t twn_conv2d_fwd_workspace_bytes(const twn_conv_desc* d) {
    int P, Q;
    if (check_conv_desc(d, &P, &Q) != TWN_OK) return 0;
    GatherGemm g{};
    SmallC sc;
    if (small_c(d, &sc)) {
        fill_conv_fwd_small_c(g, d, sc, P, Q);
        return sc.x_bytes + sc.w_bytes + splitk_bytes(g, d->variant);
    }
    fill_conv_fwd(g, d, P, Q);
    return splitk_bytes(g, d->variant);
}

extern "C" int32_t twn_conv2d_fwd(const twn_conv_desc* d, const void* X, const void* weights,
                                  const float* alpha, const twn_epilogue* ep, void* Y,
                                  void* workspace, size_t workspace_bytes, void* stream) {
    int P, Q;
    int32_t rc = check_conv_desc(d, &P, &Q);
    if (rc != TWN_OK) return rc;
    if (!X || !weights || !alpha || !Y) return TWN_ERR_NULL;
    rc = check_dtype(d->x_dtype);
    if (rc == TWN_OK) rc = check_dtype(d->y_dtype);
    if (rc == TWN_OK) rc = check_variant(d->variant, d->x_dtype);
    if (rc != TWN_OK) return rc;
    if (!aligned(weights, 16)) return TWN_ERR_ALIGN;
    if (d->x_dtype == TWN_BF16 && !aligned(X, (d->C % 8 == 0) ? 16 : 2)) return TWN_ERR_ALIGN;
    if (d->x_dtype == TWN_F32 && !aligned(X, 4)) return TWN_ERR_ALIGN;
    rc = check_out_align(d->y_dtype, d->O, d->O, Y, ep ? ep->residual : nullptr);
    if (rc != TWN_OK) return rc;

    GatherGemm g{};
    g.X = X;
    g.Wq = weights;
    g.alpha = alpha;
    set_epilogue(g, ep);
    g.Y = Y;
    if (d->variant == TWN_VAR_BF16_POSTSCALE && d->x_dtype == TWN_BF16 && d->y_dtype == TWN_BF16 && d->C == 3 &&
        d->dil_h == 1 && d->dil_w == 1 && env_int(Env::FIRST, 1) != 0) {
        // three-channel first layer: persistent kernel with the input patch widened to four channels in LDS and
        // the expanded weights resident in registers (no workspace, no preparation launch)
        FirstLayer f{};
        f.X = static_cast<const uint16_t*>(X);
        f.Wq = static_cast<const uint32_t*>(weights);
        f.alpha = alpha;
        f.scale = g.scale;
        f.shift = g.shift;
        f.residual = static_cast<const uint16_t*>(g.residual);
        f.Y = static_cast<uint16_t*>(Y);
        f.N = d->N; f.H = d->H; f.W = d->W; f.C = d->C; f.O = d->O; f.R = d->R; f.S = d->S;
        f.sh = d->stride_h; f.sw = d->stride_w; f.ph = d->pad_h; f.pw = d->pad_w; f.P = P; f.Q = Q;
        f.rows_per_group = d->O / d->alpha_groups;
        f.relu = g.relu;
        if (conv_first_applicable(f)) return launch_conv_first(f, as_stream(stream));
    }
    SmallC sc;
    if (small_c(d, &sc)) {
        // first-layer path: padded 4-channel copy of X and re-ordered codes live in the workspace
        fill_conv_fwd_small_c(g, d, sc, P, Q);
        const size_t head = sc.x_bytes + sc.w_bytes;
        if (!workspace || workspace_bytes < head + splitk_bytes(g, d->variant) || !aligned(workspace, 256))
            return TWN_ERR_WORKSPACE;
        hipStream_t st = as_stream(stream);
        uint16_t* Xp = static_cast<uint16_t*>(workspace);
        uint32_t* Wp = reinterpret_cast<uint32_t*>(static_cast<unsigned char*>(workspace) + sc.x_bytes);
        rc = launch_pad_repack_c4(static_cast<const uint16_t*>(X), d->N, d->H, d->W, d->C, d->pad_h, d->pad_w, sc.Hp,
                                  sc.Wp, Xp, static_cast<const uint32_t*>(weights), d->O, d->R, d->S, sc.Sp, Wp, st);
        if (rc != TWN_OK) return rc;
        g.X = Xp;
        g.Wq = Wp;
        return dispatch(g, d->variant, static_cast<unsigned char*>(workspace) + head, workspace_bytes - head, st);
    }
    fill_conv_fwd(g, d, P, Q);
    return dispatch(g, d->variant, workspace, workspace_bytes, as_stream(stream));
}

// One problem of twn_conv2d_fwd_pair: the checks of twn_conv2d_fwd for the product variant on bf16 tensors whose
// channel count is a multiple of 8 (no first-layer paths), then the problem descriptor.
static int32_t build_pair_problem(const twn_conv_desc* d, const void* X, const void* weights, const float* alpha,
                                  const twn_epilogue* ep, void* Y, GatherGemm* g) {
    int P, Q;
    int32_t rc = check_conv_desc(d, &P, &Q);
    if (rc != TWN_OK) return rc;
    if (!X || !weights || !alpha || !Y) return TWN_ERR_NULL;
    if (d->variant != TWN_VAR_BF16_POSTSCALE || d->x_dtype != TWN_BF16 || d->y_dtype != TWN_BF16 || d->C % 8 != 0)
        return TWN_ERR_UNSUPPORTED;
    if (!aligned(weights, 16) || !aligned(X, 16)) return TWN_ERR_ALIGN;
    rc = check_out_align(d->y_dtype, d->O, d->O, Y, ep ? ep->residual : nullptr);
    if (rc != TWN_OK) return rc;
    *g = GatherGemm{};
    g->X = X;
    g->Wq = weights;
    g->alpha = alpha;
    set_epilogue(*g, ep);
    g->Y = Y;
    fill_conv_fwd(*g, d, P, Q);
    g->splits = 1;
    g->partial = nullptr;
    return TWN_OK;
}

// Whether two problems over one input give the results of two calls when they run at the same time: neither writes what
// the other reads or writes (a second problem whose residual is the first one's output has to wait for it).
static bool pair_independent(const GatherGemm* g) {
    struct Range {
        uintptr_t at;
        uint64_t bytes;
        bool meets(const Range& o) const { return at != 0 && o.at != 0 && at < o.at + o.bytes && o.at < at + bytes; }
    };
    auto range = [](const void* p, int64_t values) { return Range{reinterpret_cast<uintptr_t>(p), static_cast<uint64_t>(values) * 2}; };
    const Range x = range(g[0].X, g[0].M / (static_cast<int64_t>(g[0].OH) * g[0].OW) * g[0].IH * g[0].IW * g[0].xs);
    Range y[2], res[2];
    for (int i = 0; i < 2; ++i) {
        y[i] = range(g[i].Y, g[i].M * g[i].ldy);
        res[i] = range(g[i].residual, g[i].M * g[i].ldy);
    }
    return !y[0].meets(y[1]) && !y[0].meets(res[1]) && !y[1].meets(res[0]) && !y[0].meets(x) && !y[1].meets(x);
}

extern "C" int32_t twn_conv2d_fwd_pair(const twn_conv_desc* d0, const twn_conv_desc* d1, const void* X,
                                       const void* weights0, const float* alpha0, const twn_epilogue* ep0, void* Y0,
                                       const void* weights1, const float* alpha1, const twn_epilogue* ep1, void* Y1,
                                       void* stream) {
    if (!d0 || !d1) return TWN_ERR_NULL;
    if (d0->N != d1->N || d0->H != d1->H || d0->W != d1->W || d0->C != d1->C) return TWN_ERR_SHAPE;
    GatherGemm g[2];
    int32_t rc = build_pair_problem(d0, X, weights0, alpha0, ep0, Y0, &g[0]);
    if (rc == TWN_OK) rc = build_pair_problem(d1, X, weights1, alpha1, ep1, Y1, &g[1]);
    if (rc != TWN_OK) return rc;
    hipStream_t st = as_stream(stream);
    const int pair_knob = env_int(Env::FWD_PAIR, 1);          // 0: never one launch, 2: whenever the tiles agree
    const bool together = pair_knob != 0 && pair_independent(g);
    const int small = together ? conv_small_tile(g, 2) : 0;
    if (small != 0) return launch_conv_small(g, 2, small, st);
    const int t0 = gather_gemm_dma_tile(g[0], true), t1 = gather_gemm_dma_tile(g[1], true);
    // One launch pays while the reduction is short: with more than 24 slabs per tile the persistent kernels with load
    // waves win back more than the saved launch (ResNet-18 b64 block heads, two launches -> one: 128 filters, K = 576:
    // 23.4 -> 19.1 us; 256 filters, K = 1152: 17.9 -> 15.9 us; 512 filters, K = 2304: 18.2 -> 19.3 us).
    const int64_t kmax = g[0].K > g[1].K ? g[0].K : g[1].K;
    if (together && t0 != 0 && t0 == t1 && (pair_knob == 2 || kmax <= 1536)) {
        rc = launch_gather_gemm_dma_batch(g, 2, t0, st);
        if (rc != TWN_ERR_UNSUPPORTED) return rc;
    }
    // dependent problems, different tile shapes or no build for the pair: one after the other, as two twn_conv2d_fwd calls
    // without a workspace
    rc = dispatch(g[0], d0->variant, nullptr, 0, st, false);
    if (rc != TWN_OK) return rc;
    return dispatch(g[1], d1->variant, nullptr, 0, st, false);
}

extern "C" size_t twn_conv2d_bwd_ste_workspace_bytes(const twn_conv_desc* d) {
    int P, Q;
    if (check_conv_desc(d, &P, &Q) != TWN_OK) return 0;
    // the data-gradient split-K partials and the weight-gradient partials use the workspace one after the other
    DxPlan p;
    plan_dx(d, P, Q, &p, false);
    size_t a = p.bytes();
    plan_dx(d, P, Q, &p, true);
    if (p.bytes() > a) a = p.bytes();
    const size_t b = weight_grad_bytes(d, P, Q);
    if (b > a) a = b;
    // more than the least the call takes: a three-channel layer's own kernel, and the padded copies
    SmallC sc;
    const size_t f = small_c(d, &sc) && d->O % 8 == 0 ? first_grad_bytes(d, first_grad_plan(d, P, Q)) : 0;
    if (f > a) a = f;
    const FilterPadPlan pad = plan_filter_pad(d, P, Q);
    const size_t c = pad.use ? pad.bytes() + twn_conv2d_bwd_ste_workspace_bytes(&pad.d) : 0;
    return a > c ? a : c;
}

// Preparation of residue classes: their codes, one copy, and the clearing of dX where a class has no taps.
static DxPrep class_prep(const twn_conv_desc* d, const DxClasses& cl, const uint32_t* packed_T, uint32_t* codes, void* dX) {
    DxPrep q{};
    q.O = d->O;
    q.packed_T = packed_T;
    q.C = d->C;
    q.wprT = static_cast<int32_t>(twn_packed_words_per_row(static_cast<int64_t>(d->R) * d->S * d->O));
    q.S = d->S;
    q.terms = 1;
    q.tb = cl.tb;
    q.codes = codes;
    if (cl.any_empty) {
        q.zero = dX;
        q.zero16 = static_cast<int64_t>(d->N) * d->H * d->W * d->C * (d->y_dtype == TWN_F32 ? 4 : 2) / 16;
    }
    return q;
}

// dX of the straight-through backward: one contraction over dY (one per residue class of a strided layer).
static int32_t data_gradient(const twn_conv_desc* d, int P, int Q, const void* dY, const uint32_t* packed_T, const float* alpha,
                             void* dX, void* workspace, size_t workspace_bytes, hipStream_t st) {
    int32_t rc = TWN_OK;
    DxPlan p;
    plan_dx(d, P, Q, &p, env_int(Env::DX_CLASSES, 1) != 0);
    if (p.classes && !(workspace && workspace_bytes >= p.bytes() && aligned(workspace, 256) && aligned(dX, 16)))
        plan_dx(d, P, Q, &p, false);            // no room for the gathered codes: the generic gather
    if (p.two && (!workspace || workspace_bytes < p.bytes() || !aligned(workspace, 256))) return TWN_ERR_WORKSPACE;
    unsigned char* ws = static_cast<unsigned char*>(workspace);
    uint32_t* codes = static_cast<uint32_t*>(workspace);
    uint16_t* scaled = reinterpret_cast<uint16_t*>(ws + p.code_bytes);
    float* one = reinterpret_cast<float*>(ws + p.code_bytes + p.scaled_bytes);
    const size_t head = p.code_bytes + p.scaled_bytes + p.one_bytes;
    const int count = p.classes ? p.cl.count : 1;
    GatherGemm* gs = p.classes ? p.cl.g : &p.g;
    for (int k = 0; k < count; ++k) {
        GatherGemm& g = gs[k];
        g.X = p.two ? static_cast<const void*>(scaled) : dY;
        g.Wq = p.classes ? codes + p.cl.tb.first_word[k] : (p.two ? codes : packed_T);
        g.alpha = p.two ? one : alpha;
        g.Y = dX;
        g.splits = 1;
        g.partial = nullptr;
    }
    if (p.two && !p.classes && d->variant == TWN_VAR_BF16_POSTSCALE) {
        // 3x3 stride-1 layers with 64 filters scale dY inside the contraction: nothing to prepare
        GatherGemm g{};
        fill_conv_bwd_data(g, d, P, Q);
        g.X = dY;
        g.Wq = packed_T;
        g.alpha = alpha;
        g.Y = dX;
        g.splits = 1;
        if (env_int(Env::TILE, 0) == 0 && env_int(Env::C64, 1) != 0 && conv_c64_applicable(g))
            return launch_conv_c64_scaled(g, alpha, d->O / d->alpha_groups, st);
    }
    if (p.two && d->variant == TWN_VAR_BF16_POSTSCALE && d->y_dtype == TWN_BF16) {
        // The alphas stay with the codes where a kernel that would run the two-term problem has a build for it (bf16 outputs):
        // nothing is scaled.  Three terms of alpha are alpha itself, so a product is exact where two of alpha * dY leave 2^-18 of it:
        // of the bf16 values of dX 1.2e-4 .. 4.5e-4 differ from the rounded exact sum, with two terms of alpha * dY 2.5e-3 (two of alpha
        // would give 1.8e-3 .. 3.3e-3, by how the alphas lie to powers of two).
        // The third product costs what grows with the columns and taps, the two-term problem its preparation; above the line that
        // one's wider tiles win.  us, two terms of alpha * dY against three of alpha: persistent kernel, 3x3, 12544 pixels, 128
        // filters over 128 channels 17.9, 14.2; 256 over 256 45.6, 41.9; 512 over 256 80.6, 79.9; 512 over 512 113, 174; 3136
        // pixels, 512 over 512 45.4, 44.5; 50176, 128 over 128 47.9, 46.2; 256 over 256 117, 151; 1x1, 512 over 128 45.1, 23.2;
        // 512 over 512 84.0, 70.9.  Residue classes, 3x3/2, 12544 pixels, 512 filters over 64 channels 67.1, 40.4; over 256 90.4,
        // 92.1; over 512 150, 161; 25088 pixels 269, 302.
        DxPlan in;
        plan_dx(d, P, Q, &in, p.classes, true);
        const int n = in.classes ? in.cl.count : 1;
        GatherGemm* g = in.classes ? in.cl.g : &in.g;
        for (int k = 0; k < n; ++k) {
            g[k].X = dY;
            g[k].Wq = in.classes ? codes + in.cl.tb.first_word[k] : packed_T;
            g[k].alpha = g[k].alpha_in = alpha;
            g[k].alpha_in_rows = d->O / d->alpha_groups;
            g[k].Y = dX;
            g[k].splits = 1;
        }
        const bool few = conv_small_tile(gs, count) != 0;
        const int tile = few && d->O <= kSmallAlphaMax ? conv_small_tile(g, n) : 0;
        const double third = static_cast<double>(d->N) * P * Q * d->O * (static_cast<double>(d->C) * d->R * d->S - 900.0);
        const bool persistent = !few && !in.classes && !p.classes && third < 4.9e9 && gather_gemm_splits(p.g) <= 1 &&
                                conv_stream_alpha_applicable(g[0]);
        const bool batch = !few && in.classes && third < 1.8e10 && env_int(Env::DX_CLASS_BATCH, 1) != 0 &&
                           gather_gemm_dma_alpha_applicable(g, n);
        if (tile != 0 || persistent || batch) {
            if (in.classes) {
                rc = launch_dx_prep(class_prep(d, in.cl, packed_T, codes, dX), st);
                if (rc != TWN_OK) return rc;
            }
            return tile != 0 ? launch_conv_small(g, n, tile, st)
                             : persistent ? launch_conv_stream_alpha(g[0], st) : launch_gather_gemm_dma_batch_alpha(g, n, st);
        }
    }
    if (p.two || p.classes) {
        DxPrep q = p.classes ? class_prep(d, p.cl, packed_T, codes, dX) : DxPrep{};
        q.O = d->O;
        if (p.two) {
            q.dY = static_cast<const uint16_t*>(dY);
            q.alpha = alpha;
            q.rows_per_group = d->O / d->alpha_groups;
            q.pixels = static_cast<int64_t>(d->N) * P * Q;
            q.scaled = scaled;
            q.one = one;
        }
        q.packed_T = packed_T;
        q.C = d->C;
        q.wprT = static_cast<int32_t>(twn_packed_words_per_row(static_cast<int64_t>(d->R) * d->S * d->O));
        q.S = d->S;
        q.terms = p.two ? 2 : 1;
        q.tb = p.classes ? p.cl.tb : p.tb;
        q.codes = codes;
        rc = launch_dx_prep(q, st);
        if (rc != TWN_OK) return rc;
    }
    if (!p.classes) return dispatch(p.g, d->variant, ws + head, workspace_bytes > head ? workspace_bytes - head : 0, st);
    // all classes in ONE launch when the dispatcher would give each of them the same tile (they are too small to be worth
    // a launch each: ResNet-18 b64, the three strided 3x3 layers 33 / 34 / 48 us as four launches, 26 / 20 / 24 us as one)
    const bool batch = env_int(Env::DX_CLASS_BATCH, 1) != 0 && count > 1;
    const int small = batch ? conv_small_tile(gs, count) : 0;
    if (small != 0) return launch_conv_small(gs, count, small, st);
    int batch_tile = batch ? gather_gemm_dma_tile(gs[0]) : 0;
    for (int k = 1; k < count && batch_tile; ++k)
        if (gather_gemm_dma_tile(gs[k]) != batch_tile) batch_tile = 0;
    if (batch_tile != 0) {
        rc = launch_gather_gemm_dma_batch(gs, count, batch_tile, st);
        if (rc != TWN_ERR_UNSUPPORTED) return rc;
    }
    // no split-K here: a class is one of several launches of a layer whose own launch would not be split either,
    // and partial tiles plus a finishing launch per class cost more than the idle CUs (ResNet-18 stage 4: 70 -> 48 us)
    for (int k = 0; k < count; ++k) {
        rc = dispatch(gs[k], d->variant, nullptr, 0, st, false);
        if (rc != TWN_OK) return rc;
    }
    return TWN_OK;
}

// The two gradients of a checked call; dW has the first `o_real` of the filters.
static int32_t bwd_run(const twn_conv_desc* d, int P, int Q, const void* X, const void* dY, const uint32_t* packed_T, const float* alpha,
                       void* dX, float* dW, float* dbias, float dW_beta, void* workspace, size_t workspace_bytes, int32_t o_real,
                       hipStream_t st) {
    int32_t rc = TWN_OK;
    if (dX) {
        rc = data_gradient(d, P, Q, dY, packed_T, alpha, dX, workspace, workspace_bytes, st);
        if (rc != TWN_OK) return rc;
    }
    if (dW || dbias) {
        WeightGrad w{};
        w.X = static_cast<const uint16_t*>(X);
        w.dY = static_cast<const uint16_t*>(dY);
        w.dW = dW;
        w.dbias = dbias;
        w.partial = static_cast<float*>(workspace);
        w.partial_floats = static_cast<int64_t>(weight_grad_bytes(d, P, Q) / sizeof(float));
        w.beta = dW_beta;
        w.o_real = o_real;
        w.N = d->N; w.H = d->H; w.W = d->W; w.C = d->C; w.O = d->O; w.R = d->R; w.S = d->S;
        w.P = P; w.Q = Q;
        w.sh = d->stride_h; w.sw = d->stride_w; w.ph = d->pad_h; w.pw = d->pad_w;
        w.dh = d->dil_h; w.dw = d->dil_w;
        w.xc = d->C;
        SmallC sc;
        const bool small = dW && small_c(d, &sc) && d->O % 8 == 0;
        const FirstGradPlan f = small && aligned(X, 4) && aligned(dY, 16) ? first_grad_plan(d, P, Q) : FirstGradPlan{};
        if (f.use && workspace_bytes >= first_grad_bytes(d, f)) {
            rc = launch_first_weight_grad(taps_shape(d, P, Q), d->pad_h, d->pad_w, f, w.X, w.dY, w.partial, st);
            const BiasGrad bias = bias_in_final_pass(w);
            if (rc == TWN_OK)
                rc = launch_first_weight_grad_sum(w.partial, f.splits, d->O, o_real, d->C, d->R, d->S, 4 * f.G, dW_beta, dW, bias, st);
            if (rc != TWN_OK || !dbias || bias.blocks > 0) return rc;
            w.dW = nullptr;                 // the bias gradient is left
        } else if (small) {
            // first-layer mode: gather from the zero-bordered 4-channel copy (rebuilt here: the call is stateless)
            uint16_t* Xp = static_cast<uint16_t*>(workspace);
            rc = launch_pad_c4(static_cast<const uint16_t*>(X), d->N, d->H, d->W, d->C, d->pad_h, d->pad_w, sc.Hp,
                               sc.Wp, Xp, st);
            if (rc != TWN_OK) return rc;
            w.X = Xp;
            w.partial = reinterpret_cast<float*>(static_cast<unsigned char*>(workspace) + sc.x_bytes);
            w.partial_floats -= static_cast<int64_t>(sc.x_bytes / sizeof(float));
            w.H = sc.Hp; w.W = sc.Wp; w.C = 8; w.S = sc.Sp / 2;
            w.ph = w.pw = 0; w.dw = 2;
            w.xc = 4;
            w.pad_sp = sc.Sp; w.c_real = d->C; w.s_real = d->S;
        }
        rc = launch_weight_grad(w, st);
    }
    return rc;
}

extern "C" int32_t twn_conv2d_bwd_ste(const twn_conv_desc* d, const void* X, const void* dY,
                                      const uint32_t* packed_T, const float* alpha,
                                      void* dX, float* dW, float* dbias, float dW_beta,
                                      void* workspace, size_t workspace_bytes, void* stream) {
    int P, Q;
    int32_t rc = check_conv_desc(d, &P, &Q);
    if (rc != TWN_OK) return rc;
    if (!dY) return TWN_ERR_NULL;
    if (dX && (!packed_T || !alpha)) return TWN_ERR_NULL;
    if (dW && !X) return TWN_ERR_NULL;
    // the int8-stored comparison variant is forward-only: the transposed codes of this call are 2-bit packed
    if (d->x_dtype != TWN_BF16 ||
        (d->variant != TWN_VAR_BF16_POSTSCALE && d->variant != TWN_VAR_BF16_ALPHA_LDS)) return TWN_ERR_UNSUPPORTED;
    rc = check_dtype(d->y_dtype);
    if (rc != TWN_OK) return rc;
    if (dW_beta != 0.0f && dW_beta != 1.0f) return TWN_ERR_UNSUPPORTED;
    if (!aligned(dY, (d->O % 8 == 0) ? 16 : 2)) return TWN_ERR_ALIGN;
    if (X && !aligned(X, (d->C % 8 == 0) ? 16 : 2)) return TWN_ERR_ALIGN;
    if (packed_T && !aligned(packed_T, 16)) return TWN_ERR_ALIGN;
    if (dW && !aligned(dW, 4)) return TWN_ERR_ALIGN;
    if (dX) {
        rc = check_out_align(d->y_dtype, d->C, d->C, dX, nullptr);
        if (rc != TWN_OK) return rc;
    }
    if (dW || dbias) {
        const size_t need = weight_grad_bytes(d, P, Q);
        if (!workspace || workspace_bytes < need || !aligned(workspace, 256)) return TWN_ERR_WORKSPACE;
    }
    hipStream_t st = as_stream(stream);
    const FilterPadPlan pad = plan_filter_pad(d, P, Q);
    if (pad.use && (dW || (dX && static_cast<int64_t>(d->N) * P * Q >= 64)) && workspace && aligned(workspace, 256) &&
        workspace_bytes >= pad.bytes() + twn_conv2d_bwd_ste_workspace_bytes(&pad.d)) {
        unsigned char* ws = static_cast<unsigned char*>(workspace);
        FilterPad f{};
        f.dY = static_cast<const uint16_t*>(dY);
        f.pixels = static_cast<int64_t>(d->N) * P * Q;
        f.O = d->O; f.O8 = pad.d.O; f.C = d->C; f.RS = d->R * d->S;
        f.wpr = static_cast<int32_t>(twn_packed_words_per_row(static_cast<int64_t>(f.RS) * d->O));
        f.wpr8 = static_cast<int32_t>(twn_packed_words_per_row(static_cast<int64_t>(f.RS) * pad.d.O));
        f.dY8 = static_cast<uint16_t*>(workspace);
        f.codes8 = reinterpret_cast<uint32_t*>(ws + pad.dy_bytes);
        f.alpha8 = reinterpret_cast<float*>(ws + pad.dy_bytes + pad.code_bytes);
        if (dX) {
            f.packed_T = packed_T;
            f.alpha = d->alpha_groups > 1 ? alpha : nullptr;
        }
        rc = launch_filter_pad(f, st);
        if (rc != TWN_OK) return rc;
        rc = bwd_run(&pad.d, P, Q, X, f.dY8, f.codes8, f.alpha ? f.alpha8 : alpha, dX, dW, nullptr, dW_beta, ws + pad.bytes(),
                     workspace_bytes - pad.bytes(), d->O, st);
        if (rc != TWN_OK || !dbias) return rc;
        return bwd_run(d, P, Q, X, dY, packed_T, alpha, nullptr, nullptr, dbias, 0.0f, workspace, workspace_bytes, d->O, st);
    }
    return bwd_run(d, P, Q, X, dY, packed_T, alpha, dX, dW, dbias, dW_beta, workspace, workspace_bytes, d->O, st);
}
