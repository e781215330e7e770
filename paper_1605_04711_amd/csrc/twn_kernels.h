// Internal launch interface between the C-ABI entry points and the kernels.
#pragma once

#include "twn_common.h"
#include "twn_mfma.h"

namespace twn {

// One implicit-GEMM problem:  Y[m][n] = epilogue( sum_k A[m][k] * code[n][k] ).
// Rows m enumerate (batch, oh, ow) of the *output* of the gather; k enumerates
// (r, s, c) with c fastest.  A[m][k] is read from the NHWC tensor `X` at
//   th = oh*sh - ph + r*dh,  tw = ow*sw - pw + s*dw
// (after an exact division by divh/divw when those are > 1), zero outside
// [0,IH) x [0,IW).  The forward convolution uses this directly; the
// backward-data pass is the same gather over dY with sh = sw = 1, negated
// padding and tap step, and div = the forward stride.
struct GatherGemm {
    const void* X;          // bf16 (MFMA path) or float32 (fp32 path), NHWC, pixel stride `xs` elements
    const void* Wq;         // packed twn2 codes [NC][wpr]  (or int8 [NC][K] for the int8-stored variant)
    const float* alpha;     // [NC / rows_per_group]
    const float* scale;     // [NC] or null
    const float* shift;     // [NC] or null
    const void* residual;   // like Y or null
    void* Y;                // [M][ldy]
    int64_t M;
    int64_t xs;             // elements between consecutive pixels of X
    int64_t ldy;
    int32_t IH, IW, IC;
    int32_t OH, OW;
    int32_t NC;             // GEMM N (output channels)
    int32_t R, S;
    int32_t sh, sw, ph, pw, dh, dw, divh, divw;
    int32_t K;              // R*S*IC
    int32_t wpr;            // packed words per row
    int32_t rows_per_group;
    int32_t relu;
    int32_t y_f32;          // 1: Y (and residual) float32, 0: bf16
    int32_t plain_gemm;     // 1: R=S=1, stride 1, no padding, OH*OW pixels == rows of X
    int32_t chunk_gather;   // 1: 16-byte chunks are valid although IC/xs are not multiples of 8 (small-C path)
    // Output row remap (strided backward-data as one stride-1 problem per residue class): row m = (n, u, v) of an
    // [N][orU][orV] grid is written to pixel (n, ora + orsh*u, orb + orsw*v) of an [N][orH][orW] image.
    // orU == 0: rows are written in order.
    int32_t orU, orV, orH, orW, ora, orb, orsh, orsw;
    float* partial;         // split-K workspace [splits][M][NC] float32 (float64 on the float32 path; null when splits == 1)
    int32_t splits;         // K is cut into this many ranges of whole 64-wide slabs
    // Backward-data with several alphas, inside the contraction: the code of reduction channel c counts alpha_in[c / alpha_in_rows]
    // times, as three bf16 terms (null: 1).  Only conv_small and the *_alpha launchers take it.
    const float* alpha_in;
    int32_t alpha_in_rows;
};

// Number of K ranges the MFMA path uses for this problem (1 = no split); a pure function of the
// shapes, so the workspace query and the launch agree.
int32_t gather_gemm_splits(const GatherGemm& g);

int32_t launch_gather_gemm_mfma(const GatherGemm& g, int variant, hipStream_t st);

// Small-C first layers (C <= 4, dilation 1): the input is copied once into a zero-bordered
// [N][H+2ph][Wp][4] bf16 tensor so that two horizontally adjacent taps of 4 channels are one
// aligned-enough 16-byte chunk, and the packed codes are re-ordered to k' = (r*Sp + s)*4 + c
// with Sp = S rounded up to even (codes of the phantom tap / channels are zero).
int32_t launch_pad_c4(const uint16_t* X, int N, int H, int W, int C, int ph, int pw, int Hp, int Wp,
                      uint16_t* Xp, hipStream_t st);
// Tap subsets of a backward-data pass whose codes are gathered into contiguous K ranges: the residue classes of a strided
// layer (at most 4: stride products up to 4), or all taps as one class.  By value to the kernel.
struct DxClassTable {
    int32_t count, sh, sw;
    int32_t r0[4], nr[4], s0[4], ns[4], wpr[4];
    int64_t first_word[5];      // offset of each class's codes in the gathered buffer, in 32-bit words
};
// Everything a backward-data pass needs prepared, in one launch; every part is optional (null pointer).
struct DxPrep {
    // dY times alpha, carried as two bf16 terms next to each other: scaled[p][0..O) high, scaled[p][O..2O) low; *one = 1
    const uint16_t* dY;
    const float* alpha;
    int32_t rows_per_group, O;
    int64_t pixels;
    uint16_t* scaled;
    float* one;
    // codes of the classes, K order (tap, term, o) with `terms` copies of every tap's O codes
    const uint32_t* packed_T;
    int32_t C, wprT, S, terms;
    DxClassTable tb;
    uint32_t* codes;
    // 16-byte units of dX to clear (classes without taps)
    void* zero;
    int64_t zero16;
    // filled by the launch: threads of each part below 2^31 and O a multiple of 8, so that divisions are multiplications
    int32_t narrow;
    FastDivU divChunks, divTap, divW[4], divNs[4];
};
int32_t launch_dx_prep(const DxPrep& p, hipStream_t st);
// Backward of a layer whose filter count is no multiple of 8, over O8 = that count rounded up: dY, the transposed codes and, with one
// alpha per filter, the alphas with zeros in the filters that do not exist.
struct FilterPad {
    const uint16_t* dY;
    const uint32_t* packed_T;       // null: no codes wanted
    const float* alpha;             // null: one alpha for all
    int64_t pixels;
    int32_t O, O8, C, RS, wpr, wpr8;
    uint16_t* dY8;
    uint32_t* codes8;
    float* alpha8;
};
int32_t launch_filter_pad(const FilterPad& p, hipStream_t st);
int32_t launch_pad_repack_c4(const uint16_t* X, int N, int H, int W, int C, int ph, int pw, int Hp, int Wp, uint16_t* Xp,
                             const uint32_t* packed, int rows, int R, int S, int Sp, uint32_t* out, hipStream_t st);
int32_t launch_gather_gemm_dma(const GatherGemm& g, int tile, hipStream_t st);
// Several small unsplit convolution problems of one tile id in one launch of the one-tile-per-workgroup kernel
// (count <= 4); gather_gemm_dma_tile names the tile the dispatcher would use for a problem there (0: none).
int32_t gather_gemm_dma_tile(const GatherGemm& g, bool instead_of_persistent = false);
int32_t launch_gather_gemm_dma_batch(const GatherGemm* gs, int count, int tile, hipStream_t st);
bool gather_gemm_dma_alpha_applicable(const GatherGemm* gs, int count);
int32_t launch_gather_gemm_dma_batch_alpha(const GatherGemm* gs, int count, hipStream_t st);
int32_t launch_gather_gemm_fp32(const GatherGemm& g, hipStream_t st);
// K ranges of the float32 path (1 = no split); with more than one, g.partial holds [splits][M][NC] float64 sums.
int32_t gather_gemm_fp32_splits(const GatherGemm& g);
// Multiplication-free comparison kernel (vector ALUs, zero codes skipped); `applicable` is a pure function of the problem.
bool conv_addsub_applicable(const GatherGemm& g);
int32_t launch_conv_addsub(const GatherGemm& g, hipStream_t st);

// Persistent variant of the direct-to-LDS kernel (workgroups walk a list of tiles, loads of the next tile run
// under the epilogue of the last); `applicable` is a pure function of the problem, `tile` one of the ids the
// direct-to-LDS launcher takes (12, 14, 15, 16, 17).
bool conv_stream_applicable(const GatherGemm& g);
int32_t launch_conv_stream(const GatherGemm& g, int tile, hipStream_t st);
int32_t launch_conv_stream_pc(const GatherGemm& g, int tile, int np, int stages, hipStream_t st);
// The same walk over problems with alpha_in.
bool conv_stream_alpha_applicable(const GatherGemm& g);
int32_t launch_conv_stream_alpha(const GatherGemm& g, hipStream_t st);

// Problems of few output tiles: up to four of them in one launch, the K slabs of a tile shared out over the waves of
// one workgroup; conv_small_tile (a pure function of the problems) names the tile, 0 when other kernels are better.
int conv_small_tile(const GatherGemm* gs, int count);
constexpr int kSmallAlphaMax = 4096;        // reduction channels with an alpha of their own that its table in LDS holds
int32_t launch_conv_small(const GatherGemm* gs, int count, int tile, hipStream_t st);

// 3x3 stride-1 convolutions over 64 input channels (forward, or backward-data with mirrored taps), bf16 in and out,
// output channels a multiple of 64: persistent kernel with the expanded weights resident in registers and the input
// patch of an 8x8 pixel tile (with halo) in LDS; `applicable` is a pure function of the problem.
bool conv_c64_applicable(const GatherGemm& g);
int32_t launch_conv_c64(const GatherGemm& g, hipStream_t st);
// The same kernel over alpha_in[c / in_rows_per_group] * X instead of X (backward-data with several alphas): the product
// is carried as two bf16 terms that are formed on the way into LDS.
int32_t launch_conv_c64_scaled(const GatherGemm& g, const float* alpha_in, int32_t in_rows_per_group, hipStream_t st);

// First layers with three input channels, bf16 in and out, dilation 1 (forward): one persistent kernel, no
// workspace and no preparation launch; `applicable` is a pure function of the problem (shapes and alignment).
struct FirstLayer {
    const uint16_t* X;
    const uint32_t* Wq;
    const float* alpha;
    const float* scale;
    const float* shift;
    const uint16_t* residual;
    uint16_t* Y;
    int32_t N, H, W, C, O, R, S, sh, sw, ph, pw, P, Q;
    int32_t rows_per_group, relu;
};
bool conv_first_applicable(const FirstLayer& f);
int32_t launch_conv_first(const FirstLayer& f, hipStream_t st);


// dW[o][c][r][s] = beta*dW + sum_{n,p,q} X[n,ih,iw,c] * dY[n,p,q,o]; dbias[o] = sum dY.
struct WeightGrad {
    const uint16_t* X;      // bf16 NHWC [N][H][W][C]
    const uint16_t* dY;     // bf16 NHWC [N][P][Q][O]
    float* dW;              // [O][C][R][S]
    float* dbias;           // [O] or null
    float* partial;         // workspace: [splits][O][R*S*C] float32; after the final pass over them [splits][O] of dbias
    int64_t partial_floats; // its size
    float beta;
    int32_t N, H, W, C, O, R, S, P, Q;
    int32_t sh, sw, ph, pw, dh, dw;
    // First-layer mode (0 = off): X is the zero-bordered 4-channel copy, a "channel" chunk of 8 is two
    // adjacent taps x 4 channels (C = 8, S = pad_sp/2, dw = 2 above), and the reduction maps
    // j' = (r*pad_sp + s)*4 + c back to [O][c_real][R][s_real], dropping the phantom tap and channels.
    int32_t pad_sp, c_real, s_real;
    int32_t xc;             // elements between consecutive pixels of X (C, or 4 in first-layer mode)
    int32_t o_real;         // filters of dW (O, or fewer where dY is padded)
};

// Bias gradient of a call, cut into groups of channels: `blocks` leading blocks of a final pass over dW's partial tiles, or a launch
// of its own (blocks = 0 in the final pass).
struct BiasGrad {
    const uint16_t* dY;
    float* dbias;
    int64_t pixels;
    int32_t O, vec;         // channels; 8 or 1 per load
    int32_t chunks_per_group, groups, blocks;
    int32_t batch;          // pixels a thread requests at a time
};
// Empty (blocks = 0) unless one launch sums all pixels, which needs no partial sums.
BiasGrad bias_in_final_pass(const WeightGrad& w);

// How the weight gradient of one layer is cut up; a pure function of the shapes, shared by the
// workspace query and the launch.
struct WgPlan {
    int32_t patch;          // 1: 128x256 tiles over 32-pixel patches (channel counts multiples of 8); 0: 128x128 tiles over 64 consecutive pixels
    int32_t pn, ph, pw;     // patch = pn images x ph rows x pw columns (pn*ph*pw = 32), powers of two
    int32_t sn, sy, sx;     // patches along batch, rows, columns
    int64_t slabs;          // reduction slabs in total
    int32_t splits;         // blockIdx.y ranges of slabs
    int32_t tiles;          // output tiles (blockIdx.x)
    int32_t ks;             // patch kernel: groups of four waves per workgroup that share a range (1 or 2)
};
int32_t launch_weight_grad(const WeightGrad& w, hipStream_t st);

// Weight gradient of filters with several taps over patches with halo (twn_bwd_weight_taps.hip).
struct WgShape {
    int32_t N, H, W, C, O, R, S, P, Q, sh, sw, dh, dw;
};
struct WgTapsPlan {
    int32_t use;                        // 0: the general kernel takes the layer
    int32_t pn, ph, pw;                 // patch of 32 output pixels: images x rows x columns, powers of two
    int32_t sn, sy, sx, slabs;          // patches along batch, rows, columns; in total
    int32_t hh, ww;                     // input rows and columns of one image of a patch
    int32_t row_slots, img_slots;       // pitch of a patch row and of an image in LDS, in pixels of 32 channels
    int32_t slots, nb;                  // pixels of a patch in LDS (with padding), loads of half of them
    int32_t stage_bytes, depth;
    int32_t tiles_o, tiles_c, groups, tiles;
    int32_t per, splits;                // patches per pixel range, ranges
};
WgTapsPlan plan_weight_grad_taps(const WgShape& w);
// The kernel and the pixel ranges of a layer's weight gradient; `first`: the shape is that of the first-layer mode.  The workspace
// query and the launch both ask this.
struct WgRoute {
    WgTapsPlan taps;            // taps.use: this kernel, otherwise the general one
    WgPlan general;
    int32_t splits;             // ranges of the kernel in use
};
WgRoute route_weight_grad(const WgShape& w, bool first);
// *bias_done: the final pass summed dbias too.
int32_t launch_weight_grad_taps(const WeightGrad& w, const WgTapsPlan& pl, bool* bias_done, hipStream_t st);

// Weight gradient of a three-channel first layer (twn_bwd_first.hip): partial tiles [splits][O][(r*G + s/4)*16 + (s%4)*4 + c],
// i.e. those of the first-layer mode above with pad_sp = 4 G.
struct FirstGradPlan {
    int32_t use;                // 0: the general kernel takes the layer
    int32_t G, J;               // blocks of four taps per filter row, columns of a partial tile
    int32_t tiles, per, splits; // tiles of 16x16 output pixels, per workgroup, ranges
};
FirstGradPlan plan_first_weight_grad(const WgShape& w);
int32_t launch_first_weight_grad(const WgShape& w, int32_t ph, int32_t pw, const FirstGradPlan& p, const uint16_t* X,
                                 const uint16_t* dY, float* partial, hipStream_t st);
// dW = beta*dW + sum of partial tiles in first-layer mode, and dbias where `bias` is not empty.
int32_t launch_first_weight_grad_sum(const float* partial, int32_t splits, int32_t O, int32_t o_real, int32_t C, int32_t R, int32_t S, int32_t pad_sp,
                                     float beta, float* dW, const BiasGrad& bias, hipStream_t st);

}  // namespace twn
