// float32 path of the ternary convolution / inner product (Eq. 2, Alg. 1 step 8) for float32 activations: implicit
// GEMM on the float64 matrix cores.  Inputs and outputs are float32; products with a code are exact and the running
// sums are float64, because float32 accumulation of cancelling sums cannot hold a 1e-5 relative bound on small
// outputs.  The codes are expanded in registers to 0 / +-2.0 (one shift and one mask give the high half of the double,
// the low half is zero; the factor is taken back exactly before the rounding to float32), alpha is applied afterwards.
//
// v_mfma_f64_16x16x4_f64 occupies the matrix core for 64 cycles and takes one double per lane and operand, so a wave
// needs 1 KB of activations and one word of codes per lane and 16-channel column for 256 cycles and more of matrix
// work: both come straight from global memory (L1, L2) and nothing is staged in LDS.  What bounds the path is the
// float64 rate (79 TFLOP/s) for large problems and latency for LeNet-sized ones, so a tile is small (16 pixels by 16,
// 32 or 64 channels) and the K blocks of a tile are shared out over the NW waves of a workgroup, whose float64 sums
// are added through LDS in a fixed order.  LeNet b64 against float64 FMAs on tiles staged in LDS, split along K over
// workgroups with a finishing launch: 4096 pixels x 64 x 800 34 -> 13.3 us, 36864 x 32 x 25 13.9 -> 9.8,
// 64 x 512 x 1024 16.3 -> 6.7, 64 x 10 x 512 12.3 -> 4.9; 1024 x 1024 x 1024 136 -> 44 (float64 floor 27).
#include "twn_kernels.h"
#include "twn_mfma.h"

namespace twn {

typedef double f64x4 __attribute__((ext_vector_type(4)));
// four floats at float alignment: global_load_dwordx4 needs dword alignment only
struct __attribute__((packed, aligned(4))) Float4 {
    float v[4];
};

enum F32Mode : int {
    kF32Gemm = 0,       // rows of X are the reduction rows
    kF32Quad = 1,       // channel count a multiple of 4: four consecutive k lie in one tap
    kF32Element = 2,    // every element finds its own tap
};

struct F32Args {
    GatherGemm g;
    FastDivU divIC, divS, divOW, divOH, divTN, divRG;
    FastDivU divParts;      // K blocks of part p of splits * NW: from blocks_q * p + blocks_r * p / parts on
    int32_t blocks_q, blocks_r;
    int64_t tiles;
    int32_t tiles_n;
    int32_t narrow;         // rows and tiles below 2^31: divisions by multiplication (a 64-bit one costs about a microsecond)
    int32_t walk;           // short kernel: row blocks per wave
};

// Parameters of one output column, requested before the sums they are applied to.  A column behind the last one reads that one's:
// with a branch per lane around the loads the compiler waits for each of them before the first activations are requested.
struct F32Column {
    float al, sc, sf;
};
__device__ __forceinline__ F32Column f32_column(const GatherGemm& g, const FastDivU& divRG, int ncol) {
    const int n = min(ncol, g.NC - 1);
    F32Column c;            // sc and sf: only what the call has
    c.al = g.alpha[g.rows_per_group >= g.NC ? 0u : fdiv_u(static_cast<uint32_t>(n), divRG)];
    if (g.scale) c.sc = g.scale[n];
    if (g.shift) c.sf = g.shift[n];
    return c;
}

__device__ __forceinline__ void f32_tail_store(const GatherGemm& g, int64_t m, int ncol, double sum, const F32Column& c) {
    float v = (static_cast<float>(sum) * c.al) * (g.scale ? c.sc : 1.0f) + (g.shift ? c.sf : 0.0f);
    const int64_t off = m * g.ldy + ncol;
    if (g.y_f32) {
        if (g.residual) v += static_cast<const float*>(g.residual)[off];
        if (g.relu) v = fmaxf(v, 0.0f);
        static_cast<float*>(g.Y)[off] = v;
    } else {
        if (g.residual) v += bf16_to_f32(static_cast<const uint16_t*>(g.residual)[off]);
        if (g.relu) v = fmaxf(v, 0.0f);
        static_cast<uint16_t*>(g.Y)[off] = f32_to_bf16(v);
    }
}

// blockIdx.x walks the tiles, blockIdx.y is the K range when g.splits > 1 (float64 sums to g.partial [split][M][NC]).
template <int NT, int NW, int MODE>
__global__ __launch_bounds__(64 * NW) void gather_gemm_f64_kernel(const F32Args args) {
    constexpr int BN = 16 * NT;
    constexpr int DEPTH = 4;                            // K blocks of 16 in flight
    __shared__ double part[NW > 1 ? NW * 16 * BN : 1];
    const GatherGemm& g = args.g;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int l16 = lane & 15, quad = lane >> 4;        // pixel / channel of the tile; which four k of a block
    const float* __restrict__ X = static_cast<const float*>(g.X);
    const uint32_t* __restrict__ Wq = static_cast<const uint32_t*>(g.Wq);

    // the wave's range of K blocks; a ragged last block is done element by element after the others
    const uint32_t p = blockIdx.y * NW + static_cast<uint32_t>(wave);
    auto first_block = [&](uint32_t q) { return static_cast<int>(args.blocks_q * q + fdiv_u(args.blocks_r * q, args.divParts)); };
    const int kb0 = first_block(p), kb1 = first_block(p + 1);
    const int kfull = (MODE == kF32Element) ? kb1 : min(kb1, g.K >> 4);

    for (int64_t t = blockIdx.x; t < args.tiles; t += gridDim.x) {
        const int64_t tm = args.narrow ? static_cast<int64_t>(fdiv_u(static_cast<uint32_t>(t), args.divTN)) : t / args.tiles_n;
        const int64_t m0 = tm * 16;
        const int n0 = static_cast<int>(t - tm * args.tiles_n) * BN;

        // columns this thread writes: one per 16-channel group (one wave), or those of its share of the summed tile
        constexpr int NE = (NW == 1) ? NT : (BN > 4 * NW ? BN / (4 * NW) : 1);
        F32Column col[NE];
#pragma unroll
        for (int i = 0; i < NE; ++i) col[i] = f32_column(g, args.divRG, n0 + (NW == 1 ? 16 * i + l16 : (threadIdx.x + i * 64 * NW) % BN));

        // rows and columns beyond the problem repeat the last one; they are not stored
        const int64_t m = min(m0 + l16, g.M - 1);
        const float* xrow;
        int ih0 = 0, iw0 = 0;
        if (MODE == kF32Gemm) {
            xrow = X + m * g.xs;
        } else {
            int64_t img;
            int oh, ow;
            if (args.narrow) {
                const uint32_t mm = static_cast<uint32_t>(m);
                const uint32_t row = fdiv_u(mm, args.divOW);
                ow = static_cast<int>(mm - row * static_cast<uint32_t>(g.OW));
                const uint32_t im = fdiv_u(row, args.divOH);
                oh = static_cast<int>(row - im * static_cast<uint32_t>(g.OH));
                img = im;
            } else {
                const int64_t row = m / g.OW;
                ow = static_cast<int>(m - row * g.OW);
                img = row / g.OH;
                oh = static_cast<int>(row - img * g.OH);
            }
            xrow = X + img * g.IH * g.IW * g.xs;
            ih0 = oh * g.sh - g.ph;
            iw0 = ow * g.sw - g.pw;
        }
        const uint32_t* wrow[NT];
#pragma unroll
        for (int j = 0; j < NT; ++j) wrow[j] = Wq + static_cast<int64_t>(min(n0 + 16 * j + l16, g.NC - 1)) * g.wpr;

        // Four consecutive elements of the lane's row from k on; an element is real if k < K and its tap lies in the
        // image.  No short cuts in the conditions: the loads of a block are issued back to back.
        struct Place {
            int c, s, th, tw;
            int64_t off;
        };
        auto place = [&](int k) {
            const uint32_t rs = fdiv_u(static_cast<uint32_t>(k), args.divIC);
            const uint32_t r = fdiv_u(rs, args.divS);
            Place q;
            q.c = k - static_cast<int>(rs) * g.IC;
            q.s = static_cast<int>(rs - r * static_cast<uint32_t>(g.S));
            q.th = ih0 + static_cast<int>(r) * g.dh;
            q.tw = iw0 + q.s * g.dw;
            q.off = static_cast<int64_t>(q.th * g.IW + q.tw) * g.xs + q.c;
            return q;
        };
        auto inside = [&](const Place& q) {
            return static_cast<uint32_t>(static_cast<unsigned>(q.th) < static_cast<unsigned>(g.IH)) &
                   static_cast<uint32_t>(static_cast<unsigned>(q.tw) < static_cast<unsigned>(g.IW));
        };
        auto load_elements = [&](int k, float (&v)[4]) {
            uint32_t real = 0;
            if (MODE == kF32Gemm) {
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const bool ok = k + i < g.K;
                    real |= static_cast<uint32_t>(ok) << i;
                    v[i] = xrow[ok ? k + i : 0];
                }
                return real;
            }
            Place q = place(k);
            const int64_t next_tap = static_cast<int64_t>(g.dw) * g.xs - g.IC;
            const int64_t next_row = static_cast<int64_t>(g.dh) * g.IW * g.xs - static_cast<int64_t>(g.S) * g.dw * g.xs;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const uint32_t ok = inside(q) & static_cast<uint32_t>(k + i < g.K);
                real |= ok << i;
                v[i] = xrow[ok ? q.off : 0];
                const bool wc = q.c + 1 == g.IC;
                q.c = wc ? 0 : q.c + 1;
                q.s += wc ? 1 : 0;
                q.tw += wc ? g.dw : 0;
                q.off += 1 + (wc ? next_tap : 0);
                const bool ws = q.s == g.S;
                q.s = ws ? 0 : q.s;
                q.th += ws ? g.dh : 0;
                q.tw = ws ? iw0 : q.tw;
                q.off += ws ? next_row : 0;
            }
            return real;
        };

        float xa[DEPTH][4];
        uint32_t wa[DEPTH][NT];
        uint32_t okv[DEPTH];            // bit i: element i is real
        auto load = [&](int d, int kb) {
            const int k = kb * 16 + quad * 4;
            if (MODE == kF32Element) {
                okv[d] = load_elements(k, xa[d]);
            } else {
                const Float4* src = reinterpret_cast<const Float4*>(xrow + k);
                okv[d] = 15u;
                if (MODE == kF32Quad) {
                    const Place q = place(k);
                    const uint32_t ok = inside(q);
                    okv[d] = ok ? 15u : 0u;
                    src = reinterpret_cast<const Float4*>(xrow + (ok ? q.off : 0));
                }
                const Float4 v = *src;
#pragma unroll
                for (int i = 0; i < 4; ++i) xa[d][i] = v.v[i];
            }
#pragma unroll
            for (int j = 0; j < NT; ++j) wa[d][j] = wrow[j][kb];
        };
        f64x4 acc[NT] = {};
        auto multiply = [&](int d) {
            double a[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) a[i] = static_cast<double>(((okv[d] >> i) & 1u) ? xa[d][i] : 0.0f);
            // codes 4*quad + i of the word sit, after this shift, at bits 0, 16, 2, 18
            uint32_t w[NT];
#pragma unroll
            for (int j = 0; j < NT; ++j) w[j] = wa[d][j] >> (4 * quad);
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int sh = 30 - ((i & 1) * 16 + (i >> 1) * 2);
#pragma unroll
                for (int j = 0; j < NT; ++j) {
                    const double b = __hiloint2double(static_cast<int>((w[j] << sh) & 0xC0000000u), 0);
                    acc[j] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[i], b, acc[j], 0, 0, 0);
                }
            }
        };

        const int n = kfull - kb0;
        int i = 0;
        if (n >= DEPTH) {
#pragma unroll
            for (int d = 0; d < DEPTH; ++d) load(d, kb0 + d);
            for (; i + 2 * DEPTH <= n; i += DEPTH) {
#pragma unroll
                for (int d = 0; d < DEPTH; ++d) {
                    multiply(d);
                    load(d, kb0 + i + d + DEPTH);
                }
            }
#pragma unroll
            for (int d = 0; d < DEPTH; ++d) {
                multiply(d);
                if (i + d + DEPTH < n) load(d, kb0 + i + d + DEPTH);
            }
            i += DEPTH;
        } else {
#pragma unroll
            for (int d = 0; d < DEPTH - 1; ++d)
                if (d < n) load(d, kb0 + d);
        }
#pragma unroll
        for (int d = 0; d < DEPTH - 1; ++d)
            if (i + d < n) multiply(d);
        if (MODE != kF32Element && kb1 > kfull && kb1 > kb0) {      // the ragged block is the last one of K
            okv[0] = load_elements(kfull * 16 + quad * 4, xa[0]);
#pragma unroll
            for (int j = 0; j < NT; ++j) wa[0][j] = wrow[j][kfull];
            multiply(0);
        }

        // register r of a lane is pixel quad + 4r, channel l16
        auto finish = [&](int64_t mo, int ncol, double sum, const F32Column& c) {
            if (mo >= g.M || ncol >= g.NC) return;
            if (g.splits > 1)
                reinterpret_cast<double*>(g.partial)[(static_cast<int64_t>(blockIdx.y) * g.M + mo) * g.NC + ncol] = sum;
            else
                f32_tail_store(g, mo, ncol, sum, c);
        };
        if (NW == 1) {
#pragma unroll
            for (int j = 0; j < NT; ++j)
#pragma unroll
                for (int r = 0; r < 4; ++r) finish(m0 + quad + 4 * r, n0 + 16 * j + l16, 0.5 * acc[j][r], col[j]);
        } else {
#pragma unroll
            for (int j = 0; j < NT; ++j)
#pragma unroll
                for (int r = 0; r < 4; ++r) part[(wave * 16 + quad + 4 * r) * BN + 16 * j + l16] = acc[j][r];
            __syncthreads();
#pragma unroll
            for (int o = 0; o < NE; ++o) {
                const int e = threadIdx.x + o * 64 * NW;
                if (e >= 16 * BN) break;
                double sum = part[e];
#pragma unroll
                for (int w = 1; w < NW; ++w) sum += part[w * 16 * BN + e];
                finish(m0 + e / BN, n0 + e % BN, 0.5 * sum, col[o]);
            }
            __syncthreads();            // the next tile reuses `part`
        }
    }
}

// Convolutions whose channel count is no multiple of 4 and whose K is at most 16 KB (KB blocks of 16): a wave walks over row
// blocks of one column block, independently of the others of its workgroup.  Where an element lies relative to its pixel and the doubles of the codes do not change
// from row block to row block: both are kept in registers, and a row block costs its loads, its bounds tests and its matrix
// work; the next block's elements are in flight while this one is multiplied.  36864 pixels x 32 channels, 5x5 over one channel
// (K = 25): 11.6 -> 8.5 us.
constexpr int kShortWaves = 4;              // independent waves per workgroup
template <int NT, int KB>
__global__ __launch_bounds__(64 * kShortWaves) void gather_gemm_f64_short_kernel(const F32Args args) {
    const GatherGemm& g = args.g;
    const int lane = threadIdx.x & 63, l16 = lane & 15, quad = lane >> 4;
    const uint32_t wave = static_cast<uint32_t>(__builtin_amdgcn_readfirstlane(
        static_cast<int>(blockIdx.x) * kShortWaves + static_cast<int>(threadIdx.x >> 6)));
    const float* __restrict__ X = static_cast<const float*>(g.X);
    const uint32_t* __restrict__ Wq = static_cast<const uint32_t*>(g.Wq);
    const uint32_t span = fdiv_u(wave, args.divTN);
    const int n0 = static_cast<int>(wave - span * static_cast<uint32_t>(args.tiles_n)) * 16 * NT;
    const int64_t rows = (g.M + 15) / 16;
    const int64_t first = static_cast<int64_t>(span) * args.walk;
    const int64_t last = first + args.walk < rows ? first + args.walk : rows;
    if (first >= last) return;

    F32Column col[NT];
    uint32_t b[KB][4][NT];                  // high halves of the codes' doubles
#pragma unroll
    for (int j = 0; j < NT; ++j) {
        col[j] = f32_column(g, args.divRG, n0 + 16 * j + l16);
        const uint32_t* wrow = Wq + static_cast<int64_t>(min(n0 + 16 * j + l16, g.NC - 1)) * g.wpr;
#pragma unroll
        for (int d = 0; d < KB; ++d) {
            const uint32_t w = wrow[d] >> (4 * quad);       // rows are padded to 128 codes
#pragma unroll
            for (int i = 0; i < 4; ++i) b[d][i][j] = (w << (30 - ((i & 1) * 16 + (i >> 1) * 2))) & 0xC0000000u;
        }
    }
    int off[KB][4], th[KB][4], tw[KB][4];   // element k against (ih0, iw0) of the pixel
#pragma unroll
    for (int d = 0; d < KB; ++d)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int k = d * 16 + quad * 4 + i;
            const uint32_t rs = fdiv_u(static_cast<uint32_t>(k), args.divIC), r = fdiv_u(rs, args.divS);
            th[d][i] = k < g.K ? static_cast<int>(r) * g.dh : -(1 << 28);       // beyond K: outside every image
            tw[d][i] = static_cast<int>(rs - r * static_cast<uint32_t>(g.S)) * g.dw;
            off[d][i] = (static_cast<int>(r) * g.dh * g.IW + tw[d][i]) * static_cast<int>(g.xs) + (k - static_cast<int>(rs) * g.IC);
        }
    float x[2][KB][4];
    auto load = [&](int64_t tm, float (&v)[KB][4]) __attribute__((always_inline)) {
        const int64_t at = tm * 16 + l16;
        const uint32_t m = static_cast<uint32_t>(at < g.M ? at : g.M - 1);
        const uint32_t row = fdiv_u(m, args.divOW), img = fdiv_u(row, args.divOH);
        const int ih0 = static_cast<int>(row - img * static_cast<uint32_t>(g.OH)) * g.sh - g.ph;
        const int iw0 = static_cast<int>(m - row * static_cast<uint32_t>(g.OW)) * g.sw - g.pw;
        const int base = ((static_cast<int>(img) * g.IH + ih0) * g.IW + iw0) * static_cast<int>(g.xs);
#pragma unroll
        for (int d = 0; d < KB; ++d)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const bool ok = (static_cast<unsigned>(ih0 + th[d][i]) < static_cast<unsigned>(g.IH)) &
                                (static_cast<unsigned>(iw0 + tw[d][i]) < static_cast<unsigned>(g.IW));
                const float t = X[ok ? base + off[d][i] : 0];
                v[d][i] = ok ? t : 0.0f;
            }
    };
    auto finish = [&](int64_t tm, const float (&v)[KB][4]) __attribute__((always_inline)) {
        f64x4 acc[NT] = {};
#pragma unroll
        for (int d = 0; d < KB; ++d)
#pragma unroll
            for (int i = 0; i < 4; ++i)
#pragma unroll
                for (int j = 0; j < NT; ++j)
                    acc[j] = __builtin_amdgcn_mfma_f64_16x16x4f64(static_cast<double>(v[d][i]),
                                                                  __hiloint2double(static_cast<int>(b[d][i][j]), 0), acc[j], 0, 0, 0);
#pragma unroll
        for (int j = 0; j < NT; ++j)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int64_t m = tm * 16 + quad + 4 * r;
                const int n = n0 + 16 * j + l16;
                if (m < g.M && n < g.NC) f32_tail_store(g, m, n, 0.5 * acc[j][r], col[j]);
            }
    };
    load(first, x[0]);
    for (int64_t t = first; t < last; t += 2) {
        if (t + 1 < last) load(t + 1, x[1]);
        finish(t, x[0]);
        if (t + 1 >= last) break;
        if (t + 2 < last) load(t + 2, x[0]);
        finish(t + 1, x[1]);
    }
}

// Sum of the K ranges in a fixed order (float64), then the same tail as the unsplit kernel.
__global__ __launch_bounds__(256) void fp32_splitk_finish_kernel(const GatherGemm g, const FastDivU divRG) {
    const int64_t i = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x;
    const int64_t total = g.M * g.NC;
    if (i >= total) return;
    const double* __restrict__ part = reinterpret_cast<const double*>(g.partial);
    double sum = 0.0;
    for (int s = 0; s < g.splits; ++s) sum += part[static_cast<int64_t>(s) * total + i];
    const int64_t m = i / g.NC;
    const int ncol = static_cast<int>(i - m * g.NC);
    f32_tail_store(g, m, ncol, sum, f32_column(g, divRG, ncol));
}

// Tile width, waves per tile and K ranges of the float32 path: a pure function of the shapes (the workspace query and
// the launch agree).  Wide tiles share the activations and their conversion between columns; they are taken while 512
// tiles (64 channels: 1024) remain and they pad the channels by no more than an eighth above 16-channel tiles.
// Waves are added to a tile up to about 1.5 per SIMD in all (4096 x 64 x 800, 512 tiles: 2 waves 22.6 us, 4 waves 13.3,
// 8 waves 14.3; 128 tiles of 64 x 512 x 1024: 4 waves 7.0, 8 waves 6.7, 16 waves 7.4), each with at least two K blocks (36864 x 32 x 25 on two
// blocks: 1 wave 9.8 us, 2 waves 13.9).  Only problems whose waves would walk more than 32 blocks on an idle chip (few
// outputs, K beyond 8192) are cut over workgroups too.
struct Fp32Plan {
    int nt, nw, splits;
    int64_t tiles;
    int32_t tiles_n;
};
static Fp32Plan fp32_plan(const GatherGemm& g) {
    const int64_t tm = (g.M + 15) / 16, nkb = (static_cast<int64_t>(g.K) + 15) / 16;
    const int64_t tn1 = (static_cast<int64_t>(g.NC) + 15) / 16;
    Fp32Plan p{1, 1, 1, 0, 0};
    for (int nt = 4; nt >= 2; nt >>= 1) {
        const int64_t tn = (tn1 + nt - 1) / nt;
        if (tn * nt * 8 > tn1 * 9 || tm * tn < (nt == 4 ? 1024 : 512)) continue;
        p.nt = nt;
        break;
    }
    const int64_t tn = (tn1 + p.nt - 1) / p.nt;
    p.tiles = tm * tn;
    p.tiles_n = static_cast<int32_t>(tn);
    while (p.nw < 16 && p.tiles * p.nw < 1536 && nkb >= 4 * p.nw && (p.nw < 8 || p.tiles <= 64)) p.nw *= 2;
    if (p.nw == 16 && nkb > 32 * p.nw && env_int(Env::F32_SPLITK, 1) != 0) {
        int64_t want = 2048 / (p.tiles * p.nw);
        if (want > nkb / (8 * p.nw)) want = nkb / (8 * p.nw);
        if (want > 16) want = 16;
        if (want > 1) p.splits = static_cast<int>(want);
    }
    return p;
}

int32_t gather_gemm_fp32_splits(const GatherGemm& g) { return fp32_plan(g).splits; }

template <int NT, int NW>
static void launch_f64(const F32Args& a, int mode, hipStream_t st) {
    // tiles beyond the grid are walked in a loop
    const dim3 grid(static_cast<unsigned>(a.tiles < (1 << 22) ? a.tiles : (1 << 22)), static_cast<unsigned>(a.g.splits));
    if (mode == kF32Gemm)
        gather_gemm_f64_kernel<NT, NW, kF32Gemm><<<grid, 64 * NW, 0, st>>>(a);
    else if (mode == kF32Quad)
        gather_gemm_f64_kernel<NT, NW, kF32Quad><<<grid, 64 * NW, 0, st>>>(a);
    else
        gather_gemm_f64_kernel<NT, NW, kF32Element><<<grid, 64 * NW, 0, st>>>(a);
}

template <int NT>
static void launch_short(F32Args& a, hipStream_t st) {
    // about two waves per SIMD, each with a walk of whole row blocks
    const int64_t rows = (a.g.M + 15) / 16;
    a.walk = static_cast<int32_t>((rows * a.tiles_n + 2047) / 2048);
    const int64_t waves = (rows + a.walk - 1) / a.walk * a.tiles_n;
    const unsigned grid = static_cast<unsigned>((waves + kShortWaves - 1) / kShortWaves);
    if (a.g.K <= 32)
        gather_gemm_f64_short_kernel<NT, 2><<<grid, 64 * kShortWaves, 0, st>>>(a);
    else
        gather_gemm_f64_short_kernel<NT, 4><<<grid, 64 * kShortWaves, 0, st>>>(a);
}

int32_t launch_gather_gemm_fp32(const GatherGemm& g, hipStream_t st) {
    const Fp32Plan p = fp32_plan(g);
    if (p.tiles <= 0) return TWN_ERR_SHAPE;
    if (g.splits > 1 && (g.splits != p.splits || !g.partial)) return TWN_ERR_WORKSPACE;
    F32Args a;
    a.g = g;
    a.divIC = make_fastdiv_u(static_cast<uint32_t>(g.IC));
    a.divS = make_fastdiv_u(static_cast<uint32_t>(g.S));
    a.tiles = p.tiles;
    a.tiles_n = p.tiles_n;
    a.narrow = g.M < (1LL << 31) - 16 && p.tiles < (1LL << 31);
    a.divOW = make_fastdiv_u(static_cast<uint32_t>(g.OW));
    a.divOH = make_fastdiv_u(static_cast<uint32_t>(g.OH));
    a.divTN = make_fastdiv_u(static_cast<uint32_t>(p.tiles_n));
    a.divRG = make_fastdiv_u(static_cast<uint32_t>(g.rows_per_group));
    const int32_t nkb = static_cast<int32_t>((static_cast<int64_t>(g.K) + 15) / 16), parts = (g.splits > 1 ? g.splits : 1) * p.nw;
    a.divParts = make_fastdiv_u(static_cast<uint32_t>(parts));
    a.blocks_q = nkb / parts;
    a.blocks_r = nkb % parts;
    a.walk = 0;
    const int mode = g.plain_gemm ? kF32Gemm : (g.IC % 4 == 0) ? kF32Quad : kF32Element;
    // short K, no taps to divide: offsets in 32 bits, rows and paddings far below the 2^28 that marks an element beyond K, one wave
    // per tile in the plan
    if (mode == kF32Element && g.K <= 64 && p.nw == 1 && g.splits <= 1 && a.narrow && g.divh == 1 && g.divw == 1 &&
        g.ph < (1 << 24) && g.pw < (1 << 24) &&
        g.M / (static_cast<int64_t>(g.OH) * g.OW) * g.IH * g.IW * g.xs < (1LL << 30) &&
        static_cast<int64_t>(g.R) * abs(g.dh) < (1 << 24) && static_cast<int64_t>(g.S) * abs(g.dw) < (1 << 24) &&
        (static_cast<int64_t>(g.R) * abs(g.dh) * g.IW + static_cast<int64_t>(g.S) * abs(g.dw)) * g.xs < (1LL << 30)) {
        if (p.nt == 4) launch_short<4>(a, st);
        else if (p.nt == 2) launch_short<2>(a, st);
        else launch_short<1>(a, st);
        return launch_status();
    }
    switch (p.nt * 32 + p.nw) {
        case 32 + 1: launch_f64<1, 1>(a, mode, st); break;
        case 32 + 2: launch_f64<1, 2>(a, mode, st); break;
        case 32 + 4: launch_f64<1, 4>(a, mode, st); break;
        case 32 + 8: launch_f64<1, 8>(a, mode, st); break;
        case 32 + 16: launch_f64<1, 16>(a, mode, st); break;
        case 64 + 1: launch_f64<2, 1>(a, mode, st); break;
        case 64 + 2: launch_f64<2, 2>(a, mode, st); break;
        case 64 + 4: launch_f64<2, 4>(a, mode, st); break;
        case 128 + 1: launch_f64<4, 1>(a, mode, st); break;
        case 128 + 2: launch_f64<4, 2>(a, mode, st); break;
        default: return TWN_ERR_UNSUPPORTED;
    }
    if (g.splits > 1) {
        const int64_t total = g.M * g.NC;
        fp32_splitk_finish_kernel<<<static_cast<unsigned>((total + 255) / 256), 256, 0, st>>>(g, a.divRG);
    }
    return launch_status();
}

}  // namespace twn
