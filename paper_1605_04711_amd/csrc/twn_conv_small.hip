// Implicit-GEMM ternary convolution / inner product for problems of few output tiles (gfx950).
//
// Same arithmetic as the other contraction kernels (bf16 activations, 2-bit codes expanded in registers to
// 0 / +-2.0, alpha/2 and the block tail in the fp32 epilogue), for launches that the memory latency bounds: a
// batch-1 layer, a classifier, the deep layers of a small batch.  Tiles of 16 or 32 pixels by 32 or 64 channels, and the
// K slabs of a tile are shared out over the NW waves of ONE workgroup, whose partial tiles are summed through LDS
// in a fixed order: no partial sums in memory and no second launch.  A wave stages its own slabs by direct-to-LDS
// loads, DEPTH slabs ahead (rows of 128 contiguous bytes: a fragment load straight into registers touches a cache line
// per lane and costs four times as long), and waits for its own loads only: there is no barrier before the final sum.
#include <mutex>

#include "twn_kernels.h"
#include "twn_lds_asm.h"
#include "twn_mfma.h"

namespace twn {

namespace {

constexpr int kProblemsMax = 4;
constexpr int kQuadRow = 544;               // bytes of one block of 32 pixels x 4 channels of a partial tile in LDS (padded)
constexpr int kPartTile = 8 * kQuadRow;     // one 32x32 partial tile
constexpr int kQuadRow16 = 272;             // ... of 16 pixels x 4 channels

int64_t small_x_bytes(const GatherGemm& g) {
    const int64_t in_rows = g.plain_gemm ? g.M : (g.M / (static_cast<int64_t>(g.OH) * g.OW)) * g.IH * g.IW;
    return ((in_rows - 1) * g.xs + (g.plain_gemm ? g.K : g.IC)) * 2;
}

struct SmallProblem {
    GatherGemm g;
    FastDivU divIC, divS, divOW, divOH, divUV, divV, divTN, divRG;
    uint32_t x_bytes, w_bytes;
    uint32_t blocks, tiles_n;
};

template <int NP>
struct SmallArgs {
    SmallProblem p[NP];
};

enum SmallMode : int {
    kSmallGemm = 0,     // rows of X are the reduction rows
    kSmallTap = 1,      // channel count a multiple of 64: a slab lies in one tap
    kSmallChunk = 2,    // channel count a multiple of 8: every 16-byte chunk finds its own tap
    kSmallTapDiv = 3,   // the same two with taps divided by a stride (strided backward-data)
    kSmallChunkDiv = 4,
};

// Bytes of LDS one wave uses: DEPTH slabs of activations and two groups of four slabs of codes.
constexpr int small_wave_bytes(int mt, int nt, int depth, bool h16) { return depth * mt * (h16 ? 2048 : 4096) + 2 * nt * 2048; }

template <int MT, int NT, int NW, int MODE_, int NP, int DEPTH, bool H16, bool ALPHA>
__global__ __launch_bounds__(64 * NW) void conv_small_kernel(const SmallArgs<NP> args) {
    constexpr bool DIV = MODE_ >= kSmallTapDiv;
    constexpr int MODE = DIV ? MODE_ - 2 : MODE_;
    constexpr int BM = H16 ? 16 : 32 * MT, BN = 32 * NT;
    constexpr int QUADS = BM * BN / 4;                          // groups of four channels of one pixel
    constexpr int QPT = QUADS > 64 * NW ? QUADS / (64 * NW) : 1;
    constexpr int STAGE = BM * 128;                             // one slab of activations: BM rows of 128 bytes
    constexpr int CODES = NT * 2048;                            // four slabs of codes: BN rows of 64 bytes
    constexpr int WAVE_BYTES = small_wave_bytes(MT, NT, DEPTH, H16);
    constexpr int NA = BM / 8, NB = 2 * NT;                     // loads of a slab / of a group of codes
    static_assert(WAVE_BYTES >= (H16 ? NT * 8 * kQuadRow16 : MT * NT * kPartTile), "the partial tile reuses the wave's own staging memory");
    static_assert(DEPTH >= 2 && DEPTH <= 5, "a wait spans at most one group of codes, and a group is requested when the one before the last is done");
    static_assert(!H16 || (MT == 1 && !ALPHA), "16-row tiles");
    extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];

    const SmallProblem& a = args.p[NP == 1 ? 0 : blockIdx.y];
    if (NP > 1 && blockIdx.x >= a.blocks) return;               // whole workgroup, before any barrier
    const GatherGemm& g = a.g;
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int lrow = lane & 31, lh = lane >> 5;

    // workgroups are dealt round-robin to the 8 XCDs; give each XCD a contiguous range of tiles
    const uint32_t nb = a.blocks, b = blockIdx.x;
    const uint32_t q = nb >> 3, r = nb & 7, xcd = b & 7, idx = b >> 3;
    const uint32_t t = (xcd < r) ? xcd * (q + 1) + idx : r * (q + 1) + (xcd - r) * q + idx;
    const uint32_t tm = fdiv_u(t, a.divTN);
    const uint32_t m0 = tm * BM;
    const int n0 = static_cast<int>((t - tm * a.tiles_n) * BN);

    const __amdgpu_buffer_rsrc_t rx = make_rsrc(g.X, a.x_bytes), rw = make_rsrc(g.Wq, a.w_bytes);

    // ---- what the output needs besides the sums: requested first, used last ----
    // Output group `i` of this thread: four consecutive channels of one pixel.  Every load is of an element that exists (columns
    // behind the last one take its parameters), no branch is a lane's own, and nothing is computed from a value here: with a branch and
    // a product per column the compiler waited for the memory four times, one column after the other, before the first slab was
    // requested (up to 2 us of a launch: batch-1 ResNet-18, 18 launches, 119 -> 104 us).
    const bool vec = (g.NC % 8 == 0) && (g.ldy % 8 == 0);
    const bool f32_res = g.residual && vec && g.y_f32, bf16_res = g.residual && vec && !g.y_f32;
    const bool one_alpha = g.rows_per_group >= g.NC;
    const float alpha0 = g.alpha[0];
    f32x4 c_alpha[QPT], c_scale[QPT], c_shift[QPT];
    int64_t yoff[QPT];
    int ncol0[QPT];
    u32x2 res16[QPT];
    f32x4 res32[QPT];
    auto params = [&](const float* v, int col) __attribute__((always_inline)) -> f32x4 {
        f32x4 r;
#pragma unroll
        for (int e = 0; e < 4; ++e) r[e] = v[col + e < g.NC ? col + e : g.NC - 1];
        return r;
    };
#pragma unroll
    for (int i = 0; i < QPT; ++i) {
        const int qd = i * 64 * NW + tid;                       // [pixel][BN / 4]
        const uint32_t m = m0 + qd / (BN / 4);
        ncol0[i] = n0 + (qd % (BN / 4)) * 4;
        if (qd >= QUADS || m >= static_cast<uint32_t>(g.M)) ncol0[i] = g.NC;
        if (!one_alpha) {
#pragma unroll
            for (int e = 0; e < 4; ++e)
                c_alpha[i][e] = g.alpha[fdiv_u(static_cast<uint32_t>(ncol0[i] + e < g.NC ? ncol0[i] + e : g.NC - 1), a.divRG)];
        }
        if (g.scale) c_scale[i] = params(g.scale, ncol0[i]);
        if (g.shift) c_shift[i] = params(g.shift, ncol0[i]);
        int64_t orow = m;
        if (g.orU != 0) {
            const uint32_t n = fdiv_u(m, a.divUV);
            const uint32_t rem = m - n * static_cast<uint32_t>(g.orU * g.orV);
            const uint32_t u = fdiv_u(rem, a.divV);
            const uint32_t v = rem - u * static_cast<uint32_t>(g.orV);
            orow = (static_cast<int64_t>(n) * g.orH + g.ora + g.orsh * static_cast<int>(u)) * g.orW + g.orb + g.orsw * static_cast<int>(v);
        }
        yoff[i] = orow * g.ldy + ncol0[i];
        const int64_t ro = ncol0[i] < g.NC ? yoff[i] : 0;
        if (bf16_res) res16[i] = *reinterpret_cast<const u32x2*>(static_cast<const uint16_t*>(g.residual) + ro);
        if (f32_res) res32[i] = *reinterpret_cast<const f32x4*>(static_cast<const float*>(g.residual) + ro);
    }

    // ---- addresses: load i of a slab covers rows 8i .. 8i+7 (eight lanes each); LDS row r keeps logical 16-byte
    // chunk c at position c ^ ((r >> 1) & 7), so that 16 rows of one chunk fall in 16 different bank groups ----
    const int kc[2] = {(lane & 7) ^ ((lane >> 4) & 3), (lane & 7) ^ (4 + ((lane >> 4) & 3))};   // rows of even / odd i
    uint32_t base[NA];              // byte offset of the row (GEMM) or first pixel of its image (convolution)
    int ih0[NA], iw0[NA];
#pragma unroll
    for (int i = 0; i < NA; ++i) {
        const uint32_t m = m0 + i * 8 + (lane >> 3);
        const bool ok = m < static_cast<uint32_t>(g.M);
        if constexpr (MODE == kSmallGemm) {
            base[i] = ok ? m * static_cast<uint32_t>(g.xs) * 2u : kBufOutside;
            ih0[i] = iw0[i] = 0;
        } else {
            const uint32_t tt = fdiv_u(m, a.divOW);
            const int ow = static_cast<int>(m - tt * static_cast<uint32_t>(g.OW));
            const uint32_t img = fdiv_u(tt, a.divOH);
            const int oh = static_cast<int>(tt - img * static_cast<uint32_t>(g.OH));
            base[i] = img * static_cast<uint32_t>(g.IH) * static_cast<uint32_t>(g.IW);
            ih0[i] = ok ? oh * g.sh - g.ph : -(1 << 28);
            iw0[i] = ow * g.sw - g.pw;
        }
    }
    // codes: load i of a group covers channels 16i .. 16i+15 (four lanes each, 64 bytes = four slabs of a channel);
    // the slab of position c in row r is c ^ ((r >> 2) & 3)
    uint32_t boff[NB];
#pragma unroll
    for (int i = 0; i < NB; ++i) {
        const int row = i * 16 + (lane >> 2);
        const int col = n0 + row;
        boff[i] = (col < g.NC) ? static_cast<uint32_t>(col) * static_cast<uint32_t>(g.wpr) * 4u + ((lane & 3) ^ ((row >> 2) & 3)) * 16u
                               : kBufOutside;
    }

    // this wave's slabs: a contiguous range
    const int KT = k_slabs(g.K);
    const int per = (KT + NW - 1) / NW;
    const int s0 = wave * per;
    const int ns = (s0 + per <= KT) ? per : (KT > s0 ? KT - s0 : 0);
    unsigned char* mine = smem + wave * WAVE_BYTES;
    const uint32_t lds_mine = static_cast<uint32_t>(reinterpret_cast<uintptr_t>(
        (__attribute__((address_space(3))) unsigned char*)mine));

    auto tap_offset = [&](int i, int rr, int ss, int c, bool kok) __attribute__((always_inline)) -> uint32_t {
        int th = ih0[i] + rr * g.dh, tw = iw0[i] + ss * g.dw;
        bool ok = kok;
        if constexpr (DIV) {
            if (g.divh > 1) {       // wave-uniform: strided backward-data
                const int d = th / g.divh;
                ok = ok & (th >= 0) & (d * g.divh == th);
                th = d;
            }
            if (g.divw > 1) {
                const int d = tw / g.divw;
                ok = ok & (tw >= 0) & (d * g.divw == tw);
                tw = d;
            }
        }
        ok = ok & (static_cast<unsigned>(th) < static_cast<unsigned>(g.IH)) & (static_cast<unsigned>(tw) < static_cast<unsigned>(g.IW));
        const uint32_t off = ((base[i] + static_cast<uint32_t>(th * g.IW + tw)) * static_cast<uint32_t>(g.xs) + c) * 2u;
        return ok ? off : kBufOutside;
    };
    // slab s of the range -> stage st (and, with the first slab of a group, the codes of the group)
    auto fetch = [&](int s, int st) __attribute__((always_inline)) {
        const int kt = s0 + s;
        if ((s & 3) == 0) {
            unsigned char* dst = mine + DEPTH * STAGE + ((s >> 2) & 1) * CODES;
#pragma unroll
            for (int i = 0; i < NB; ++i) buf_dma16(rw, boff[i], static_cast<uint32_t>(kt) * 16u, dst + i * 1024);
        }
        unsigned char* dst = mine + st * STAGE;
        if constexpr (MODE == kSmallGemm) {
#pragma unroll
            for (int i = 0; i < NA; ++i) {
                const int k = kt * 64 + kc[i & 1] * 8;
                buf_dma16(rx, k < g.K ? base[i] + static_cast<uint32_t>(k) * 2u : kBufOutside, 0u, dst + i * 1024);
            }
        } else if constexpr (MODE == kSmallTap) {
            const uint32_t rs = fdiv_u(static_cast<uint32_t>(kt) * 64u, a.divIC);         // wave-uniform
            const int c = kt * 64 - static_cast<int>(rs) * g.IC;
            const int rr = static_cast<int>(fdiv_u(rs, a.divS));
            const int ss = static_cast<int>(rs) - rr * g.S;
#pragma unroll
            for (int i = 0; i < NA; ++i) buf_dma16(rx, tap_offset(i, rr, ss, c + kc[i & 1] * 8, true), 0u, dst + i * 1024);
        } else {
            int c[2], rr[2], ss[2];
            bool kok[2];
#pragma unroll
            for (int e = 0; e < 2; ++e) {
                const int k = kt * 64 + kc[e] * 8;
                const uint32_t rs = fdiv_u(static_cast<uint32_t>(k), a.divIC);
                c[e] = k - static_cast<int>(rs) * g.IC;
                rr[e] = static_cast<int>(fdiv_u(rs, a.divS));
                ss[e] = static_cast<int>(rs) - rr[e] * g.S;
                kok[e] = k < g.K;
            }
#pragma unroll
            for (int i = 0; i < NA; ++i)
                buf_dma16(rx, tap_offset(i, rr[i & 1], ss[i & 1], c[i & 1], kok[i & 1]), 0u, dst + i * 1024);
        }
    };

    f32x16 acc[MT][NT];
    f32x4 acc16[2 * NT];            // H16: blocks of 16 channels
#pragma unroll
    for (int cb = 0; cb < 2 * NT; ++cb) acc16[cb] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
    for (int mi = 0; mi < MT; ++mi)
#pragma unroll
        for (int ni = 0; ni < NT; ++ni)
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[mi][ni][e] = 0.0f;

    // the terms of alpha_in: [term][channel], whole slabs; requested before the first slabs, written after
    const int span = (g.IC + 63) & ~63;
    uint16_t* const terms = reinterpret_cast<uint16_t*>(smem + NW * WAVE_BYTES);
    const uint32_t lds_terms = static_cast<uint32_t>(reinterpret_cast<uintptr_t>(
        (__attribute__((address_space(3))) unsigned char*)(smem + NW * WAVE_BYTES)));
    float my_alpha = 0.0f;
    if constexpr (ALPHA) {
        if (tid < g.IC) my_alpha = g.alpha_in[tid / g.alpha_in_rows];
    }

#pragma unroll
    for (int d = 0; d < DEPTH; ++d)
        if (d < ns) fetch(d, d);

    if constexpr (ALPHA) {
        for (int c = tid; c < span; c += 64 * NW) {
            const float v = c == tid ? my_alpha : (c < g.IC ? g.alpha_in[c / g.alpha_in_rows] : 0.0f);
            uint16_t t[kAlphaTerms];
            alpha_terms(v, t);
#pragma unroll
            for (int k = 0; k < kAlphaTerms; ++k) terms[k * span + c] = t[k];
        }
        __syncthreads();
    }

    uint32_t aoff[4];               // this lane's fragment of step kk inside a stage (row lrow; the next 32 rows: + 4096)
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) aoff[kk] = lds_mine + lrow * 128 + (((lh * 4 + kk) ^ ((lrow >> 1) & 7)) * 16);

    int st = 0;
    for (int sg = 0; sg < ns; sg += 4) {
        static_for<4>([&](auto p_tag) __attribute__((always_inline)) {
            constexpr int p = decltype(p_tag)::value;
            const int s = sg + p;
            if (s >= ns) return;                                // wave-uniform
            // slab s (and its codes) landed: younger loads may stay in flight, unless the range ends before them
            if (s + DEPTH - 1 < ns) {
                constexpr int younger = (DEPTH - 1) * NA + ((p + DEPTH - 1 >= 4) ? NB : 0);
                asm volatile("s_waitcnt vmcnt(%0)" ::"n"(younger) : "memory");
            } else {
                asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
            }
            if constexpr (H16) {
                // Lane group q = lane / 16 holds k = 16q .. 16q+15 of the slab, one word of codes per channel: eight k to each of two MFMAs.
                const int r16 = lane & 15, q4 = lane >> 4;
                uint32_t cw[2 * NT];
                u32x4 x2[2];
                const uint32_t cbase = lds_mine + DEPTH * STAGE + ((sg >> 2) & 1) * CODES + r16 * 64 + ((p ^ ((r16 >> 2) & 3)) * 16) + q4 * 4;
                static_for<2 * NT>([&](auto c_tag) __attribute__((always_inline)) {
                    constexpr int cb = decltype(c_tag)::value;
                    lds_read32<cb * 1024>(cw[cb], cbase);
                });
                const uint32_t xbase = lds_mine + st * STAGE + r16 * 128 + (((q4 * 2) ^ ((r16 >> 1) & 7)) * 16);
                lds_read128<0>(x2[0], xbase);
                lds_read128<0>(x2[1], xbase ^ 16);
                lds_wait<0>();
                lds_ready<2 * NT>(cw);
                lds_ready<2>(x2);
                if (s + DEPTH < ns) fetch(s + DEPTH, st);           // every read of this stage has returned
#pragma unroll
                for (int kk = 0; kk < 2; ++kk)
#pragma unroll
                    for (int cb = 0; cb < 2 * NT; ++cb) {
                        u32x4 wf;
#pragma unroll
                        for (int e = 0; e < 4; ++e) {
                            const int i = kk * 4 + e;
                            wf[e] = (cw[cb] & (0xC000C000u >> (14 - 2 * i))) << (14 - 2 * i);
                        }
                        acc16[cb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, wf), __builtin_bit_cast(bf16x8, x2[kk]),
                                                                            acc16[cb], 0, 0, 0);
                    }
                st = (st + 1 == DEPTH) ? 0 : st + 1;
                return;
            }
            u32x2 w[NT];
            u32x4 x[4][MT];
            u32x4 al[4][kAlphaTerms];
            constexpr int TERMS = ALPHA ? kAlphaTerms : 1;
            constexpr int READS = MT + (ALPHA ? TERMS : 0);         // of a step
            const uint32_t cbase = lds_mine + DEPTH * STAGE + ((sg >> 2) & 1) * CODES + lrow * 64 + lh * 8 + ((p ^ ((lrow >> 2) & 3)) * 16);
            lds_read64_n<NT, 32 * 64>(w, cbase);
#pragma unroll
            for (int kk = 0; kk < 4; ++kk) {
                lds_read128_n<MT, 4096>(x[kk], aoff[kk] + st * STAGE);
                if constexpr (ALPHA) {
                    // reduction channel of this half's chunk
                    uint32_t c = static_cast<uint32_t>((s0 + s) * 64 + (lh * 4 + kk) * 8);
                    if constexpr (MODE == kSmallTap) {
                        const uint32_t first = static_cast<uint32_t>(s0 + s) * 64u;          // wave-uniform
                        c -= fdiv_u(first, a.divIC) * static_cast<uint32_t>(g.IC);
                    } else if constexpr (MODE == kSmallChunk) {
                        c -= fdiv_u(c, a.divIC) * static_cast<uint32_t>(g.IC);
                    }
#pragma unroll
                    for (int k = 0; k < TERMS; ++k)
                        lds_read128<0>(al[kk][k], lds_terms + static_cast<uint32_t>(k * span + static_cast<int>(c)) * 2u);
                }
            }
            static_for<4>([&](auto kk_tag) __attribute__((always_inline)) {
                constexpr int kk = decltype(kk_tag)::value;
                lds_wait<(3 - kk) * READS>();
                if constexpr (kk == 0) lds_ready<NT>(w);
                lds_ready<MT>(x[kk]);
                if constexpr (ALPHA) lds_ready<TERMS>(al[kk]);
                if constexpr (kk == 3) {
                    if (s + DEPTH < ns) fetch(s + DEPTH, st);   // every read of this stage has returned
                }
                u32x4 wf[TERMS][NT];
#pragma unroll
                for (int ni = 0; ni < NT; ++ni)
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        constexpr int half = (kk & 1) * 4;
                        const int i = half + e;                 // field i of both half-words -> bits [14,15] of two bf16
                        if constexpr (ALPHA) {
                            typedef short s16x2 __attribute__((ext_vector_type(2)));
                            const uint32_t f = w[ni][kk >> 1] << (14 - 2 * i), sign = f & 0x80008000u;
                            const uint32_t on = __builtin_bit_cast(uint32_t, __builtin_bit_cast(s16x2, f << 1) >> 15);
#pragma unroll
                            for (int k = 0; k < TERMS; ++k) wf[k][ni][e] = (al[kk][k][e] & on) ^ sign;
                        } else {
                            wf[0][ni][e] = (w[ni][kk >> 1] & (0xC000C000u >> (14 - 2 * i))) << (14 - 2 * i);
                        }
                    }
#pragma unroll
                for (int mi = 0; mi < MT; ++mi)
#pragma unroll
                    for (int ni = 0; ni < NT; ++ni)
#pragma unroll
                        for (int k = 0; k < TERMS; ++k)
                            acc[mi][ni] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, wf[k][ni]),
                                                                                  __builtin_bit_cast(bf16x8, x[kk][mi]),
                                                                                  acc[mi][ni], 0, 0, 0);
            });
            st = (st + 1 == DEPTH) ? 0 : st + 1;
        });
    }

    // ---- partial tiles -> LDS, each wave over its own staging memory: [mi][ni][q4*2 + lh][pixel] of four channels ----
    if constexpr (H16) {
#pragma unroll
        for (int cb = 0; cb < 2 * NT; ++cb)
            *reinterpret_cast<f32x4*>(mine + (cb * 4 + (lane >> 4)) * kQuadRow16 + (lane & 15) * 16) = acc16[cb];
    } else
#pragma unroll
    for (int mi = 0; mi < MT; ++mi)
#pragma unroll
        for (int ni = 0; ni < NT; ++ni)
#pragma unroll
            for (int q4 = 0; q4 < 4; ++q4) {
                unsigned char* dst = mine + (mi * NT + ni) * kPartTile + (q4 * 2 + lh) * kQuadRow + lrow * 16;
                *reinterpret_cast<f32x4*>(dst) = f32x4{acc[mi][ni][q4 * 4], acc[mi][ni][q4 * 4 + 1], acc[mi][ni][q4 * 4 + 2],
                                                       acc[mi][ni][q4 * 4 + 3]};
            }
    __syncthreads();

    // ---- sum in wave order, y = relu?((alpha*acc)*scale + shift + residual) ----
#pragma unroll
    for (int i = 0; i < QPT; ++i) {
        if (ncol0[i] >= g.NC) continue;
        const int qd = i * 64 * NW + tid;
        const int pix = qd / (BN / 4), c4 = qd % (BN / 4);
        const unsigned char* src = H16 ? smem + c4 * kQuadRow16 + pix * 16
                                       : smem + ((pix >> 5) * NT + (c4 >> 3)) * kPartTile + (c4 & 7) * kQuadRow + (pix & 31) * 16;
        f32x4 s = *reinterpret_cast<const f32x4*>(src);
#pragma unroll
        for (int w = 1; w < NW; ++w) s += *reinterpret_cast<const f32x4*>(src + w * WAVE_BYTES);
        float v[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            // codes were +-2
            const float mul = (ALPHA ? 1.0f : 0.5f * (one_alpha ? alpha0 : c_alpha[i][e])) * (g.scale ? c_scale[i][e] : 1.0f);
            v[e] = s[e] * mul + (g.shift ? c_shift[i][e] : 0.0f);
        }
        if (vec && !g.y_f32) {
            if (g.residual) {
                v[0] += __uint_as_float(res16[i][0] << 16);
                v[1] += __uint_as_float(res16[i][0] & 0xFFFF0000u);
                v[2] += __uint_as_float(res16[i][1] << 16);
                v[3] += __uint_as_float(res16[i][1] & 0xFFFF0000u);
            }
            if (g.relu) {
#pragma unroll
                for (int e = 0; e < 4; ++e) v[e] = fmaxf(v[e], 0.0f);
            }
            u32x2 pk;
            pk[0] = pack_bf16x2(v[0], v[1]);
            pk[1] = pack_bf16x2(v[2], v[3]);
            *reinterpret_cast<u32x2*>(static_cast<uint16_t*>(g.Y) + yoff[i]) = pk;
        } else if (vec) {
            if (g.residual) {
#pragma unroll
                for (int e = 0; e < 4; ++e) v[e] += res32[i][e];
            }
            if (g.relu) {
#pragma unroll
                for (int e = 0; e < 4; ++e) v[e] = fmaxf(v[e], 0.0f);
            }
            *reinterpret_cast<f32x4*>(static_cast<float*>(g.Y) + yoff[i]) = f32x4{v[0], v[1], v[2], v[3]};
        } else {
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                if (ncol0[i] + e >= g.NC) continue;
                const int64_t off = yoff[i] + e;
                if (g.y_f32) {
                    if (g.residual) v[e] += static_cast<const float*>(g.residual)[off];
                    if (g.relu) v[e] = fmaxf(v[e], 0.0f);
                    static_cast<float*>(g.Y)[off] = v[e];
                } else {
                    if (g.residual) v[e] += bf16_to_f32(static_cast<const uint16_t*>(g.residual)[off]);
                    if (g.relu) v[e] = fmaxf(v[e], 0.0f);
                    static_cast<uint16_t*>(g.Y)[off] = f32_to_bf16(v[e]);
                }
            }
        }
    }
}

int small_mode(const GatherGemm& g) {
    if (g.plain_gemm) return kSmallGemm;
    const int mode = (!g.chunk_gather && g.IC % 64 == 0) ? kSmallTap : kSmallChunk;
    return g.divh > 1 || g.divw > 1 ? mode + 2 : mode;
}

SmallProblem make_problem(const GatherGemm& g, int bm, int bn) {
    SmallProblem p;
    p.g = g;
    p.divIC = make_fastdiv_u(static_cast<uint32_t>(g.IC));
    p.divS = make_fastdiv_u(static_cast<uint32_t>(g.S));
    p.divOW = make_fastdiv_u(static_cast<uint32_t>(g.OW));
    p.divOH = make_fastdiv_u(static_cast<uint32_t>(g.OH));
    p.divUV = make_fastdiv_u(g.orU ? static_cast<uint32_t>(g.orU) * static_cast<uint32_t>(g.orV) : 1u);
    p.divV = make_fastdiv_u(g.orU ? static_cast<uint32_t>(g.orV) : 1u);
    p.x_bytes = static_cast<uint32_t>(small_x_bytes(g));
    p.w_bytes = static_cast<uint32_t>(static_cast<int64_t>(g.NC) * g.wpr * 4);
    p.tiles_n = static_cast<uint32_t>((g.NC + bn - 1) / bn);
    p.divTN = make_fastdiv_u(p.tiles_n);
    p.divRG = make_fastdiv_u(static_cast<uint32_t>(g.rows_per_group));
    p.blocks = static_cast<uint32_t>((g.M + bm - 1) / bm) * p.tiles_n;
    return p;
}

template <int MT, int NT, int NW, int MODE, int NP, bool ALPHA, bool H16>
int32_t launch_small_build(const SmallArgs<NP>& a, uint32_t width, int count, hipStream_t st) {
    // the table of terms takes the third slab's place where both do not fit
    constexpr int DEPTH = H16 ? 5 : ALPHA && NT == 2 ? 2 : 3;
    constexpr int STAGES = NW * small_wave_bytes(MT, NT, DEPTH, H16);
    constexpr int MOST = STAGES + (ALPHA ? kSmallAlphaMax * 2 * kAlphaTerms : 0);
    static_assert(MOST <= 160 * 1024, "LDS budget");
    const int SMEM = STAGES + (ALPHA ? ((a.p[0].g.IC + 63) & ~63) * 2 * kAlphaTerms : 0);
    auto k = conv_small_kernel<MT, NT, NW, MODE, NP, DEPTH, H16, ALPHA>;
    // more than 64 KB of dynamic LDS has to be allowed once per kernel
    static std::once_flag once;
    static bool allowed = false;
    std::call_once(once, [&] {
        allowed = hipFuncSetAttribute(reinterpret_cast<const void*>(k), hipFuncAttributeMaxDynamicSharedMemorySize,
                                      MOST) == hipSuccess;
    });
    if (!allowed) return TWN_ERR_HIP;
    k<<<dim3(width, static_cast<unsigned>(count)), dim3(64 * NW), SMEM, st>>>(a);
    return launch_status();
}

template <int MT, int NT, int NW, bool H16, int MODE, int NP>
int32_t launch_small_kernel(const SmallArgs<NP>& a, uint32_t width, int count, hipStream_t st) {
    if (!a.p[0].g.alpha_in) return launch_small_build<MT, NT, NW, MODE, NP, false, H16>(a, width, count, st);
    if constexpr (!H16) {
        if (a.p[0].g.IC <= kSmallAlphaMax) return launch_small_build<MT, NT, NW, MODE, NP, true, false>(a, width, count, st);
    }
    return TWN_ERR_UNSUPPORTED;
}

template <int MT, int NT, int NW, bool H16 = false>
int32_t launch_small_tile(const GatherGemm* gs, int count, hipStream_t st) {
    if (count == 1) {
        SmallArgs<1> a;
        a.p[0] = make_problem(gs[0], H16 ? 16 : 32 * MT, 32 * NT);
        const uint32_t width = a.p[0].blocks;
        switch (small_mode(gs[0])) {
            case kSmallGemm: return launch_small_kernel<MT, NT, NW, H16, kSmallGemm, 1>(a, width, 1, st);
            case kSmallTap: return launch_small_kernel<MT, NT, NW, H16, kSmallTap, 1>(a, width, 1, st);
            case kSmallChunk: return launch_small_kernel<MT, NT, NW, H16, kSmallChunk, 1>(a, width, 1, st);
            case kSmallTapDiv: return launch_small_kernel<MT, NT, NW, H16, kSmallTapDiv, 1>(a, width, 1, st);
            default: return launch_small_kernel<MT, NT, NW, H16, kSmallChunkDiv, 1>(a, width, 1, st);
        }
    }
    SmallArgs<kProblemsMax> a{};
    uint32_t width = 0;
    bool tap = true;
    for (int c = 0; c < count; ++c) {
        a.p[c] = make_problem(gs[c], H16 ? 16 : 32 * MT, 32 * NT);
        if (a.p[c].blocks > width) width = a.p[c].blocks;
        tap = tap && gs[c].IC % 64 == 0 && !gs[c].chunk_gather;
    }
    return tap ? launch_small_kernel<MT, NT, NW, H16, kSmallTap, kProblemsMax>(a, width, count, st)
               : launch_small_kernel<MT, NT, NW, H16, kSmallChunk, kProblemsMax>(a, width, count, st);
}

}  // namespace

// Tile (16 or 32 pixels x 32 or 64 channels, number of waves: 608, 1108, 1208, 1204) for `count` problems in one launch, 0 when the
// other kernels are better or the shapes do not fit.  The lines are multiples of the 256 CUs of the chip they were measured on and no
// question to the device: the workspace query has to give the same answer without one.  Measured per dependent launch (us, against the split-K launch pair
// and the persistent kernels that ran such problems before):
//   * up to 256 tiles of 16 pixels by 32 channels (one alpha; MFMAs of 16x16): eight waves per tile.  The tiles of a batch-1 layer
//     leave most CUs idle, and the ones at work are bound by what their own load path brings: half the rows are half of that,
//     and five slabs in flight fit where three of 32 rows did (49, 512, 4608: 7.7 -> 6.8; 196, 256, 2304: 5.9 -> 5.2).  Against tiles
//     of 32 pixels in 504 inner products of 1 to 500 rows, 10 to 8192 columns and K of 64 to 16384: 0.97 to 1.18 times as fast, 1.07 in
//     the mean, also where rows above the sixteenth read the codes again (1, 1000, 512: 3.56 -> 3.31; 16, 8192, 16384: 16.2 -> 14.1; 32,
//     4096, 16384: 14.4 -> 14.1; 24, 4096, 512: 3.56 -> 3.63; 500, 256, 4096: 6.04 -> 5.80).  Several problems in one launch count as the
//     largest each: residue classes of 195 tiles in a grid of 300 took a second round (13x11x9 <- 512, 96 channels 2x2/2: 8.9, with tiles of 32
//     pixels 7.2)
//   * up to 256 tiles of 32x32: eight waves per tile, one tile per CU (M, N, K = 49, 512, 4608: 10.8 -> 8.1; 784, 128, 1152:
//     11.6 -> 5.1; 1, 1000, 512: 5.1 -> 3.6).  Two such workgroups do not fit a CU: 1568, 256, 2304, 392 tiles of 32x32 or
//     196 of 32x64, takes 8.1 with the former and 6.4 with the latter
//   * up to 256 tiles of 32x64: eight waves (784, 512, 4608: 25.9 -> 10.7).  Above that
//   * up to 512 tiles of 32x64: four waves, two workgroups per CU (3136, 256, 2304: 26.2 -> 11.7), where the persistent
//     kernels cannot run (channel counts that are no multiple of 64, float32 outputs, divided taps: 13.8 -> 7.2) or K has
//     at least 16 slabs; with shorter K they win (6272, 128, 576: 6.4 against 7.5).
// Beyond 512 tiles the other kernels' larger tiles win (12544, 128, 1152: 8.9 against 16.4), and beyond K = 16384 one
// workgroup per tile is too few for the loads: K ranges over several workgroups win (64, 64, 32768: 15.2 against 22.8;
// 128, 128, 16384: 13.2 against 13.0).
int conv_small_tile(const GatherGemm* gs, int count) {
    if (count < 1 || count > kProblemsMax || env_int(Env::SMALL, 1) == 0) return 0;
    // an override that names or shapes another kernel means problems of every size
    if (env_int(Env::TILE, 0) != 0 || env_int(Env::STREAM, 1) == 0 || env_int(Env::BUFLOAD, 1) == 0 || env_set(Env::STREAM_KS) ||
        env_set(Env::STREAM_PC) || env_set(Env::STREAM_PC_STAGES) || env_set(Env::STREAM_OCC))
        return 0;
    int64_t t16 = 0, t11 = 0, t12 = 0;
    bool persistent = true, one_alpha = true;
    int kt = 0;
    for (int c = 0; c < count; ++c) {
        const GatherGemm& g = gs[c];
        if (!g.chunk_gather && (g.IC % 8 != 0 || g.xs % 8 != 0)) return 0;
        if (g.M <= 0 || g.M >= (1LL << 31) - 128) return 0;
        if (count > 1 && (g.divh > 1 || g.divw > 1)) return 0;      // several problems have undivided builds only
        if (!g.plain_gemm && g.M % (static_cast<int64_t>(g.OH) * g.OW) != 0) return 0;
        const int64_t xb = small_x_bytes(g), wb = static_cast<int64_t>(g.NC) * g.wpr * 4;
        if (xb <= 0 || xb >= (1LL << 31) || wb >= (1LL << 31)) return 0;
        const int64_t rows = (g.M + 31) / 32;
        const int64_t tiles16 = (g.M + 15) / 16 * ((g.NC + 31) / 32);
        if (tiles16 > t16) t16 = tiles16;
        t11 += rows * ((g.NC + 31) / 32);
        one_alpha = one_alpha && !g.alpha_in;
        t12 += rows * ((g.NC + 63) / 64);
        const bool slabs = g.plain_gemm ? g.K % 64 == 0 : (g.IC % 64 == 0 && g.divh == 1 && g.divw == 1 && g.orU == 0);
        persistent = persistent && slabs && !g.y_f32 && g.NC % 8 == 0 && g.ldy % 8 == 0 && !g.chunk_gather;
        if (k_slabs(g.K) > kt) kt = k_slabs(g.K);
    }
    if (kt > 256) return 0;
    if (t16 * count <= 256 && one_alpha) return 608;        // each problem has as many workgroups as the largest
    if (t11 <= 256) return 1108;
    if (t12 <= 256) return 1208;
    if (t12 <= 512 && (kt >= 16 || !persistent)) return 1204;
    return 0;
}

int32_t launch_conv_small(const GatherGemm* gs, int count, int tile, hipStream_t st) {
    switch (tile) {
        case 608: return launch_small_tile<1, 1, 8, true>(gs, count, st);
        case 1108: return launch_small_tile<1, 1, 8>(gs, count, st);
        case 1208: return launch_small_tile<1, 2, 8>(gs, count, st);
        case 1204: return launch_small_tile<1, 2, 4>(gs, count, st);
        default: return TWN_ERR_UNSUPPORTED;
    }
}

}  // namespace twn
