// Persistent implicit-GEMM ternary convolution / inner product with dedicated load waves, gfx950
// (Eq. 2, Alg. 1 step 8; also the undivided backward-data pass of Alg. 1 step 9).
//
// Arithmetic, tile walk and epilogue are those of conv_stream_kernel.  What differs is who issues the
// direct-to-LDS loads.  A wave needs about 64 cycles to issue one 16-byte-per-lane buffer load to LDS and the
// few vector instructions that form its address, and it issues in order: in a kernel whose waves both load and
// multiply, a slab of a 128x128 tile costs a wave 5 loads = 320+ cycles during which it starts no MFMA, next to
// 512 cycles of MFMA work (measured: steps that carry loads take 300-500 cycles, the others about 100).  Here
// four extra waves per workgroup do nothing but stage slabs (each takes every fourth 1 KB load of a slab), and
// the WM*WN compute waves never touch vector memory in the main loop: their instruction stream is MFMAs,
// fragment reads and code expansion only.  Hand-over per slab, as before, is one s_barrier: a load wave waits
// for its own loads of the next slab (s_waitcnt vmcnt) before it arrives, a compute wave arrives in the middle
// of the current slab; after the barrier the load waves refill the stage of the previous slab.  Four stages,
// so that a load has two slab times to land.
//
// What a wave issues per slab is what bounds it.  A load wave that formed every address anew and fetched codes 16 bytes per
// filter (64 cache lines touched by one load) took 400 cycles for three loads, against 256 of MFMA work in a slab of a 64x128
// tile.  So the per-lane part of an address is formed once per filter tap (the channel slab travels in the scalar offset), the rows of
// a tap are tested once per row of taps, the scalar state advances by additions, and
// codes come in chunks of CS slabs, CS*16 contiguous bytes per filter (16 or 32 lines per load, and lines of 128 bytes are fetched
// from L2 that much less often); there are three chunk buffers, so that a chunk is requested together with the activations of its first
// slab whatever the lengths of its neighbours at a tile's end.  In a compute wave, eight MFMAs alone take 265 cycles, with four
// independent vector instructions after each (the expansion of a 64-row wave tile) 369 when every second one needs the result of the one
// before, 317 otherwise: parts of two words alternate, and scalar work sits between MFMAs too.  All of it against the
// kernel before (us, same bits): GEMM 8192x4096x4096 205 -> 195; 3x3 layers 180000 pixels, 256 -> 256 channels 164 -> 158;
// 8192, 512 -> 512 36.4 -> 32.9; 12544, 256 -> 256 18.3 -> 17.5; 50176, 128 -> 128 17.8 -> 17.0; 3136, 512 -> 512 19.7 both
// (one workgroup per CU).  Then, of a load wave's loop, the waits by nesting, one branch back per slab and 4 instead of 7 vector
// instructions per load and tap (by instruction count alone: the same addresses formed behind the loads or between them were slower): 2303
// pixels, 64 -> 512 channels 7x7 17.9 -> 15.0; 5x5 over 128 channels 16.1 -> 14.9; 3136, 512 -> 512 19.6 -> 19.0; 2303x512x3072 14.7 -> 13.9.
//
// DEEP (two MFMAs per step and wave): a step is 64 cycles, less than an LDS read takes.  Fragments lie in four sets and
// are requested a step further ahead; all reads of a slab have landed when it ends.
//
// ALPHA: backward-data with several alphas (alpha_in of the problem).  alpha of a reduction channel, as three bf16 terms
// (all of a float's 24 bits), replaces the 2 of its codes, and a fragment of dY is multiplied by each: against two terms of alpha * dY
// side by side, half the slabs, a third of the fragment reads per MFMA and no launch that scales dY, for half as many products again.
// The terms lie in LDS; a step reads those of the step after the next (the same for all lanes of a half).  dX with the scaling
// launch before (us): 64x28x28, 128 -> 128 channels 3x3 47.9 -> 46.2; 64x14x14, 128 17.9 -> 14.2; 256 45.6 -> 41.9; 64x7x7, 256
// filters over 512 25.9 -> 24.6; 1x1, 20x56x56, 512 filters over 128 53.6 -> 24.9.  Which of the two runs is decided in data_gradient.
#include <mutex>

#include "twn_kernels.h"
#include "twn_lds_asm.h"
#include "twn_mfma.h"
#include "twn_stream_epilogue.h"

namespace twn {

struct StreamPcArgs {
    GatherGemm g;
    FastDivU divOW, divOH;      // GEMM row -> (image, oh, ow)
    FastDivU divTN;             // tile -> (row block, column block)
    uint32_t x_bytes, w_bytes, y_bytes;  // sizes for the buffer descriptors
    uint32_t tiles, tiles_n;
    int32_t KT;                 // K / 64
    int32_t spt;                // 64-channel slabs per tap (IC / 64; all slabs without taps)
};

constexpr int kLoadWaves = 4;
constexpr int kCodeBufs = 3;

template <int BM, int BN, int WM, int WN, int STAGES, bool GEMM, int OCC, int CS, bool ALPHA = false>
// (the second launch bound is in waves per SIMD)
__global__ __launch_bounds__(64 * (WM * WN + kLoadWaves), (OCC * (WM * WN + kLoadWaves) + 3) / 4)
void conv_stream_pc_kernel(const StreamPcArgs a) {
    constexpr int NP = kLoadWaves;
    constexpr int NWC = WM * WN;                   // compute waves
    constexpr int TM = BM / WM, TN = BN / WN;
    constexpr int MI = TM / 32, NI = TN / 32;
    constexpr int TERMS = ALPHA ? kAlphaTerms : 1;
    constexpr bool DEEP = MI * NI * TERMS <= 2;
    constexpr int STAGE_BYTES = BM * 128;          // activations of one slab
    constexpr int CHUNK_BYTES = BN * CS * 16;      // codes of CS slabs
    constexpr int LX = BM / 8 / NP;                // 1 KB activation loads per load wave and slab
    constexpr int CR = 64 / CS;                    // filters per code load
    constexpr int LB = BN / CR / NP;               // code loads per load wave and chunk
    constexpr int EPI_CH = TN < 64 ? TN : 64;      // channels staged at a time
    constexpr int EPI_ROW = EPI_CH * 2 + 16;
    constexpr int EPI_WAVE = 32 * EPI_ROW;         // one block of 32 pixel rows per wave
    constexpr bool EPI_OWN = NWC * EPI_WAVE > STAGE_BYTES;      // output staging outside the pipeline stages
    static_assert(BM % 32 == 0 && BN % 64 == 0 && TN % 32 == 0 && TM % 32 == 0, "tile shape");
    static_assert(BM % (8 * NP) == 0 && BN % (CR * NP) == 0 && (CS == 2 || CS == 4), "whole loads for every load wave");
    static_assert((STAGE_BYTES & (STAGE_BYTES - 1)) == 0, "the stages are walked by a mask");
    static_assert(STAGES == 4, "a chunk is requested three slabs ahead, and three buffers hold at least that much");
    static_assert(BN <= 64 * NWC, "one compute thread per column loads the column parameters");
    static_assert(MI <= 8 && NI <= 4, "fragment reads use immediate offsets");
    static_assert(LB <= LX && LX + LB < 64, "waits of the load waves");

    extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];
    unsigned char* const codes = smem + STAGES * STAGE_BYTES;
    float* const colbuf = reinterpret_cast<float*>(codes + kCodeBufs * CHUNK_BYTES);        // [2][2][BN]: mul, add of even / odd tiles
    unsigned char* const epi_own = reinterpret_cast<unsigned char*>(colbuf + 4 * BN);
    uint16_t* const terms = reinterpret_cast<uint16_t*>(epi_own + (EPI_OWN ? NWC * EPI_WAVE : 0));   // ALPHA: [term][channel] of alpha_in

    const GatherGemm& g = a.g;
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);

    // ---- this workgroup's tiles (as in conv_stream_kernel: each XCD owns a contiguous range) ----
    const uint32_t G = gridDim.x, b = blockIdx.x;
    const uint32_t xcd = b & 7, j = b >> 3;
    const uint32_t gx = (G + 7 - xcd) >> 3;
    const uint32_t q = a.tiles >> 3, r = a.tiles & 7;
    const uint32_t count_x = q + (xcd < r ? 1u : 0u);
    const uint32_t start_x = xcd * q + (xcd < r ? xcd : r);
    if (j >= count_x) return;                               // whole workgroup, before any barrier
    const uint32_t n_my = (count_x - j + gx - 1) / gx;
    auto tile_id = [&](uint32_t i) __attribute__((always_inline)) -> uint32_t { return start_x + j + i * gx; };

    const int KT = a.KT;

    if (wave >= NWC) {
        // =================================== load wave ===================================
        const int p = wave - NWC;
        const __amdgpu_buffer_rsrc_t rx = make_rsrc(g.X, a.x_bytes), rw = make_rsrc(g.Wq, a.w_bytes);
        // Activations: load i is row block p + NP*i.  LDS row r keeps logical 16-byte chunk c at position c ^ ((r >> 1) & 7):
        // the swizzle is applied by choosing which chunk of the row this lane fetches.
        const int kc = (lane & 7) ^ ((p & 1) * 4 + ((lane >> 4) & 3));
        // Codes: load i is the block of CR filters p + NP*i; a filter's CS slabs lie in an order that spreads the filters over
        // the banks, chosen the same way.
        const int cq = (lane % CS) ^ ((lane / CS) / (16 / CS) % CS);
        uint32_t voff[LX];           // byte offset of the row (GEMM) / of tap (0,0) (convolution), wrapping where that lies outside
        uint32_t xcur[LX];           // ... of the present tap, kBufOutside where it lies outside the image
        // row and column of tap (0,0); the column also kNowhere while the taps' row lies outside the image, and both where there is no
        // pixel.  No tap brings kNowhere back (conv_stream_applicable).
        uint32_t ih0[LX], iw0[LX], iw[LX];
        constexpr uint32_t kNowhere = 0x80000000u;
        uint32_t coff[LB];
        auto tile_setup = [&](uint32_t t) __attribute__((always_inline)) {
            const uint32_t tm = fdiv_u(t, a.divTN);
            const uint32_t tn = t - tm * a.tiles_n;
#pragma unroll
            for (int i = 0; i < LX; ++i) {
                const uint32_t m = tm * BM + static_cast<uint32_t>((p + NP * i) * 8 + (lane >> 3));
                const bool rv = m < static_cast<uint32_t>(g.M);
                if (GEMM) {
                    xcur[i] = rv ? (m * static_cast<uint32_t>(g.xs) + static_cast<uint32_t>(kc * 8)) * 2u : kBufOutside;
                } else {
                    const uint32_t tt = fdiv_u(m, a.divOW);
                    const int ow = static_cast<int>(m - tt * static_cast<uint32_t>(g.OW));
                    const uint32_t img = fdiv_u(tt, a.divOH);
                    const int oh = static_cast<int>(tt - img * static_cast<uint32_t>(g.OH));
                    const int hh = oh * g.sh - g.ph, ww = ow * g.sw - g.pw;
                    // 32-bit wrapping arithmetic: the true offset of every tap that passes the bounds test
                    // lies in [0, 2^31)
                    const uint32_t pix = (img * static_cast<uint32_t>(g.IH) + static_cast<uint32_t>(hh)) *
                                             static_cast<uint32_t>(g.IW) + static_cast<uint32_t>(ww);
                    voff[i] = (pix * static_cast<uint32_t>(g.xs) + static_cast<uint32_t>(kc * 8)) * 2u;
                    ih0[i] = rv ? static_cast<uint32_t>(hh) : kNowhere;
                    iw0[i] = static_cast<uint32_t>(ww);
                    iw[i] = ih0[i] < static_cast<uint32_t>(g.IH) ? iw0[i] : kNowhere;
                }
            }
#pragma unroll
            for (int i = 0; i < LB; ++i) {
                const uint32_t ncol = tn * BN + static_cast<uint32_t>((p + NP * i) * CR + lane / CS);
                coff[i] = (ncol < static_cast<uint32_t>(g.NC)) ? ncol * static_cast<uint32_t>(g.wpr) * 4u + static_cast<uint32_t>(cq) * 16u
                                                               : kBufOutside;
            }
        };
        // the loads of this wave for stream position (tile lt, slab lk); returns how many they are
        uint32_t lt = 0;
        int lk = 0, ss = 0;                             // slab of the tile, tap of its row
        uint32_t soff = 0;                              // bytes of the tap's channels before the slab
        uint32_t tap_h = 0, tap_w = 0, tap_off = 0;     // the tap's offset in rows, columns, bytes (wrapping, as above)
        uint32_t fill = 0;                              // stage (bytes) and chunk buffer they go to
        int cb = 0;
        const uint32_t dh = static_cast<uint32_t>(g.dh), dw = static_cast<uint32_t>(g.dw);
        const uint32_t strS = dw * static_cast<uint32_t>(g.xs) * 2u;
        const uint32_t strR = dh * static_cast<uint32_t>(g.IW) * static_cast<uint32_t>(g.xs) * 2u - static_cast<uint32_t>(g.S) * strS;
        const uint32_t tap_bytes = static_cast<uint32_t>(a.spt) * 128u;
        auto issue = [&]() __attribute__((always_inline)) -> int {
            if (lt >= n_my) return 0;
            if (!GEMM && soff == 0) {
#pragma unroll
                for (int i = 0; i < LX; ++i)
                    xcur[i] = iw[i] + tap_w < static_cast<uint32_t>(g.IW) ? voff[i] + tap_off : kBufOutside;
            }
#pragma unroll
            for (int i = 0; i < LX; ++i) buf_dma16(rx, xcur[i], soff, smem + fill + (p + NP * i) * 1024);
            fill = (fill + STAGE_BYTES) % (STAGES * STAGE_BYTES);
            int n = LX;
            if (lk % CS == 0) {
                // slabs behind the last one are not read: at the last filter they would lie outside the tensor
                const bool in_k = lk + cq < KT;
#pragma unroll
                for (int i = 0; i < LB; ++i)
                    buf_dma16(rw, in_k ? coff[i] : kBufOutside, static_cast<uint32_t>(lk) * 16u, codes + cb * CHUNK_BYTES + (p + NP * i) * 1024);
                cb = (cb + 1 == kCodeBufs) ? 0 : cb + 1;
                n += LB;
            }
            ++lk;
            soff += 128u;
            if (!GEMM && soff == tap_bytes) {
                soff = 0;
                tap_w += dw;
                tap_off += strS;
                if (++ss == g.S) {
                    ss = 0;
                    tap_w = 0;
                    tap_h += dh;
                    tap_off += strR;
#pragma unroll
                    for (int i = 0; i < LX; ++i) iw[i] = ih0[i] + tap_h < static_cast<uint32_t>(g.IH) ? iw0[i] : kNowhere;
                }
            }
            if (lk == KT) {
                lk = ss = 0;
                soff = tap_h = tap_w = tap_off = 0;
                if (++lt < n_my) tile_setup(tile_id(lt));
            }
            return n;
        };
        // Waits until no more of this wave's loads are in flight than n, the loads of the youngest position (LX, with codes LX + LB,
        // none at the end) or of the youngest two (at least LX + LB).  A wave issues an instruction in four or five cycles at best
        // and a taken branch costs several: what this loop executes per slab bounds a lone tile, so the waits are nested, the
        // stricter ones behind the weaker.
        auto wait_loads = [&](int n) __attribute__((always_inline)) {
            asm volatile("" ::: "memory");
            __builtin_amdgcn_s_waitcnt(vmcnt_imm(LX + LB));
            if (n <= LX) {
                __builtin_amdgcn_s_waitcnt(vmcnt_imm(LX));
                if (n == 0) __builtin_amdgcn_s_waitcnt(vmcnt_imm(0));
            }
        };

        tile_setup(tile_id(0));
        issue();
        const int second = issue();
        int last = issue();                                 // loads of the youngest position
        wait_loads(last == 0 ? second : second + last);
        __builtin_amdgcn_s_barrier();                       // first slab landed
        for (uint32_t t = 0; t < n_my; ++t) {
            int k = KT;
            do {
                // hand-over of a slab: the next slab has landed (the youngest position may stay in flight)
                wait_loads(last);
                __builtin_amdgcn_s_barrier();
                asm volatile("" ::: "memory");
                last = issue();                             // refill the stage of the slab before
            } while (--k != 0);
            __builtin_amdgcn_s_barrier();                   // the one of the epilogue
        }
        return;
    }

    // =================================== compute wave ===================================
    const int wm = wave / WN, wn = wave % WN;
    const int lrow = lane & 31, lh = lane >> 5;

    // ---- per-column parameters, loaded one tile ahead (thread c < BN owns column c of the tile) --------
    float cp_alpha = 0.0f, cp_scale = 1.0f, cp_shift = 0.0f;
    auto colparam_load = [&](uint32_t t) __attribute__((always_inline)) {
        const uint32_t tm = fdiv_u(t, a.divTN);
        const int ncol = static_cast<int>((t - tm * a.tiles_n) * BN) + tid;
        cp_alpha = 0.0f;
        cp_scale = 1.0f;
        cp_shift = 0.0f;
        if (tid < BN && ncol < g.NC) {
            const int ag = (g.rows_per_group >= g.NC) ? 0 : ncol / g.rows_per_group;
            cp_alpha = ALPHA ? 2.0f : g.alpha[ag];
            if (g.scale) cp_scale = g.scale[ncol];
            if (g.shift) cp_shift = g.shift[ncol];
        }
    };

    f32x16 acc[MI][NI];
    auto acc_clear = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int mi = 0; mi < MI; ++mi)
#pragma unroll
            for (int ni = 0; ni < NI; ++ni)
#pragma unroll
                for (int e = 0; e < 16; ++e) acc[mi][ni][e] = 0.0f;
    };

    const uint32_t lds_base = static_cast<uint32_t>(reinterpret_cast<uintptr_t>(
        (__attribute__((address_space(3))) unsigned char*)smem));
    // step kk's fragments lie at a_lane ^ kk*16 of a stage
    const uint32_t a_lane = lds_base + (wm * TM + lrow) * 128 + (((lh * 4) ^ ((lrow >> 1) & 7)) * 16);
    // codes of slab q of a chunk lie at code_lane ^ q*16 of a chunk buffer
    const uint32_t code_lane = lds_base + STAGES * STAGE_BYTES + (wn * TN + lrow) * (CS * 16) + (lrow / (16 / CS) % CS) * 16 + lh * 8;
    uint32_t code_buf = 0, code_q = 0;          // buffer (bytes) and place in the chunk (bytes) of the next slab's codes
    int code_k = 0;                             // that slab's number in its tile
    auto code_addr = [&]() __attribute__((always_inline)) { return (code_lane ^ code_q) + code_buf; };
    auto code_advance = [&]() __attribute__((always_inline)) {
        code_q += 16;
        code_k = (code_k + 1 == KT) ? 0 : code_k + 1;
        if (code_k == 0 || code_q == CS * 16) {
            code_q = 0;
            code_buf = (code_buf == (kCodeBufs - 1) * CHUNK_BYTES) ? 0 : code_buf + CHUNK_BYTES;
        }
    };

    u32x2 breg[NI], bnext[NI];      // packed codes of the slab being multiplied / of the next slab
    constexpr int SETS = DEEP ? 4 : 2;
    u32x4 afrag[SETS][MI];  // activation fragments of step kk in set kk % SETS
    u32x4 bfrag[2][TERMS][NI];      // expanded codes of step kk in set kk & 1; ALPHA: times each term
    u32x4 al[2][TERMS];             // ALPHA: the terms of step kk in set kk & 1
    int c_cur = 0, c_next = 0;      // ALPHA: first reduction channel of the slab being multiplied / of the next
    const uint32_t term_base = static_cast<uint32_t>(reinterpret_cast<uintptr_t>(
        (__attribute__((address_space(3))) uint16_t*)terms)) + static_cast<uint32_t>(lh) * 64u;
    const uint32_t term_step = static_cast<uint32_t>(a.spt) * 128u;      // 64 * spt channels of two bytes
    auto after = [&](int c) __attribute__((always_inline)) { return c + 64 == a.spt * 64 ? 0 : c + 64; };

    uint32_t kmask[8];
    kmask[0] = sgpr_const<static_cast<int>(0xC000C000u >> 14)>();
    kmask[1] = sgpr_const<static_cast<int>(0xC000C000u >> 12)>();
    kmask[2] = sgpr_const<static_cast<int>(0xC000C000u >> 10)>();
    kmask[3] = sgpr_const<static_cast<int>(0xC000C000u >> 8)>();
    kmask[4] = sgpr_const<static_cast<int>(0xC000C000u >> 6)>();
    kmask[5] = sgpr_const<static_cast<int>(0xC000C000u >> 4)>();
    kmask[6] = sgpr_const<static_cast<int>(0xC000C000u >> 2)>();
    kmask[7] = sgpr_const<static_cast<int>(0xC000C000u)>();
    // Expansion of the codes of word e of a fragment, in two parts (mask, shift): an instruction that needs the result of the one
    // before it waits another four cycles, so the parts of two words are interleaved.
    uint32_t field[4 * NI];
    auto expand = [&](auto kk_tag, auto q_tag, auto part_tag, const u32x2* br, u32x4 (*out)[NI]) __attribute__((always_inline)) {
        constexpr int kk = decltype(kk_tag)::value, ni = decltype(q_tag)::value / 4, e = decltype(q_tag)::value % 4;
        constexpr int i = (kk & 1) * 4 + e;
        uint32_t& f = field[ni * 4 + e];
        if constexpr (decltype(part_tag)::value == 0) {
            f = ALPHA ? br[ni][kk >> 1] << (14 - 2 * i) : br[ni][kk >> 1] & kmask[i];
        } else if constexpr (ALPHA) {
            typedef short s16x2 __attribute__((ext_vector_type(2)));
            const uint32_t sign = f & 0x80008000u;
            const uint32_t on = __builtin_bit_cast(uint32_t, __builtin_bit_cast(s16x2, f << 1) >> 15);
#pragma unroll
            for (int k = 0; k < TERMS; ++k) out[k][ni][e] = (al[kk & 1][k][e] & on) ^ sign;
        } else {
            out[0][ni][e] = f << (14 - 2 * i);
        }
    };

    // One MFMA step (see gather_gemm_dma_kernel): fragment reads and code expansion of the next step are placed
    // between the MFMAs of this one, evenly and reads first; no vector-memory instruction in here.  The codes of the next slab are
    // requested in step CODES, behind the hand-over, and expanded in step 3.
    constexpr int CODES = DEEP ? 1 : 2;
    // What a slab leaves behind for the next (scalars, expanded codes, the codes themselves) is formed between the MFMAs of step 3
    // and held there: a compute wave that is alone on its SIMD issues one instruction in four cycles at best, and what the
    // compiler moves behind the last MFMA, to where it is used, runs while the matrix core stands still.
    uint32_t st_cur = 0, st_next = STAGE_BYTES;      // stage (bytes) of the slab being multiplied / of the next
    int left = KT;                                   // slabs of the tile that are still to be multiplied
    auto step = [&](auto kk_tag) __attribute__((always_inline)) {
        constexpr int KK = decltype(kk_tag)::value;
        constexpr int NM = MI * NI * TERMS;
        constexpr int SET = KK & 1, NSET = SET ^ 1;
        constexpr int KN = (KK + 1) & 3;
        // activation fragments requested here: without DEEP those of the next step; with it step 2's in step 0, 3's in 1, and
        // both of the next slab's first ones in step 2, so that none is in flight when the slab ends
        constexpr int RA = DEEP ? (KK + 2) & 3 : KN;
        constexpr int P_RA = DEEP ? (KK == 3 ? 0 : KK == 2 ? 2 * MI : MI) : MI;
        constexpr int P_RB = (KK == CODES) ? 1 : 0;
        constexpr int P_AL = ALPHA ? TERMS : 0;
        constexpr int P_R = P_RB + P_RA + P_AL;
        constexpr int P_D = 8 * NI;             // two parts of every word
        constexpr int P_S = (KK == CODES + 1 ? 1 : 0) + (KK == 3 ? 1 : 0);
        constexpr int P = P_R + P_D + P_S;
        const uint32_t a_stage = a_lane + ((DEEP ? KK >= 2 : KK == 3) ? st_next : st_cur);
        const int al_c = KK < 2 ? c_cur : c_next;
        auto read = [&](auto p_tag) __attribute__((always_inline)) {
            constexpr int pp = decltype(p_tag)::value;
            if constexpr (pp < P_RB) {
                lds_read64_n<NI, 32 * CS * 16>(bnext, code_addr());
            } else if constexpr (pp < P_RB + P_RA) {
                constexpr int r = pp - P_RB, kk = (RA + r / MI) & 3;
                lds_read128<(r % MI) * 32 * 128>(afrag[kk % SETS][r % MI], a_stage ^ (kk * 16));
            } else {
                // terms of the step after the next, whose set the expansion before this step has used up
                constexpr int term = pp - P_RB - P_RA;
                const uint32_t at = term_base + static_cast<uint32_t>(al_c) * 2u + term * term_step;
                lds_read128<((KK + 2) & 3) * 16>(al[SET][term], at);
            }
        };
        static_for<NM>([&](auto j_tag) __attribute__((always_inline)) {
            constexpr int jj = decltype(j_tag)::value;
            constexpr int mi = jj % (MI * NI) / NI, ni = jj % NI;      // ALPHA: all products with one term, then the next
            acc[mi][ni] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(
                __builtin_bit_cast(bf16x8, bfrag[SET][jj / (MI * NI)][ni]),
                __builtin_bit_cast(bf16x8, afrag[KK % SETS][mi]), acc[mi][ni], 0, 0, 0);
            __builtin_amdgcn_sched_barrier(0);
            static_for<P>([&](auto p_tag) __attribute__((always_inline)) {
                constexpr int pp = decltype(p_tag)::value;
                if constexpr (pp * NM / P == jj) {
                    if constexpr (pp < P_R) {
                        read(p_tag);
                    } else if constexpr (pp < P_R + P_D) {
                        constexpr int d = pp - P_R;             // word 2w mask, word 2w+1 mask, word 2w shift, word 2w+1 shift
                        expand(std::integral_constant<int, KN>{}, std::integral_constant<int, d / 4 * 2 + (d & 1)>{},
                               std::integral_constant<int, (d >> 1) & 1>{}, KK == 3 ? bnext : breg, bfrag[NSET]);
                    } else if constexpr (KK == CODES + 1 && pp == P_R + P_D) {
                        code_advance();
                        asm volatile("" : "+s"(code_q), "+s"(code_k), "+s"(code_buf));
                    } else {
                        --left;
                        st_cur = st_next;
                        st_next = (st_next == (STAGES - 1) * STAGE_BYTES) ? 0u : st_next + STAGE_BYTES;
                        if constexpr (ALPHA) {
                            // the slab after a tile's last one is the first of the next tile
                            c_cur = c_next;
                            c_next = (left == 1) ? 0 : after(c_cur);
                            if (left == 0) c_next = KT > 1 ? after(0) : 0;
                            asm volatile("" : "+s"(c_cur), "+s"(c_next));
                        }
                        asm volatile("" : "+s"(left), "+s"(st_cur), "+s"(st_next));
                    }
                }
            });
            __builtin_amdgcn_sched_barrier(0);
        });
        if constexpr (KK == 3) {
#pragma unroll
            for (int ni = 0; ni < NI; ++ni) breg[ni] = bnext[ni];
            lds_ready<NI>(breg);
        }
        lds_ready<TERMS * NI>(&bfrag[NSET][0][0]);
        if constexpr (!DEEP) {
            lds_wait<0>();
            lds_ready<MI>(afrag[NSET]);
            if constexpr (ALPHA) lds_ready<TERMS>(al[SET]);
        } else if constexpr (KK == 1) {
            lds_wait<MI + NI>();                // younger: step 3's fragments and the codes
            lds_ready<MI>(afrag[2 % SETS]);
        } else if constexpr (KK == 2) {
            lds_wait<2 * MI>();                 // younger: the next slab's first fragments
            lds_ready<MI>(afrag[3 % SETS]);
        } else if constexpr (KK == 3) {
            lds_wait<0>();
            lds_ready<MI>(afrag[0]);
            lds_ready<MI>(afrag[1]);
        }
        if constexpr (KK == 2) lds_ready<NI>(bnext);
        __builtin_amdgcn_sched_barrier(0);
    };

    // ---- epilogue of the tile the compute stream has just finished (as in conv_stream_kernel) ----
    const uint32_t ldyB = static_cast<uint32_t>(g.ldy) * 2u;
    TileStoreLane<EPI_CH> store_lane;
    store_lane.init(lane, ldyB);
    uint32_t ct = 0;
    auto epilogue = [&](uint32_t free_stage) __attribute__((always_inline)) {
        float* cmul = colbuf + (ct & 1u) * (2 * BN);
        float* cadd = cmul + BN;
        if (tid < BN) {
            cmul[tid] = 0.5f * cp_alpha * cp_scale;      // codes were +-2
            cadd[tid] = cp_shift;
        }
        // every wave has finished reading the stage of the last slab, and the column parameters are visible
        // (a bare s_barrier does not wait for this wave's LDS writes)
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
        const uint32_t t = tile_id(ct);
        const uint32_t tm = fdiv_u(t, a.divTN);
        const uint32_t m0 = tm * BM;
        const int n0 = static_cast<int>((t - tm * a.tiles_n) * BN);
        // the output descriptors are built here, per tile: scalar registers are scarce in the main loop
        uint32_t yb = a.y_bytes;
        asm volatile("" : "+s"(yb));
        const __amdgpu_buffer_rsrc_t ry = make_rsrc(g.Y, yb);
        const __amdgpu_buffer_rsrc_t rr = make_rsrc(g.residual ? g.residual : g.Y, yb);
        const uint32_t relu_floor = g.relu ? 0u : 0x80008000u;
        // one opaque offset: with known low bits the compiler would form every staging address as an OR of its own
        uint32_t staging = (EPI_OWN ? 0u : free_stage) + static_cast<uint32_t>(wave) * EPI_WAVE;
        asm volatile("" : "+s"(staging));
        store_tile_bf16<MI, NI, EPI_CH>(acc, cmul + wn * TN, cadd + wn * TN, (EPI_OWN ? epi_own : smem) + staging, store_lane, ry, rr,
                                        g.residual != nullptr, m0 + static_cast<uint32_t>(wm * TM), n0 + wn * TN,
                                        static_cast<uint32_t>(g.M), g.NC, ldyB, relu_floor, lane);
        acc_clear();
        ++ct;
        if (ct < n_my) colparam_load(tile_id(ct));
    };

    // ---- prologue: column parameters of the first tile; the load waves bring the first slab ----
    colparam_load(tile_id(0));
    acc_clear();
    if constexpr (ALPHA) {
        const int span = a.spt * 64;
        for (int c = tid; c < span; c += 64 * NWC) {
            const float v = c < g.IC ? g.alpha_in[c / g.alpha_in_rows] : 0.0f;
            uint16_t t[kAlphaTerms];
            alpha_terms(v, t);
#pragma unroll
            for (int k = 0; k < kAlphaTerms; ++k) terms[k * span + c] = t[k];
        }
        c_next = KT > 1 ? after(0) : 0;
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");      // visible after the barrier
    }
    __builtin_amdgcn_s_barrier();                           // first slab landed (the load waves waited for it)
    asm volatile("" ::: "memory");
    lds_read64_n<NI, 32 * CS * 16>(breg, code_addr());
    lds_read128_n<MI, 32 * 128>(afrag[0], a_lane);
    if constexpr (DEEP) lds_read128_n<MI, 32 * 128>(afrag[1], a_lane ^ 16);
    code_advance();
    if constexpr (ALPHA) {
#pragma unroll
        for (int k = 0; k < TERMS; ++k) {
            lds_read128<0>(al[0][k], term_base + k * term_step);
            lds_read128<16>(al[1][k], term_base + k * term_step);
        }
    }
    lds_wait<0>();
    lds_ready<NI>(breg);
    lds_ready<MI>(afrag[0]);
    if constexpr (DEEP) lds_ready<MI>(afrag[1]);
    if constexpr (ALPHA) {
        lds_ready<TERMS>(al[0]);
        lds_ready<TERMS>(al[1]);
    }
    static_for<4 * NI>([&](auto q_tag) __attribute__((always_inline)) {
        expand(std::integral_constant<int, 0>{}, q_tag, std::integral_constant<int, 0>{}, breg, bfrag[0]);
        expand(std::integral_constant<int, 0>{}, q_tag, std::integral_constant<int, 1>{}, breg, bfrag[0]);
    });

    // hand-over: the load waves have seen the next slab land; the stage of the previous slab is free
    auto hand_over = [&]() __attribute__((always_inline)) {
        asm volatile("" ::: "memory");
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
    };
    do {
        do {
            step(std::integral_constant<int, 0>{});
            if constexpr (DEEP) hand_over();
            step(std::integral_constant<int, 1>{});
            if constexpr (!DEEP) hand_over();
            step(std::integral_constant<int, 2>{});
            step(std::integral_constant<int, 3>{});
        } while (left != 0);
        left = KT;
        epilogue(st_cur == 0 ? (STAGES - 1) * STAGE_BYTES : st_cur - STAGE_BYTES);
    } while (ct < n_my);
}

// ---- host side ------------------------------------------------------------------------------------------

namespace {

int pc_num_cus() {
    static std::once_flag once;
    static int cus = 256;
    std::call_once(once, [] {
        int dev = 0;
        hipDeviceProp_t p;
        if (hipGetDevice(&dev) == hipSuccess && hipGetDeviceProperties(&p, dev) == hipSuccess && p.multiProcessorCount > 0)
            cus = p.multiProcessorCount;
    });
    return cus;
}

constexpr int kStreamAlphaMax = 1024;       // reduction channels of the table of terms: two workgroups per CU still fit

template <int BM, int BN, int WM, int WN, int STAGES, bool GEMM, int OCC, int CS, bool ALPHA = false>
int32_t launch_pc_kernel(const StreamPcArgs& a, hipStream_t st) {
    constexpr int EPI = WM * WN * 32 * ((BN / WN < 64 ? BN / WN : 64) * 2 + 16);        // output staging, where no stage holds it
    constexpr int SMEM = STAGES * BM * 128 + kCodeBufs * BN * CS * 16 + 4 * BN * 4 + (EPI > BM * 128 ? EPI : 0) +
                         (ALPHA ? kStreamAlphaMax * 2 * kAlphaTerms : 0);
    constexpr int THREADS = 64 * (WM * WN + kLoadWaves);
    static_assert(SMEM <= 160 * 1024 / OCC, "LDS budget");
    static_assert(THREADS <= 1024, "workgroup size");
    auto k = conv_stream_pc_kernel<BM, BN, WM, WN, STAGES, GEMM, OCC, CS, ALPHA>;
    static std::once_flag once;
    static int per_cu = 0;
    std::call_once(once, [&] {
        if (hipFuncSetAttribute(reinterpret_cast<const void*>(k), hipFuncAttributeMaxDynamicSharedMemorySize, SMEM) !=
            hipSuccess)
            return;
        int n = 0;
        if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, k, THREADS, SMEM) == hipSuccess && n > 0) per_cu = n;
    });
    if (per_cu <= 0) return TWN_ERR_HIP;
    int occ = per_cu;
    const int cap = env_int(Env::STREAM_OCC, 0);
    if (cap > 0 && cap < occ) occ = cap;
    int64_t grid = static_cast<int64_t>(pc_num_cus()) * occ;
    if (grid > a.tiles) grid = a.tiles;
    k<<<dim3(static_cast<unsigned>(grid)), dim3(THREADS), SMEM, st>>>(a);
    return launch_status();
}

template <int BM, int BN, int WM, int WN, int STAGES, int OCC, int CS, bool ALPHA = false>
int32_t launch_pc_tile(const GatherGemm& g, hipStream_t st) {
    const int64_t tiles_n = (g.NC + BN - 1) / BN;
    const int64_t tiles = ((g.M + BM - 1) / BM) * tiles_n;
    if (tiles <= 0 || tiles >= (1LL << 31)) return TWN_ERR_SHAPE;
    StreamPcArgs a;
    a.g = g;
    a.divOW = make_fastdiv_u(static_cast<uint32_t>(g.OW));
    a.divOH = make_fastdiv_u(static_cast<uint32_t>(g.OH));
    a.divTN = make_fastdiv_u(static_cast<uint32_t>(tiles_n));
    a.spt = (g.plain_gemm ? g.K : g.IC) / 64;
    const int64_t in_rows = g.plain_gemm ? g.M : (g.M / (static_cast<int64_t>(g.OH) * g.OW)) * g.IH * g.IW;
    a.x_bytes = static_cast<uint32_t>(((in_rows - 1) * g.xs + (g.plain_gemm ? g.K : g.IC)) * 2);
    a.w_bytes = static_cast<uint32_t>(static_cast<int64_t>(g.NC) * g.wpr * 4);
    a.y_bytes = static_cast<uint32_t>(((g.M - 1) * g.ldy + g.NC) * 2);
    a.tiles = static_cast<uint32_t>(tiles);
    a.tiles_n = static_cast<uint32_t>(tiles_n);
    a.KT = g.K / 64;
    return g.plain_gemm ? launch_pc_kernel<BM, BN, WM, WN, STAGES, true, OCC, CS, ALPHA>(a, st)
                        : launch_pc_kernel<BM, BN, WM, WN, STAGES, false, OCC, CS, ALPHA>(a, st);
}

}  // namespace

// Same tile ids and applicability (conv_stream_applicable) as launch_conv_stream; `np` load waves and `stages` (four of each).
int32_t launch_conv_stream_pc(const GatherGemm& g, int tile, int np, int stages, hipStream_t st) {
    if (np != kLoadWaves || stages != 4) return TWN_ERR_UNSUPPORTED;
    switch (tile) {
        case 14: return launch_pc_tile<64, 128, 1, 4, 4, 2, 4>(g, st);
        case 15: return launch_pc_tile<128, 128, 1, 4, 4, 2, 2>(g, st);
        case 16: return launch_pc_tile<128, 64, 2, 2, 4, 2, 4>(g, st);
        case 17: return launch_pc_tile<128, 256, 1, 4, 4, 1, 4>(g, st);
        case 18: return launch_pc_tile<256, 128, 2, 2, 4, 1, 4>(g, st);
        default: return TWN_ERR_UNSUPPORTED;
    }
}

// Undivided backward-data with several alphas (alpha_in).
bool conv_stream_alpha_applicable(const GatherGemm& g) {
    return g.IC <= kStreamAlphaMax && g.NC > 64 && env_int(Env::TILE, 0) == 0 && env_int(Env::STREAM, 1) != 0 &&
           !env_set(Env::STREAM_PC) && !env_set(Env::STREAM_KS) && !env_set(Env::STREAM_PC_STAGES) && !env_set(Env::STREAM_OCC) &&
           env_int(Env::BUFLOAD, 1) != 0 && conv_stream_applicable(g);
}
// The codes of 32 columns times three terms are 28 vector instructions a step: beside the six MFMAs of a 64-row wave tile they bound the
// kernel, beside the twelve of a 128-row one they do not.  128x128 tiles, one workgroup per CU, win where they leave the
// busiest CU no more rows than 64x128 tiles do and K is long enough to hide an epilogue that nothing overlaps (us, 64x128 -> 128x128:
// 3x3, 50176 pixels, 128 filters over 128 channels 45.9 -> 42.2; 12544, 256 over 256 40.6 -> 36.6; 9216, 512 over 200 69.6 -> 58.1;
// 18816, 128 over 128 20.4 -> 18.4; 1x1, 50176, 512 over 128 22.1 -> 21.1, but 256 over 128 13.4 -> 13.9; more rows for the busiest
// CU: 12544, 128 over 128 14.4 -> 18.8; 7840, 256 over 256 24.7 -> 31.5).
int32_t launch_conv_stream_alpha(const GatherGemm& g, hipStream_t st) {
    const int64_t cols = (g.NC + 127) / 128;
    const int64_t cus = pc_num_cus();
    auto busiest = [&](int bm) { return ((g.M + bm - 1) / bm * cols + cus - 1) / cus * bm; };
    if (g.K >= 512 && busiest(128) <= busiest(64)) return launch_pc_tile<128, 128, 1, 4, 4, 1, 4, true>(g, st);
    return launch_pc_tile<64, 128, 1, 4, 4, 2, 4, true>(g, st);
}

}  // namespace twn
