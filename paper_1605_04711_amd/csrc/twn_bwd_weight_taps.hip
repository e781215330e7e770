// Weight gradient of filters with several taps (Alg. 1 steps 9-10):
//   dW[o][c][r][s] = sum_{n,p,q} X[n, p*sh-ph+r*dh, q*sw-pw+s*dw, c] * dY[n,p,q,o]
// for channel counts that are multiples of 8, bf16 MFMA with float32 accumulation, gfx950.
//
// The general kernel treats every (tap, channel) as a column of a GEMM and fetches X once per tap.  Here a wave owns 64
// filters x 16 channels x 9 taps: the input patch of 32 output pixels (with halo) is fetched ONCE and all taps read
// their shifted windows of it, and the eight waves of a workgroup are two channel blocks times four slices of the
// PIXELS, whose sums are added through LDS: a workgroup dumps a tile of 64 x 32 x 9.
//   * A slab is 32 output pixels (a patch of pn images x ph rows x pw columns, powers of two).  The two waves of a slice
//     share its stages: dY as 32 x 64 channels, X as (input pixels of the patch) x 32 channels, by direct-to-LDS loads in
//     runs of 64 bytes (four lanes; runs of 32 bytes cost twice the address cycles), DEPTH stages.
//   * Fragments (8 consecutive pixels of one channel per lane) come from the transposing LDS read: 8 reads of dY and 18
//     of X for 36 MFMAs of 16x16x32, fetched across the slab boundary.  The eight pixels of a read pass must fall in
//     different banks: the two channel blocks of a pixel trade places in every second patch row, and the pitches of a
//     row and of an image are padded where that is not enough.
//   * Partial tiles are laid out as dW itself ([filter][channel][tap]): a tile is 64 contiguous runs, and the final sum
//     over workgroups is a plain element-wise pass.
// More than nine taps: groups of nine per workgroup (the patch covers the whole filter).
// Measured against the general kernel (us, with the final pass; stride 1, 3x3): 131072 pixels, 128 -> 128 channels 55 -> 48.6
// (793 TFLOP/s); 8192, 512 -> 512: 51 -> 43; 6272, 128 -> 128: 25.6 -> 17.4; 392, 512 -> 512: 26 -> 12.  A round of four
// slabs takes 0.83 us, 2000 clocks, against 1152 of MFMAs on a SIMD (512 -> 512, kernel alone: 8192 pixels, 32 rounds, 41.4 us;
// 4096 pixels, 16 rounds, 28.0), and about 15 us of a launch do not depend on the rounds; 8.5 where one range writes dW itself
// (2048 and 512 pixels: 16 and 4 rounds, 22.1 and 11.9 us).  Over the VGG-7 layers the matrix pipe works 0.30 of a launch's
// nominal clocks and LDS 0.17, 1 % of it lost to bank conflicts.  Starting half of the waves half a slab later, reading
// fragments four or five taps ahead, and stages private to each wave (no barrier) were all slower or equal.
#include <mutex>

#include "twn_bias_grad.h"
#include "twn_kernels.h"
#include "twn_lds_asm.h"

namespace twn {

namespace {

constexpr int kTapsPer = 9;                             // taps of one workgroup
constexpr int kWaves = 8;
constexpr int kWC = 2;                                  // channel blocks of 16 of a workgroup
constexpr int kSlices = kWaves / kWC;                   // slices of the pixels
constexpr int kPitch = kWC * 16 * kTapsPer + 4;         // floats per filter of the output tile in LDS (pad: see the store)
constexpr int kTileF = 64 * kPitch;
constexpr int kSmemMax = 160 * 1024;
constexpr int kDumpBytes = 36 * 1024;                   // one wave's accumulators, one float4 per lane each
constexpr int kTapsMax = 64;
constexpr int kSlotsMax = 128;                          // input pixels of a patch (four loads of a plane)

struct TapsArgs {
    const uint16_t* X;
    const uint16_t* dY;
    float* dW;
    float* partial;
    float beta;
    int32_t H, W, C, O, S, P, Q, N, RS;
    int32_t o_real;             // filters of dW: those behind them pad dY and are summed into nothing
    int32_t sh, sw, ph, pw, dh, dw;
    WgTapsPlan pl;
    FastDivU divSX, divSY, divRow, divImg, divS;
    FastDivU divTC, divG;       // workgroup -> (filter block, channel block, tap group)
    uint32_t dy_bytes, x_bytes;
    int32_t kx[5], ky[5], kn[5];    // what bit b of a slab's pixel index adds to its column, row, image
    int32_t aligned_out;        // dW (and the partial sums) 16-byte aligned
};

template <int OFFSET>
__device__ __forceinline__ void tr_read(u32x2& v, uint32_t addr) {
    asm volatile("ds_read_b64_tr_b16 %0, %1 offset:%2" : "=v"(v) : "v"(addr), "n"(OFFSET));
}

// column, row and image of pixel k of a slab
__device__ __forceinline__ void pixel_of(const TapsArgs& a, int k, int& dx, int& dy, int& dn) {
    dx = dy = dn = 0;
#pragma unroll
    for (int b = 0; b < 5; ++b) {
        const int bit = (k >> b) & 1;
        dx += bit * a.kx[b];
        dy += bit * a.ky[b];
        dn += bit * a.kn[b];
    }
}

template <int NB, int DEPTH>
__global__ __launch_bounds__(64 * kWaves, 2) void weight_grad_taps_kernel(const TapsArgs a) {
    constexpr int PER = 2 + NB;                         // loads of a slab per wave
    static_assert(DEPTH >= 3, "a slab is handed over while the previous one is multiplied");
    static_assert(PER == 5 || PER == 6, "the slots of the loads between two hand-overs");
    extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];
    const WgTapsPlan& pl = a.pl;
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int li = lane & 15, lg = lane >> 4;

    // workgroups are dealt round-robin to the 8 XCDs; an XCD gets a contiguous run of (pixel range, tile), tile fastest:
    // the tiles of one range read the same dY and X
    uint32_t t;
    {
        const uint32_t nb = gridDim.x, b = blockIdx.x, q = nb >> 3, r = nb & 7, xcd = b & 7, idx = b >> 3;
        t = (xcd < r) ? xcd * (q + 1) + idx : r * (q + 1) + (xcd - r) * q + idx;
    }
    const uint32_t tiles = static_cast<uint32_t>(pl.tiles);
    const uint32_t range = t / tiles;
    t -= range * tiles;
    const uint32_t tq = fdiv_u(t, a.divG);
    const int tap0 = static_cast<int>(t - tq * pl.groups) * kTapsPer;
    const uint32_t to = fdiv_u(tq, a.divTC);
    const int cb = wave % kWC, ks = wave / kWC;
    const int c_tile = static_cast<int>(tq - to * pl.tiles_c) * (16 * kWC);
    const int o0 = static_cast<int>(to) * 64;
    const int begin = static_cast<int>(range) * pl.per;
    const int end = (begin + pl.per < pl.slabs) ? begin + pl.per : pl.slabs;
    // slice ks multiplies the slabs begin + ks, begin + ks + 4, ...; every slice runs the same number of rounds (the
    // barriers are workgroup-wide), a round past the slice's last slab loads zeros
    const int rounds = (end - begin + kSlices - 1) / kSlices;

    const __amdgpu_buffer_rsrc_t rdy = make_rsrc(a.dY, a.dy_bytes), rx = make_rsrc(a.X, a.x_bytes);
    unsigned char* mine = smem + ks * (DEPTH * pl.stage_bytes);             // the slice's stages
    const uint32_t lds_mine = static_cast<uint32_t>(reinterpret_cast<uintptr_t>(
        (__attribute__((address_space(3))) unsigned char*)mine));

    // ---- loads of dY (half of them each): eight pixels per load, eight lanes each; pixel k keeps 16-byte chunk c at position
    // c ^ 2*swz(k), swz = (bit 1, bit 3) of k: the two groups of four pixels of a read pass then hit different banks ----
    uint32_t voffA[2];
    int ady[2], adx[2], adn[2];
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const int k = (cb * 2 + i) * 8 + (lane >> 3);
        const int o = o0 + (((lane & 7) ^ (2 * (((k >> 1) & 1) | ((k >> 2) & 2)))) * 8);
        pixel_of(a, k, adx[i], ady[i], adn[i]);
        voffA[i] = (o < a.O) ? (((static_cast<uint32_t>(adn[i]) * a.P + ady[i]) * a.Q + adx[i]) * a.O + o) * 2u : kBufOutside;
    }
    // ---- loads of X (half of the patch each): four lanes per input pixel, 16-byte chunk q of a pixel's 32 channels; the
    // two halves (channel blocks) trade places in odd patch rows ----
    uint32_t voffB[NB];
    int by[NB], bx[NB];
#pragma unroll
    for (int i = 0; i < NB; ++i) {
        const uint32_t ci = static_cast<uint32_t>((cb * NB + i) * 64 + lane);
        const uint32_t slot = ci >> 2, q = ci & 3;
        const uint32_t im = fdiv_u(slot, a.divImg);
        const uint32_t rem = slot - im * pl.img_slots;
        const uint32_t y = fdiv_u(rem, a.divRow);
        const uint32_t x = rem - y * pl.row_slots;
        const int c = c_tile + static_cast<int>(((q >> 1) ^ (y & 1)) * 16 + (q & 1) * 8);
        const bool ok = im < static_cast<uint32_t>(pl.pn) && y < static_cast<uint32_t>(pl.hh) && x < static_cast<uint32_t>(pl.ww) && c < a.C;
        by[i] = ok ? static_cast<int>(y) : (1 << 28);       // never passes the row test
        bx[i] = static_cast<int>(x);
        voffB[i] = (((im * a.H + y) * a.W + x) * a.C + c) * 2u;
    }

    // The loads of a slab one by one (issue_setup fixes the slab, everything in it wave-uniform)
    struct {
        unsigned char *sA, *sB;
        uint32_t offA, offB;
        int ih, iw, remN, remP, remQ;
    } ld;
    auto issue_setup = [&](int i, int stage) __attribute__((always_inline)) {
        ld.sA = mine + stage * pl.stage_bytes;
        ld.sB = ld.sA + 4096 + cb * (NB * 1024);
        const int slab = begin + ks + i * kSlices;
        const bool live = slab < end;
        const uint32_t su = static_cast<uint32_t>(slab);
        const uint32_t t1 = fdiv_u(su, a.divSX);
        const int q0 = static_cast<int>(su - t1 * pl.sx) * pl.pw;
        const uint32_t tn = fdiv_u(t1, a.divSY);
        const int p0 = static_cast<int>(t1 - tn * pl.sy) * pl.ph;
        const int n0 = static_cast<int>(tn) * pl.pn;
        ld.offA = ((static_cast<uint32_t>(n0) * a.P + p0) * a.Q + q0) * a.O * 2u;
        ld.ih = live ? p0 * a.sh - a.ph : -(1 << 29);
        ld.iw = q0 * a.sw - a.pw;
        // may stand for a negative offset: arithmetic is modulo 2^32, and only pixels inside the image use it
        ld.offB = ((static_cast<uint32_t>(n0) * a.H + static_cast<uint32_t>(ld.ih)) * a.W + static_cast<uint32_t>(ld.iw)) * a.C * 2u;
        ld.remN = live ? a.N - n0 : 0;
        ld.remP = a.P - p0;
        ld.remQ = a.Q - q0;
    };
    auto issue_load = [&](auto j_tag) __attribute__((always_inline)) {
        constexpr int j = decltype(j_tag)::value;
        if constexpr (j < 2) {
            const bool ok = (adn[j] < ld.remN) & (ady[j] < ld.remP) & (adx[j] < ld.remQ);
            buf_dma16(rdy, ok ? voffA[j] + ld.offA : kBufOutside, 0u, ld.sA + (cb * 2 + j) * 1024);
        } else {
            constexpr int b = j - 2;
            const bool ok = (static_cast<unsigned>(ld.ih + by[b]) < static_cast<unsigned>(a.H)) &
                            (static_cast<unsigned>(ld.iw + bx[b]) < static_cast<unsigned>(a.W));
            const uint32_t off = ok ? voffB[b] + ld.offB : kBufOutside;
            buf_dma16(rx, off, 0u, ld.sB + b * 1024);
        }
    };

    // ---- fragment addresses: lane li of a group of 16 supplies pixel li >> 2, channels 4*(li & 3) .. + 3 of the four
    // pixels 8*lg + 4*hv + 0..3, and receives its own channel li of all four ----
    uint32_t adrA[4], adrB[2];
    {
        const int k = lg * 8 + (li >> 2);                   // hv = 1: + 4, same swizzle
        const int swz = ((k >> 1) & 1) | ((k >> 2) & 2);
#pragma unroll
        for (int ob = 0; ob < 4; ++ob) adrA[ob] = lds_mine + k * 128 + ((ob ^ swz) * 32) + (li & 3) * 8;
#pragma unroll
        for (int hv = 0; hv < 2; ++hv) {
            int dx, dy, dn;
            pixel_of(a, k + 4 * hv, dx, dy, dn);
            adrB[hv] = lds_mine + 4096 + (dn * pl.img_slots + dy * pl.row_slots + dx) * 64 + ((cb ^ (dy & 1)) * 32) + (li & 3) * 8;
        }
    }
    uint32_t tapoff[kTapsPer], tapxor[kTapsPer];            // wave-uniform; a tap in an odd row finds the halves swapped
#pragma unroll
    for (int i = 0; i < kTapsPer; ++i) {
        const int tap = (tap0 + i < a.RS) ? tap0 + i : tap0;        // a tap past the last one: computed, never written
        const int r = static_cast<int>(fdiv_u(static_cast<uint32_t>(tap), a.divS)), s = tap - r * a.S;
        tapoff[i] = static_cast<uint32_t>((r * a.dh * pl.row_slots + s * a.dw) * 64);
        tapxor[i] = static_cast<uint32_t>((r * a.dh) & 1) * 32u;
    }

    f32x4 acc[4][kTapsPer];
#pragma unroll
    for (int ob = 0; ob < 4; ++ob)
#pragma unroll
        for (int i = 0; i < kTapsPer; ++i) acc[ob][i] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};

    // ---- software pipeline: slab `it` is multiplied tap by tap, the X fragments of tap i read AHEAD taps before.  Before
    // tap 6 the next slab is handed over (own loads waited for, barrier: then the partner's have landed too and the stage
    // of the previous slab is free to be refilled), so that the reads of taps 6 to 8 fetch its first fragments.  LDS reads
    // complete in issue order, so s_waitcnt lgkmcnt(number of younger reads) is exact. ----
    constexpr int AHEAD = 3, RING = AHEAD + 1;
    u32x2 fa[2][4][2], fb[RING][2];
    static_assert(kTapsPer == 9 && RING == 4, "the ring advances by one entry per slab");
    auto read_b = [&](auto e_tag, int tap, uint32_t stage_off) __attribute__((always_inline)) {
        constexpr int e = decltype(e_tag)::value;
        const uint32_t off = stage_off + tapoff[tap];
#pragma unroll
        for (int hv = 0; hv < 2; ++hv) tr_read<0>(fb[e][hv], (adrB[hv] ^ tapxor[tap]) + off);
    };
    // (the last loads of slab DEPTH - 2 are issued by the first round)
#pragma unroll
    for (int d = 0; d < DEPTH - 1; ++d) {
        issue_setup(d, d);
        if (d < DEPTH - 2) static_for<PER>(issue_load);
        else static_for<3>(issue_load);
    }
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"((DEPTH - 3) * PER + 3) : "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
#pragma unroll
    for (int ob = 0; ob < 4; ++ob) {
        tr_read<0>(fa[0][ob][0], adrA[ob]);
        tr_read<512>(fa[0][ob][1], adrA[ob]);
    }
    static_for<AHEAD>([&](auto i_tag) __attribute__((always_inline)) { read_b(i_tag, decltype(i_tag)::value, 0u); });

    int stage = 0, fill = DEPTH - 1;
    // one slab; PHASE = it % 4 selects the ring position, PHASE % 2 the register set of the dY fragments
    auto slab = [&](int it, auto phase_tag) __attribute__((always_inline)) {
        constexpr int PHASE = decltype(phase_tag)::value, CUR = PHASE & 1;
        const int next = (stage + 1 == DEPTH) ? 0 : stage + 1;
        const uint32_t so = static_cast<uint32_t>(stage * pl.stage_bytes), sn = static_cast<uint32_t>(next * pl.stage_bytes);
        static_for<kTapsPer>([&](auto i_tag) __attribute__((always_inline)) {
            constexpr int i = decltype(i_tag)::value;
            constexpr int E = (PHASE + i) % RING, ENEW = (PHASE + i + AHEAD) % RING;    // 9 taps advance the ring by 9 = 1 (mod 4)
            if constexpr (i == kTapsPer - AHEAD) {
                asm volatile("s_waitcnt vmcnt(%0)" ::"n"((DEPTH - 3) * PER) : "memory");
                __builtin_amdgcn_s_barrier();
                asm volatile("" ::: "memory");
                issue_setup(it + DEPTH - 1, fill);
            }
            if constexpr (i >= kTapsPer - AHEAD) {
                // the next slab's dY fragments: 3 + 3 + 2 reads
                constexpr int f0 = (i - (kTapsPer - AHEAD)) * 3, f1 = (f0 + 3 < 8) ? f0 + 3 : 8;
                static_for<f1 - f0>([&](auto d_tag) __attribute__((always_inline)) {
                    constexpr int f = f0 + decltype(d_tag)::value;
                    tr_read<(f & 1) * 512>(fa[CUR ^ 1][f >> 1][f & 1], adrA[f >> 1] + sn);
                });
                read_b(std::integral_constant<int, ENEW>{}, i + AHEAD - kTapsPer, sn);
            } else {
                read_b(std::integral_constant<int, ENEW>{}, i + AHEAD, so);
            }
            // reads issued after those this tap needs
            constexpr int younger = (i == 0) ? 4 : (i < 6) ? 6 : (i == 6) ? 9 : (i == 7) ? 12 : 14;
            lds_wait<younger>();
            if constexpr (i == 0) {
#pragma unroll
                for (int ob = 0; ob < 4; ++ob) lds_ready<2>(fa[CUR][ob]);
            }
            lds_ready<2>(fb[E]);
            const u32x4 bv = {fb[E][0][0], fb[E][0][1], fb[E][1][0], fb[E][1][1]};
#pragma unroll
            for (int ob = 0; ob < 4; ++ob) {
                const u32x4 av = {fa[CUR][ob][0][0], fa[CUR][ob][0][1], fa[CUR][ob][1][0], fa[CUR][ob][1][1]};
                acc[ob][i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, av), __builtin_bit_cast(bf16x8, bv),
                                                                     acc[ob][i], 0, 0, 0);
            }
            // the loads of slab it + DEPTH - 1, one behind a tap's MFMAs: taps 6, 7, 8 of this round, 0, 1, (2) of the next
            __builtin_amdgcn_sched_barrier(0);
            constexpr int j = (i >= kTapsPer - 3) ? i - (kTapsPer - 3) : i + 3;
            if constexpr (j < PER) issue_load(std::integral_constant<int, j>{});
            __builtin_amdgcn_sched_barrier(0);
        });
        stage = next;
        fill = (fill + 1 == DEPTH) ? 0 : fill + 1;
    };
    for (int it = 0; it < rounds; it += 4) {
        slab(it, std::integral_constant<int, 0>{});
        if (it + 1 < rounds) slab(it + 1, std::integral_constant<int, 1>{});
        if (it + 2 < rounds) slab(it + 2, std::integral_constant<int, 2>{});
        if (it + 3 < rounds) slab(it + 3, std::integral_constant<int, 3>{});
    }
    // the fragments fetched ahead for the slab after the last one are never used: let them and the trailing loads land
    // before registers and LDS are reused
    lds_wait<0>();
#pragma unroll
    for (int ob = 0; ob < 4; ++ob) {
        lds_ready<2>(fa[0][ob]);
        lds_ready<2>(fa[1][ob]);
    }
#pragma unroll
    for (int e = 0; e < RING; ++e) lds_ready<2>(fb[e]);
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");

    // ---- the slices' sums: 2, 3 onto 0, 1, and those two through output tiles (a fixed order) ----
    auto dump = [&](int slot) __attribute__((always_inline)) {
        f32x4* dst = reinterpret_cast<f32x4*>(smem + slot * kDumpBytes) + lane;
#pragma unroll
        for (int ob = 0; ob < 4; ++ob)
#pragma unroll
            for (int i = 0; i < kTapsPer; ++i) dst[(ob * kTapsPer + i) * 64] = acc[ob][i];
    };
    auto add = [&](int slot) __attribute__((always_inline)) {
        const f32x4* src = reinterpret_cast<const f32x4*>(smem + slot * kDumpBytes) + lane;
#pragma unroll
        for (int ob = 0; ob < 4; ++ob)
#pragma unroll
            for (int i = 0; i < kTapsPer; ++i) acc[ob][i] += src[(ob * kTapsPer + i) * 64];
    };
    __syncthreads();                    // every wave is done with its stages
    if (ks >= 2) dump((ks - 2) * kWC + cb);
    __syncthreads();
    if (ks < 2) add(ks * kWC + cb);
    __syncthreads();
    const float* tile = reinterpret_cast<const float*>(smem);
    if (ks < 2) {
        // [filter][channel*9 + tap], a pitch of 4 modulo 16: the 64 lanes of a store fall in 64 different banks
        float* mine_t = reinterpret_cast<float*>(smem) + ks * kTileF;
#pragma unroll
        for (int ob = 0; ob < 4; ++ob)
#pragma unroll
            for (int i = 0; i < kTapsPer; ++i)
#pragma unroll
                for (int e = 0; e < 4; ++e) mine_t[(ob * 16 + lg * 4 + e) * kPitch + (cb * 16 + li) * kTapsPer + i] = acc[ob][i][e];
    }
    __syncthreads();

    // ---- [filter][channel][tap] runs of the tile -> dW (one range) or this range's partial sums ----
    const int taps = (a.RS - tap0 < kTapsPer) ? a.RS - tap0 : kTapsPer;
    const int64_t row = static_cast<int64_t>(a.C) * a.RS;
    float* out = (pl.splits == 1) ? a.dW : a.partial + static_cast<int64_t>(range) * a.O * row;
    const bool accumulate = pl.splits == 1 && a.beta != 0.0f;
    if (a.RS == kTapsPer && !accumulate && a.aligned_out && o0 + 64 <= a.o_real && c_tile + 16 * kWC <= a.C) {
        // whole tile, nine taps: a filter's run is contiguous and 16-byte aligned
        constexpr int Q = 36 * kWC, N = 64 * Q / (64 * kWaves);      // float4 per filter; per thread (rounded down)
        auto copy = [&](int i) __attribute__((always_inline)) {
            const int o = i / Q, j = (i - o * Q) * 4;
            const f32x4 v = *reinterpret_cast<const f32x4*>(tile + o * kPitch + j) +
                            *reinterpret_cast<const f32x4*>(tile + kTileF + o * kPitch + j);
            store16_through(out + (o0 + o) * row + static_cast<int64_t>(c_tile) * kTapsPer + j, __builtin_bit_cast(u32x4, v));
        };
#pragma unroll
        for (int n = 0; n < N; ++n) copy(n * 64 * kWaves + tid);
        if (N * 64 * kWaves < 64 * Q && N * 64 * kWaves + tid < 64 * Q) copy(N * 64 * kWaves + tid);
        return;
    }
    for (int i = tid; i < 64 * 144 * kWC; i += 64 * kWaves) {
        const int o = i / (144 * kWC), j = i - o * (144 * kWC);
        const int c = j / kTapsPer, tap = j - c * kTapsPer;
        if (o0 + o >= a.o_real || c_tile + c >= a.C || tap >= taps) continue;
        const float v = tile[o * kPitch + j] + tile[kTileF + o * kPitch + j];
        float* dst = out + (o0 + o) * row + static_cast<int64_t>(c_tile + c) * a.RS + tap0 + tap;
        *dst = accumulate ? a.beta * *dst + v : v;
    }
}

// dW = beta*dW + sum over ranges of the first n elements of partial[range], `pitch` elements apart, element by element.  PARTS threads share the ranges of four elements (every
// PARTS-th each, then their sums in order): with one, a bank of 64 x 64 filters is 36 workgroups that read 224 ranges one
// after the other (8.8 us; with eight 5.3).
template <int PARTS, bool BIAS>
__global__ __launch_bounds__(256) void weight_grad_sum_kernel(const float* __restrict__ partial, int splits, int64_t pitch, int64_t n,
                                                              float beta, float* __restrict__ dW, const BiasGrad bias) {
    constexpr int COLS = 256 / PARTS;
    __shared__ f32x4 red[BIAS ? kBiasLds / 4 : PARTS > 1 ? 256 : 1];
    const int block = final_pass_block<256, BIAS>(bias, reinterpret_cast<float*>(red));
    if (block < 0) return;
    const int col = threadIdx.x % COLS, part = threadIdx.x / COLS;
    const int64_t id = (static_cast<int64_t>(block) * COLS + col) * 4;
    f32x4 s = {0.0f, 0.0f, 0.0f, 0.0f};
    if (id < n) {
#pragma unroll 8
        for (int sp = part; sp < splits; sp += PARTS) s += *reinterpret_cast<const f32x4*>(partial + sp * pitch + id);
    }
    if constexpr (PARTS > 1) {
        red[threadIdx.x] = s;
        __syncthreads();
        if (part != 0) return;
#pragma unroll
        for (int p = 1; p < PARTS; ++p) s += red[p * COLS + col];
    }
    if (id >= n) return;
    if (beta == 0.0f && (reinterpret_cast<uintptr_t>(dW) & 15) == 0) {
        *reinterpret_cast<f32x4*>(dW + id) = s;
        return;
    }
#pragma unroll
    for (int e = 0; e < 4; ++e) dW[id + e] = (beta != 0.0f) ? beta * dW[id + e] + s[e] : s[e];
}

// The five bits of a slab's pixel index in terms of its column, row and image.  Bits 0 and 1 are the four pixels a group of
// lanes reads, bit 3 the two groups of a read pass, bits 2 and 4 separate passes: four neighbours of a row in the first,
// neighbouring rows (whose halves are swapped) in the second, where the patch has them.
struct PixelBits {
    int32_t kx[5], ky[5], kn[5];
};
PixelBits pixel_bits(const WgTapsPlan& p) {
    PixelBits m{};
    int x = 1, y = 1, n = 1;
    auto take_x = [&](int b) { if (x < p.pw) { m.kx[b] = x; x *= 2; return true; } return false; };
    auto take_y = [&](int b) { if (y < p.ph) { m.ky[b] = y; y *= 2; return true; } return false; };
    auto take_n = [&](int b) { if (n < p.pn) { m.kn[b] = n; n *= 2; return true; } return false; };
    for (int b : {0, 1})
        if (!take_x(b) && !take_y(b)) take_n(b);
    for (int b : {3, 2, 4})
        if (!take_y(b) && !take_x(b)) take_n(b);
    return m;
}

// Bank passes of an X fragment read relative to a conflict-free one: a pass serves eight pixels of 32 bytes.
int b_read_passes(const WgTapsPlan& p, const PixelBits& m) {
    int worst = 1;
    for (int hv = 0; hv < 2; ++hv)
        for (int pass = 0; pass < 2; ++pass) {
            int used[8] = {0};
            for (int i = 0; i < 8; ++i) {
                const int k = pass * 16 + (i >> 2) * 8 + hv * 4 + (i & 3);
                int dx = 0, dy = 0, dn = 0;
                for (int b = 0; b < 5; ++b) {
                    const int bit = (k >> b) & 1;
                    dx += bit * m.kx[b]; dy += bit * m.ky[b]; dn += bit * m.kn[b];
                }
                const int n = ++used[((dn * p.img_slots + dy * p.row_slots + dx) & 3) * 2 + (dy & 1)];
                if (n > worst) worst = n;
            }
        }
    return worst;
}

}  // namespace

// A pure function of the shapes (the workspace query and the launch agree).  Costs are clocks of a CU per slab and wave: 144
// for the MFMAs, 16 per load, 4 per transposing read and bank pass.
static WgTapsPlan make_taps_plan(const WgShape& w) {
    WgTapsPlan best{};
    best.use = 0;
    if (w.sh != 1 || w.sw != 1 || w.R * w.S < 4 || w.R * w.S > kTapsMax || w.C % 8 != 0 || w.O % 8 != 0) return best;
    // an override that shapes the general kernel means multi-tap filters too
    if (env_int(Env::WG_TAPS, 1) == 0 || env_int(Env::BUFLOAD, 1) == 0 || env_set(Env::WG_BLOCKS) || env_set(Env::WG_KS) ||
        env_set(Env::WG_ROWS_SPLITS) || env_set(Env::WG_XCD))
        return best;
    // small filter banks over few pixels: the fixed part (first loads, the sum over slices, the final pass: 12 us) is more than
    // the general kernel's whole time (25088 pixels, 64 x 64 channels: 18.2 against 16.1 us; 6272 pixels, 128 x 128: 17.4
    // against 25.6; 200704 pixels, 64 x 64: 33.5 against 39.4)
    const int64_t pixels = static_cast<int64_t>(w.N) * w.P * w.Q;
    if (static_cast<int64_t>(w.O) * w.C < 8192 && pixels < 65536) return best;
    const int64_t dyb = static_cast<int64_t>(w.N) * w.P * w.Q * w.O * 2, xb = static_cast<int64_t>(w.N) * w.H * w.W * w.C * 2;
    if (dyb >= (1LL << 31) || xb >= (1LL << 31) || static_cast<int64_t>(w.O) * w.C * w.R * w.S >= (1LL << 28)) return best;
    double best_cost = 0;
    for (int lw = 5; lw >= 0; --lw)
        for (int lh = 5 - lw; lh >= 0; --lh) {
            WgTapsPlan p{};
            p.pw = 1 << lw; p.ph = 1 << lh; p.pn = 32 >> (lw + lh);
            p.sx = (w.Q + p.pw - 1) / p.pw; p.sy = (w.P + p.ph - 1) / p.ph; p.sn = (w.N + p.pn - 1) / p.pn;
            const int64_t slabs = static_cast<int64_t>(p.sx) * p.sy * p.sn;
            if (slabs >= (1 << 30)) continue;
            p.slabs = static_cast<int32_t>(slabs);
            const int64_t hh = p.ph - 1 + static_cast<int64_t>(w.R - 1) * w.dh + 1;
            const int64_t ww = p.pw - 1 + static_cast<int64_t>(w.S - 1) * w.dw + 1;
            if (hh * ww * p.pn > kSlotsMax) continue;
            p.hh = static_cast<int32_t>(hh); p.ww = static_cast<int32_t>(ww);
            // pitches: the smallest padding without bank conflicts
            const PixelBits bits = pixel_bits(p);
            int passes = 100;
            for (int row = p.ww; row < p.ww + 4 && passes > 1; ++row)
                for (int img = p.hh * row; img < p.hh * row + (p.pn > 1 ? 8 : 1) && passes > 1; ++img) {
                    WgTapsPlan c = p;
                    c.row_slots = row; c.img_slots = img;
                    c.slots = (p.pn - 1) * img + p.hh * row;
                    if (c.slots > kSlotsMax) continue;
                    const int n = b_read_passes(c, bits);
                    if (n < passes) {
                        passes = n;
                        p.row_slots = row; p.img_slots = img; p.slots = c.slots;
                    }
                }
            if (passes == 100) continue;
            p.nb = p.slots <= 96 ? 3 : 4;
            const double lds = 32.0 + 72.0 * passes + 8.0 * (2 + p.nb), dma = 32.0 + 0.5 * p.slots * 2;
            double per = lds > dma ? lds : dma;
            if (per < 144.0) per = 144.0;
            const double cost = per * static_cast<double>(p.slabs);
            if (!best.use || cost < best_cost) {
                best = p;
                best.use = 1;
                best_cost = cost;
            }
        }
    if (!best.use) return best;
    best.stage_bytes = 4096 + best.nb * 2048;
    best.depth = best.nb == 3 ? 4 : 3;          // what 160 KB of LDS hold
    static_assert(kSlices * 4 * (4096 + 3 * 2048) <= kSmemMax && kSlices * 3 * (4096 + 4 * 2048) <= kSmemMax, "stages fit");
    best.tiles_o = (w.O + 63) / 64;
    best.tiles_c = (w.C + 16 * kWC - 1) / (16 * kWC);
    best.groups = (w.R * w.S + kTapsPer - 1) / kTapsPer;
    const int64_t tiles = static_cast<int64_t>(best.tiles_o) * best.tiles_c * best.groups;
    if (tiles >= (1 << 24)) { best.use = 0; return best; }
    best.tiles = static_cast<int32_t>(tiles);
    // pixel ranges: rounds of 256 workgroups (one per CU), each with a fixed part (launch, first loads, the sum over its
    // waves: about 10 us worth of slabs' clocks is 12 slab times of eight waves), plus the traffic of the partial sums
    const double slab_us = best_cost / best.slabs * kWaves / 2400.0;        // one slab for each slice
    const double tensor_mb = static_cast<double>(w.O) * w.C * w.R * w.S * 4e-6;
    double best_us = 1e30;
    for (int s = 1; s <= 256; s = (s < 16) ? s + 1 : s + s / 8) {
        if (s > best.slabs) break;
        const int per = (best.slabs + s - 1) / s;
        const int splits = (best.slabs + per - 1) / per;
        const double rounds = static_cast<double>((tiles * splits + 255) / 256);
        const double us = rounds * (4.0 + slab_us * 1.5 * ((per + kSlices - 1) / kSlices)) + (splits > 1 ? 3.0 + 2.0 * splits * tensor_mb / 5.0 : 0.0);
        if (us < best_us) {
            best_us = us;
            best.per = per;
            best.splits = splits;
        }
    }
    return best;
}

WgTapsPlan plan_weight_grad_taps(const WgShape& w) {
    // a plan takes microseconds to find and a training loop asks for the same few again and again: the last ones are
    // kept per thread, by shape
    struct Kept {
        WgShape shape;
        uint32_t generation;
        WgTapsPlan plan;
    };
    constexpr int kKept = 64;
    static thread_local Kept kept[kKept] = {};
    uint32_t h = 0;
    const int32_t* v = reinterpret_cast<const int32_t*>(&w);
    for (size_t i = 0; i < sizeof(w) / sizeof(int32_t); ++i) h = h * 31u + static_cast<uint32_t>(v[i]);
    Kept& k = kept[(h ^ (h >> 16)) % kKept];
    const uint32_t gen = g_env_generation.load(std::memory_order_relaxed);
    if (k.generation != gen || __builtin_memcmp(&k.shape, &w, sizeof(w)) != 0) {
        k.plan = make_taps_plan(w);
        k.shape = w;
        k.generation = gen;
    }
    return k.plan;
}

template <int NB, int DEPTH>
static int32_t launch_taps(const TapsArgs& a, hipStream_t st) {
    auto k = weight_grad_taps_kernel<NB, DEPTH>;
    static std::once_flag once;
    static bool allowed = false;
    std::call_once(once, [&] {
        allowed = hipFuncSetAttribute(reinterpret_cast<const void*>(k), hipFuncAttributeMaxDynamicSharedMemorySize, kSmemMax) ==
                  hipSuccess;
    });
    if (!allowed) return TWN_ERR_HIP;
    int smem = kSlices * DEPTH * a.pl.stage_bytes;
    if (smem < 2 * kTileF * 4) smem = 2 * kTileF * 4;
    if (smem > kSmemMax) return TWN_ERR_UNSUPPORTED;
    static_assert(2 * kTileF * 4 >= 2 * kWC * kDumpBytes && 2 * kTileF * 4 <= kSmemMax, "the sums over the slices reuse the stages");
    k<<<dim3(static_cast<unsigned>(a.pl.tiles) * a.pl.splits), dim3(64 * kWaves), smem, st>>>(a);
    return launch_status();
}

int32_t launch_weight_grad_taps(const WeightGrad& w, const WgTapsPlan& pl, bool* bias_done, hipStream_t st) {
    *bias_done = false;
    TapsArgs a;
    a.X = w.X; a.dY = w.dY; a.dW = w.dW; a.partial = w.partial; a.beta = w.beta;
    a.H = w.H; a.W = w.W; a.C = w.C; a.O = w.O; a.S = w.S; a.P = w.P; a.Q = w.Q; a.N = w.N; a.RS = w.R * w.S; a.o_real = w.o_real;
    a.sh = w.sh; a.sw = w.sw; a.ph = w.ph; a.pw = w.pw; a.dh = w.dh; a.dw = w.dw;
    a.pl = pl;
    a.divSX = make_fastdiv_u(pl.sx); a.divSY = make_fastdiv_u(pl.sy);
    a.divRow = make_fastdiv_u(pl.row_slots); a.divImg = make_fastdiv_u(pl.img_slots);
    a.divS = make_fastdiv_u(w.S);
    a.divTC = make_fastdiv_u(pl.tiles_c); a.divG = make_fastdiv_u(pl.groups);
    a.dy_bytes = static_cast<uint32_t>(static_cast<int64_t>(w.N) * w.P * w.Q * w.O * 2);
    a.x_bytes = static_cast<uint32_t>(static_cast<int64_t>(w.N) * w.H * w.W * w.C * 2);
    const PixelBits bits = pixel_bits(pl);
    for (int b = 0; b < 5; ++b) {
        a.kx[b] = bits.kx[b];
        a.ky[b] = bits.ky[b];
        a.kn[b] = bits.kn[b];
    }
    a.aligned_out = aligned(w.dW, 16) && aligned(w.partial, 16);
    int32_t rc;
    if (pl.nb == 3) rc = launch_taps<3, 4>(a, st);
    else if (pl.nb == 4) rc = launch_taps<4, 3>(a, st);
    else return TWN_ERR_UNSUPPORTED;
    if (rc != TWN_OK || pl.splits == 1) return rc;
    const int64_t row = static_cast<int64_t>(w.C) * a.RS, n = row * w.o_real, pitch = row * w.O;       // multiples of 8
    const BiasGrad bias = bias_in_final_pass(w);
    *bias_done = bias.blocks > 0;
    if (pl.splits >= 32 && n / 4 < 256 * 256)
        launch_final_pass(weight_grad_sum_kernel<8, false>, weight_grad_sum_kernel<8, true>, (n / 4 + 31) / 32, 256, bias, st, w.partial, pl.splits,
                          pitch, n, w.beta, w.dW);
    else
        launch_final_pass(weight_grad_sum_kernel<1, false>, weight_grad_sum_kernel<1, true>, (n / 4 + 255) / 256, 256, bias, st, w.partial, pl.splits,
                          pitch, n, w.beta, w.dW);
    return launch_status();
}

}  // namespace twn
