// Weight gradient of a three-channel first layer (Alg. 1 steps 9-10), filters up to 7x7, strides up to 2, dilation 1, gfx950:
//   dW[o][c][r][s] = sum_{n,p,q} X[n, p*sh-ph+r, q*sw-pw+s, c] * dY[n,p,q,o]
// The general kernel gathers X once per tap from a zero-bordered four-channel copy that a launch of its own makes: 16 KB of
// gathered activations per 32 pixels against 4 KB of dY.  Here a workgroup walks 16x16 tiles of output pixels:
//   * the input patch of a tile (with halo) is read once, two pixels (12 bytes) per lane, and widened to four channels on its
//     way into LDS; dY comes by direct-to-LDS loads, three tiles ahead (X: two, in registers);
//   * a column block of the product is four taps x four channels of one filter row, and the transposing LDS read takes the
//     address of every (pixel, tap) from a lane of its own: all taps read shifted windows of the one patch, and eight
//     consecutive pixels of a column arrive in a register pair with no further step;
//   * a wave owns 64 filters x all columns (at most 14 accumulator tiles of 32x32, one wave per SIMD) for four of the sixteen
//     pixel rows, reading the fragments of a row while the row before is multiplied (4 + 2 NT reads for 2 NT MFMAs); the
//     waves are summed through LDS and the workgroup writes one partial tile in the layout of the general kernel's
//     first-layer mode.
// ResNet-18 stem, batch 64 (802816 pixels, 64 filters 7x7/2): copy, product and final pass 83 -> 52 us; VGG-7, batch 128
// (131072 pixels, 128 filters 3x3): 30 -> 21.  dY and X at the rate of a large copy: 25 and 7.
#include <mutex>

#include "twn_kernels.h"
#include "twn_lds_asm.h"
#include "twn_mfma.h"

namespace twn {

namespace {

constexpr int kTile = 16;                               // output rows and columns of a tile
constexpr int kDyBytes = kTile * kTile * 128;           // 256 pixels x 64 filters
constexpr int kDyStages = 4;
constexpr int kXLoads = 3;                              // pixel pairs per lane and patch
constexpr int kDyLoads = kDyBytes / 4096;               // direct loads per wave and tile

struct FirstGradArgs {
    const uint16_t* X;
    const uint16_t* dY;
    float* partial;             // [splits][O][J], J = R * G * 16
    int32_t N, H, W, O, P, Q, sh, sw, ph, pw, xoff;
    int32_t G, units, J;        // column blocks of four taps per filter row; R * G; 16 * units
    int32_t PW, pairs, npairs;  // patch columns (even), pairs per patch row, pairs of a patch
    int32_t patch_bytes;
    int32_t tiles, per;         // per workgroup
    FastDivU divTX, divTY, divPairs;
    uint32_t x_bytes, dy_bytes;
};

__device__ __forceinline__ u32x2 tr_read(uint32_t addr) {
    u32x2 v;
    asm volatile("ds_read_b64_tr_b16 %0, %1" : "=v"(v) : "v"(addr));
    return v;
}
__device__ __forceinline__ bf16x8 join(const u32x2& lo, const u32x2& hi) {
    return __builtin_bit_cast(bf16x8, u32x4{lo[0], lo[1], hi[0], hi[1]});
}

template <int NT>
__global__ __launch_bounds__(256, 1) void first_weight_grad_kernel(const FirstGradArgs a) {
    extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];
    unsigned char* const patches = smem + kDyStages * kDyBytes;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int o0 = static_cast<int>(blockIdx.y) * 64;
    const int first = static_cast<int>(blockIdx.x) * a.per;
    const int last = first + a.per < a.tiles ? first + a.per : a.tiles;
    const __amdgpu_buffer_rsrc_t rx = make_rsrc(a.X, a.x_bytes), ry = make_rsrc(a.dY, a.dy_bytes);

    struct At { int img, oh, ow; };
    auto place = [&](int t) __attribute__((always_inline)) {
        const uint32_t row = fdiv_u(static_cast<uint32_t>(t), a.divTX);
        const uint32_t img = fdiv_u(row, a.divTY);
        return At{static_cast<int>(img), static_cast<int>(row - img * ((a.P + kTile - 1) / kTile)) * kTile,
                  (t - static_cast<int>(row) * ((a.Q + kTile - 1) / kTile)) * kTile};
    };
    // this wave's part of dY: 1 KB blocks of eight pixels; 16-byte chunk c of pixel p lies at position c ^ 2 (p & 3), so that the
    // four pixels of a transposing read fall in different banks
    auto load_dy = [&](int t, const At& at, int stage) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < kDyLoads; ++i) {
            const int px = (wave * kDyLoads + i) * 8 + (lane >> 3);
            const int oh = at.oh + px / kTile, ow = at.ow + px % kTile, o = o0 + ((lane & 7) ^ (2 * (px & 3))) * 8;
            const bool ok = t < last && oh < a.P && ow < a.Q && o < a.O;
            const uint32_t off = static_cast<uint32_t>(((at.img * a.P + oh) * a.Q + ow) * a.O + o) * 2u;
            buf_dma16(ry, ok ? off : kBufOutside, 0u, smem + stage * kDyBytes + (wave * kDyLoads + i) * 1024);
        }
    };
    typedef uint32_t u32x3 __attribute__((ext_vector_type(3)));
    u32x3 xr[kXLoads];
    auto load_x = [&](int t, const At& at) __attribute__((always_inline)) {
        const int h0 = at.oh * a.sh - a.ph, x0 = at.ow * a.sw - a.pw - a.xoff;
#pragma unroll
        for (int i = 0; i < kXLoads; ++i) {
            const int idx = i * 256 + tid;
            const int r = static_cast<int>(fdiv_u(static_cast<uint32_t>(idx), a.divPairs));
            const int h = h0 + r, x = x0 + 2 * (idx - r * a.pairs);
            // x and W are even: both pixels of a pair lie inside or neither
            const bool ok = t < last && idx < a.npairs && static_cast<unsigned>(h) < static_cast<unsigned>(a.H) &&
                            static_cast<unsigned>(x) < static_cast<unsigned>(a.W);
            const uint32_t off = static_cast<uint32_t>((at.img * a.H + h) * a.W + x) * 6u;
            xr[i] = __builtin_bit_cast(u32x3, __builtin_amdgcn_raw_buffer_load_b96(rx, ok ? off : kBufOutside, 0, 0));
        }
    };
    auto store_x = [&](int buf) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < kXLoads; ++i) {
            const int idx = i * 256 + tid;
            if (idx < a.npairs)
                *reinterpret_cast<u32x4*>(patches + buf * a.patch_bytes + idx * 16) =
                    u32x4{xr[i][0], xr[i][1] & 0xFFFFu, (xr[i][1] >> 16) | (xr[i][2] << 16), xr[i][2] >> 16};
        }
    };

    // Fragment addresses.  A transposing read of 16 lanes: lane L receives element L & 3 of the 8-byte rows whose addresses lanes
    // (L >> 2) + 4 e supply, e = 0..3.  Lane group g covers columns (g & 1) * 16 .. +15 of a 32-wide block and pixels
    // (g >> 1) * 8 .. +7 of the row in two reads; lane `s` of the group supplies block of four (s & 3), pixel (s >> 2).
    const int g = lane >> 4, s4 = lane & 3, e = (lane >> 2) & 3;
    const int px0 = (g >> 1) * 8 + e;                   // + 4 for the second read
    const uint32_t lds = static_cast<uint32_t>(
        reinterpret_cast<uintptr_t>((__attribute__((address_space(3))) unsigned char*)smem));
    uint32_t aoff[2];
#pragma unroll
    for (int ot = 0; ot < 2; ++ot) {
        const int chunk = ot * 4 + (g & 1) * 2 + (s4 >> 1);
        aoff[ot] = lds + static_cast<uint32_t>(px0 * 128 + (chunk ^ (2 * e)) * 16 + (s4 & 1) * 8);
    }
    uint32_t boff[NT];
#pragma unroll
    for (int t = 0; t < NT; ++t) {
        int u = 2 * t + (g & 1);
        if (u >= a.units) u = 0;                        // a block that is not stored
        const int r = u / a.G, tg = u - r * a.G;
        boff[t] = lds + kDyStages * kDyBytes + static_cast<uint32_t>((r * a.PW + px0 * a.sw + tg * 4 + s4 + a.xoff) * 8);
    }
    const uint32_t four_px = static_cast<uint32_t>(4 * a.sw * 8), row_bytes = static_cast<uint32_t>(a.sh * a.PW * 8);

    f32x16 acc[2][NT];
#pragma unroll
    for (int ot = 0; ot < 2; ++ot)
#pragma unroll
        for (int t = 0; t < NT; ++t)
#pragma unroll
            for (int k = 0; k < 16; ++k) acc[ot][t][k] = 0.0f;

    u32x2 fa[2][2][2], fb[2][NT][2];
    auto read_row = [&](int row, int stage, int buf, u32x2 (&ra)[2][2], u32x2 (&rb)[NT][2]) __attribute__((always_inline)) {
        const uint32_t da = static_cast<uint32_t>(stage * kDyBytes + row * kTile * 128);
        const uint32_t db = static_cast<uint32_t>(buf * a.patch_bytes) + static_cast<uint32_t>(row) * row_bytes;
#pragma unroll
        for (int ot = 0; ot < 2; ++ot) {
            ra[ot][0] = tr_read(aoff[ot] + da);
            ra[ot][1] = tr_read(aoff[ot] + da + 4 * 128);
        }
#pragma unroll
        for (int t = 0; t < NT; ++t) {
            rb[t][0] = tr_read(boff[t] + db);
            rb[t][1] = tr_read(boff[t] + db + four_px);
        }
    };
    auto landed = [&](u32x2 (&ra)[2][2], u32x2 (&rb)[NT][2]) __attribute__((always_inline)) {
        lds_wait<0>();
        lds_ready<4>(&ra[0][0]);
        lds_ready<2 * NT>(&rb[0][0]);
    };

    // ---- prologue: dY of three tiles, X of two ----
    At at0 = place(first);                              // at0, at1, at2: tiles t, t + 1, t + 2
    load_x(first, at0);
    load_dy(first, at0, 0);
    At at1 = place(first + 1), at2 = place(first + 2);
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_waitcnt(vmcnt_imm(0));
    store_x(0);
    load_dy(first + 1, at1, 1);
    load_x(first + 1, at1);
    load_dy(first + 2, at2, 2);
    for (int t = first; t < last; ++t) {
        const int k = t - first, stage = k & 3, buf = k & 1;
        // dY of this tile and its patch are complete in every wave (see below), and nobody reads the tile before any more
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
        // the patch of the next tile: its loads and everything older, dY of the next tile among it, must have landed; only the
        // loads of dY issued after it stay in flight
        __builtin_amdgcn_s_waitcnt(vmcnt_imm(kDyLoads));
        store_x(buf ^ 1);
        const At at3 = place(t + 3);
        load_x(t + 2, at2);
        load_dy(t + 3, at3, (k + 3) & 3);
        asm volatile("" ::: "memory");
        read_row(wave * 4, stage, buf, fa[0], fb[0]);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            landed(fa[i & 1], fb[i & 1]);
            __builtin_amdgcn_sched_barrier(0);
            if (i < 3) read_row(wave * 4 + i + 1, stage, buf, fa[(i + 1) & 1], fb[(i + 1) & 1]);
            __builtin_amdgcn_sched_barrier(0);
            // Past the edge of the output dY is zero, but the windows of such pixels still hold X: zero as well, so that an
            // infinity there stays out of taps whose sum does not contain it (0.2-0.3 us of a launch; a loop body of its own
            // for such tiles doubles the accumulators' registers: 45 -> 102 us for the stem).
            const int inside = at0.oh + wave * 4 + i < a.P ? a.Q - at0.ow : 0;        // pixels of this row
            if (__builtin_expect(inside < kTile, 0)) {
                const int left = inside - (g >> 1) * 8;
#pragma unroll
                for (int d = 0; d < 4; ++d) {
                    const uint32_t keep = left >= 2 * d + 2 ? 0xFFFFFFFFu : left == 2 * d + 1 ? 0xFFFFu : 0u;
#pragma unroll
                    for (int n = 0; n < NT; ++n) fb[i & 1][n][d >> 1][d & 1] &= keep;
                }
            }
#pragma unroll
            for (int n = 0; n < NT; ++n)
#pragma unroll
                for (int ot = 0; ot < 2; ++ot)
                    acc[ot][n] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(join(fa[i & 1][ot][0], fa[i & 1][ot][1]),
                                                                         join(fb[i & 1][n][0], fb[i & 1][n][1]), acc[ot][n], 0, 0, 0);
            __builtin_amdgcn_sched_barrier(0);
        }
        at0 = at1;
        at1 = at2;
        at2 = at3;
    }
    // loads past the last tile still target LDS
    __builtin_amdgcn_s_waitcnt(vmcnt_imm(0));
    asm volatile("" ::: "memory");
    __syncthreads();

    // ---- sum over the waves, 32 filters at a time, and the partial tile ----
    f32x4* red = reinterpret_cast<f32x4*>(smem);        // [wave][NT][4][64]
    float* out = a.partial + static_cast<int64_t>(blockIdx.x) * a.O * a.J;
#pragma unroll
    for (int ot = 0; ot < 2; ++ot) {
#pragma unroll
        for (int t = 0; t < NT; ++t)
#pragma unroll
            for (int q4 = 0; q4 < 4; ++q4) {
                const f32x16& v = acc[ot][t];
                red[((wave * NT + t) * 4 + q4) * 64 + lane] = f32x4{v[q4 * 4], v[q4 * 4 + 1], v[q4 * 4 + 2], v[q4 * 4 + 3]};
            }
        __syncthreads();
        for (int item = tid; item < NT * 256; item += 256) {
            f32x4 v = red[item];
#pragma unroll
            for (int w = 1; w < 4; ++w) v += red[w * NT * 256 + item];
            const int l = item & 63, q4 = (item >> 6) & 3, t = item >> 8;
            const int j = t * 32 + (l & 31), o = o0 + ot * 32 + q4 * 8 + (l >> 5) * 4;
            if (j < a.J)
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    if (o + i < a.O) out[static_cast<int64_t>(o + i) * a.J + j] = v[i];
        }
        __syncthreads();
    }
}

template <int NT>
int32_t launch(const FirstGradArgs& a, dim3 grid, hipStream_t st) {
    auto k = first_weight_grad_kernel<NT>;
    constexpr int kMost = 160 * 1024;
    static std::once_flag once;
    static bool allowed = false;
    std::call_once(once, [&] {
        allowed = hipFuncSetAttribute(reinterpret_cast<const void*>(k), hipFuncAttributeMaxDynamicSharedMemorySize, kMost) == hipSuccess;
    });
    if (!allowed) return TWN_ERR_HIP;
    k<<<grid, 256, kDyStages * kDyBytes + 2 * a.patch_bytes, st>>>(a);
    return launch_status();
}

}  // namespace

FirstGradPlan plan_first_weight_grad(const WgShape& w) {
    FirstGradPlan p{};
    if (w.C != 3 || w.O % 8 != 0 || w.R > 7 || w.S > 7 || w.sh > 2 || w.sw > 2 || w.dh != 1 || w.dw != 1 || w.W % 2 != 0) return p;
    const int64_t tx = (w.Q + kTile - 1) / kTile, ty = (w.P + kTile - 1) / kTile, tiles = tx * ty * w.N;
    if (static_cast<int64_t>(w.N) * w.H * w.W * 6 >= (1LL << 31) || static_cast<int64_t>(w.N) * w.P * w.Q * w.O * 2 >= (1LL << 31) ||
        tiles >= (1LL << 30))
        return p;
    p.G = (w.S + 3) / 4;
    p.J = w.R * p.G * 16;
    p.tiles = static_cast<int32_t>(tiles);
    // one workgroup per CU; fewer where a range costs more (its partial tile, written and read: 0.34 us per MB) than the tiles
    // it saves (0.7 us each)
    const int groups = (w.O + 63) / 64;
    int64_t splits = groups < 256 ? 256 / groups : 1;
    if (splits > tiles) splits = tiles;
    const double mb = static_cast<double>(w.O) * p.J * 4e-6;
    double best = 1e30;
    for (int64_t s = splits; s >= 1; s /= 2) {
        const int64_t per = (tiles + s - 1) / s, used = (tiles + per - 1) / per;
        const double us = 0.7 * static_cast<double>(per) + 0.34 * mb * static_cast<double>(used);
        if (us < best) {
            best = us;
            p.per = static_cast<int32_t>(per);
            p.splits = static_cast<int32_t>(used);
        }
    }
    p.use = 1;
    return p;
}

int32_t launch_first_weight_grad(const WgShape& w, int32_t ph, int32_t pw, const FirstGradPlan& p, const uint16_t* X,
                                 const uint16_t* dY, float* partial, hipStream_t st) {
    FirstGradArgs a{};
    a.X = X; a.dY = dY; a.partial = partial;
    a.N = w.N; a.H = w.H; a.W = w.W; a.O = w.O; a.P = w.P; a.Q = w.Q;
    a.sh = w.sh; a.sw = w.sw; a.ph = ph; a.pw = pw;
    a.xoff = pw & 1;            // a patch starts at an even column: its pairs are four-byte aligned
    a.G = p.G; a.units = w.R * p.G; a.J = p.J;
    a.PW = ((kTile - 1) * w.sw + 4 * p.G + a.xoff + 1) & ~1;
    a.pairs = a.PW / 2;
    a.npairs = ((kTile - 1) * w.sh + w.R) * a.pairs;
    a.patch_bytes = a.npairs * 16;
    if (a.npairs > kXLoads * 256 || kDyStages * kDyBytes + 2 * a.patch_bytes > 160 * 1024) return TWN_ERR_UNSUPPORTED;
    a.tiles = p.tiles; a.per = p.per;
    a.divTX = make_fastdiv_u((w.Q + kTile - 1) / kTile);
    a.divTY = make_fastdiv_u((w.P + kTile - 1) / kTile);
    a.divPairs = make_fastdiv_u(a.pairs);
    a.x_bytes = static_cast<uint32_t>(static_cast<int64_t>(w.N) * w.H * w.W * 6);
    a.dy_bytes = static_cast<uint32_t>(static_cast<int64_t>(w.N) * w.P * w.Q * w.O * 2);
    const dim3 grid(static_cast<unsigned>(p.splits), static_cast<unsigned>((w.O + 63) / 64));
    const int nt = (a.units + 1) / 2;
    if (nt <= 2) return launch<2>(a, grid, st);
    if (nt <= 5) return launch<5>(a, grid, st);
    return launch<7>(a, grid, st);
}

}  // namespace twn
