// One block's part of a bias gradient, for its own launch and for the blocks that a final pass over partial tiles of dW carries.
#pragma once

#include <type_traits>

#include "twn_common.h"
#include "twn_kernels.h"

namespace twn {

constexpr int kBiasThreads = 512;
// LDS of a block, in floats (8 channels; single channels take an eighth of it)
constexpr int kBiasLds = kBiasThreads * 8;

// Group `group` of channels over pixels begin..end, dest[channel].  The sums are those of 512 threads, also in a block of fewer (a
// thread then takes several of their places in turn) or more: the result does not depend on the launch that carries the block.
// BATCH pixels are requested at once, those behind the last as the batch's first and counted as zeros: a loop over the rest behind one
// over whole batches costs the fetch of code that is only skipped, and lanes with and without a whole batch take turns.  One request of
// a wave is a cache line per lane, so a batch must not be much more than a thread's pixels: bias_groups.
template <int VEC, int THREADS, int BATCH>
__device__ __forceinline__ void bias_grad_group(const BiasGrad& b, int group, int64_t begin, int64_t end, float* __restrict__ dest,
                                                float* __restrict__ red) {
    const int chunk0 = group * b.chunks_per_group;
    const int left = (b.O + VEC - 1) / VEC - chunk0;
    const int gc = left < b.chunks_per_group ? left : b.chunks_per_group;      // chunks of VEC channels in this block
    const int rows = static_cast<int>(kBiasThreads / static_cast<uint32_t>(gc));
    for (int t = threadIdx.x; t < kBiasThreads; t += THREADS) {
        const int row = static_cast<int>(static_cast<uint32_t>(t) / static_cast<uint32_t>(gc)), ch = (chunk0 + t - row * gc) * VEC;
        float acc[VEC];
#pragma unroll
        for (int v = 0; v < VEC; ++v) acc[v] = 0.0f;
        if (row < rows) {
            const uint16_t* src = b.dY + ch;
            using Values = std::conditional_t<VEC == 8, u32x4, uint32_t>;
            auto load = [&](const uint16_t* at) -> Values {
                if constexpr (VEC == 8) return *reinterpret_cast<const u32x4*>(at);
                else return *at;
            };
            auto add = [&](const Values& x) {
                if constexpr (VEC == 8) {
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        acc[(2 * i) % VEC] += __uint_as_float(x[i] << 16);
                        acc[(2 * i + 1) % VEC] += __uint_as_float(x[i] & 0xFFFF0000u);
                    }
                } else {
                    acc[0] += __uint_as_float(x << 16);
                }
            };
            for (int64_t p = begin + row; p < end; p += BATCH * rows) {
                Values x[BATCH];
#pragma unroll
                for (int u = 0; u < BATCH; ++u) x[u] = load(src + (p + u * rows < end ? p + u * rows : p) * b.O);
#pragma unroll
                for (int u = 0; u < BATCH; ++u) {
                    if (p + u * rows >= end) x[u] = Values{};
                    add(x[u]);
                }
            }
        }
#pragma unroll
        for (int v = 0; v < VEC; ++v) red[t * VEC + v] = acc[v];     // [row][channel of the group]
    }
    __syncthreads();
    // column sums in two stages: `parts` threads per channel add runs of rows, then one adds the parts
    const int nch = gc * VEC, most = VEC == 8 ? kBiasThreads / VEC : 32;
    const int parts = kBiasThreads / nch < most ? kBiasThreads / nch : most;
    const int each = (rows + parts - 1) / parts;
    constexpr int TURNS = THREADS < kBiasThreads ? kBiasThreads / THREADS : 1;
    // 8 channels: eight rows a part, 64 parts; one: a row or two, 8 to 32 parts
    constexpr int kRows = VEC == 8 ? 8 : 1, kParts = VEC == 8 ? 16 : 8;
    float s[TURNS];
#pragma unroll
    for (int u = 0; u < TURNS; ++u) {
        const int t = threadIdx.x + u * THREADS, part = static_cast<int>(static_cast<uint32_t>(t) / static_cast<uint32_t>(nch)), c = t - part * nch;
        s[u] = 0.0f;
        if (part < parts) {
            const int last = (part + 1) * each < rows ? (part + 1) * each : rows;
#pragma unroll kRows
            for (int r = part * each; r < last; ++r) s[u] += red[r * nch + c];
        }
    }
    __syncthreads();
#pragma unroll
    for (int u = 0; u < TURNS; ++u) {
        const int t = threadIdx.x + u * THREADS, part = static_cast<int>(static_cast<uint32_t>(t) / static_cast<uint32_t>(nch)), c = t - part * nch;
        if (part < parts) red[part * nch + c] = s[u];
    }
    __syncthreads();
    for (int c = threadIdx.x; c < nch; c += THREADS) {
        float t = 0.0f;
#pragma unroll kParts
        for (int i = 0; i < parts; ++i) t += red[i * nch + c];
        if (chunk0 * VEC + c < b.O) dest[chunk0 * VEC + c] = t;
    }
    __syncthreads();        // the next group of channels reuses the rows
}

// The first b.blocks blocks of a final pass sum dbias, all pixels of a group each: its result in the block's place among the
// others, or -1 after a bias gradient.  Their own launch costs 4-5 us behind the final pass, which leaves most of the chip idle
// in layers of few pixels (us of a forward and backward: 3565 pixels, 40 -> 72 channels 5x5/2 37.1 -> 34.7).
template <int THREADS, bool BIAS>
__device__ __forceinline__ int final_pass_block(const BiasGrad& b, float* __restrict__ red) {
    if constexpr (!BIAS) return static_cast<int>(blockIdx.x);
    const int block = static_cast<int>(blockIdx.x) - b.blocks;
    if (block >= 0) return block;
    for (int group = blockIdx.x; group < b.groups; group += b.blocks) {
        if (b.vec == 8 && b.batch == 1) bias_grad_group<8, THREADS, 1>(b, group, 0, b.pixels, b.dbias, red);
        else if (b.vec == 8) bias_grad_group<8, THREADS, 4>(b, group, 0, b.pixels, b.dbias, red);
        else bias_grad_group<1, THREADS, 8>(b, group, 0, b.pixels, b.dbias, red);
    }
    return -1;
}

// One final pass of `blocks` blocks, with those of the bias gradient in front where there is one.
template <typename... Params, typename... Args>
void launch_final_pass(void (*plain)(Params...), void (*with_bias)(Params...), int64_t blocks, int threads, const BiasGrad& bias, hipStream_t st,
                       Args... args) {
    (bias.blocks > 0 ? with_bias : plain)<<<static_cast<unsigned>(blocks + bias.blocks), threads, 0, st>>>(args..., bias);
}

}  // namespace twn
