// Threshold ternarization on gfx950 (Sec. 2.3: rule of thumb for Delta, Eq. 3
// codes, Eq. 5 alpha; Alg. 1 steps 3-7).  HBM-streaming kernels:
//
//   abs_sum           pass 1: per-block float64 partial sums of |W|
//   mask_pack_flat    pass 2: Delta from the partials, then one more stream of W:
//                     masked float64 sum, count, and the 2-bit codes written in
//                     the same pass (flat layouts: R*S == 1 and K % 128 == 0)
//   mask_pack_gather  pass 2 for any [rows][C][R][S] layout: one thread per output
//                     word of the normal and of the transposed copy; the normal
//                     words also carry the masked sum and count
//   pack_gather       codes only (transposed copy of flat layouts, per-filter groups)
//   filter_pack       one Delta and alpha per filter: statistics and codes of 16 filters per workgroup
//   group_stats       one block per group for other groups and for filters that filter_pack does not take
//
// The block of pass 2 that delivers its partials last sums them in a fixed order -> Delta, alpha, nnz (see deliver()).
// All floating-point sums run in a fixed order: results are bit-identical from run to run; no floating-point atomics.
#include <mutex>

#include "twn_common.h"

namespace twn {

constexpr int kTernThreads = 256;
constexpr int kChunk = kTernThreads * 16;   // weights per block iteration
constexpr int kMaxBlocks = 4096;

struct TernWorkspace {
    double p1[kMaxBlocks];     // pass-1 partial sums of |W|; from slot kMaxPass1 on the tickets of pass 2
    double p2[kMaxBlocks];     // pass-2 partial masked sums
    uint64_t cnt[kMaxBlocks];  // pass-2 partial counts
};
// Tickets of pass 2, in lines of their own at the end of p1: sixteen that the blocks share out, and one that the last block
// of each of them takes.  Pass 1 zeroes them.
constexpr int kTickets = 17, kTicketStep = 16;
constexpr int kMaxPass1 = kMaxBlocks - kTickets * kTicketStep;

// This thread's whole float4s of the ragged chunk that starts at `base`, zeros behind the last one.  The at most three weights behind
// all float4s are taken one by one by the thread that would own their float4, after its others.  Element by element in all threads,
// and with a branch per element around every load, the code alone was up to 1.1 us of an update of few weights (16x16: 4.1, so 2.8).
__device__ __forceinline__ void load_tail(const float* __restrict__ p, int64_t base, int64_t n, float4* v) {
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const int64_t idx = base + static_cast<int64_t>(j * kTernThreads + threadIdx.x) * 4;
        v[j] = float4{0.0f, 0.0f, 0.0f, 0.0f};
        if (idx + 3 < n) v[j] = *reinterpret_cast<const float4*>(p + idx);
    }
}
__device__ __forceinline__ bool owns_last(int64_t n) { return static_cast<int>(threadIdx.x) == static_cast<int>(n / 4 % kTernThreads); }

// The block that takes the ragged chunk behind `nfull` whole ones: fewer than 2^28 chunks, as tensors have fewer than 2^40 weights.
__device__ __forceinline__ int tail_block(int64_t nfull, int nblk) {
    return static_cast<int>(static_cast<uint32_t>(nfull) % static_cast<uint32_t>(nblk));
}

// Pass 1 of block `bid` out of `nblk` cooperating blocks: float64 partial sum of |W| -> partial[bid].
__device__ __forceinline__ void abs_sum_body(const float* __restrict__ W, int64_t n, double* __restrict__ partial,
                                             int bid, int nblk) {
    __shared__ double scratch[16];
    const int tid = threadIdx.x;
    const int64_t nfull = n / kChunk;          // chunks that need no bounds test
    double acc = 0.0;
    auto load4 = [&](int64_t c, float4* v) {
        const float4* src = reinterpret_cast<const float4*>(W + c * kChunk);
#pragma unroll
        for (int j = 0; j < 4; ++j) v[j] = src[j * kTernThreads + tid];
    };
    // software pipeline: the next chunk's loads are in flight while this one is summed
    int64_t c = bid;
    float4 cur[4];
    if (c < nfull) load4(c, cur);
    while (c < nfull) {
        const int64_t nx = c + nblk;
        float4 nxt[4];
        if (nx < nfull) load4(nx, nxt);
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            acc += static_cast<double>(fabsf(cur[j].x));
            acc += static_cast<double>(fabsf(cur[j].y));
            acc += static_cast<double>(fabsf(cur[j].z));
            acc += static_cast<double>(fabsf(cur[j].w));
        }
        if (nx < nfull) {
#pragma unroll
            for (int j = 0; j < 4; ++j) cur[j] = nxt[j];
        }
        c = nx;
    }
    // ragged tail (at most one chunk), taken by one block after its full chunks; element by element behind bounds tests it was
    // sixteen memory latencies.  Requested before the full chunks it would keep 16 registers more alive in all blocks.
    if (nfull * kChunk < n && bid == tail_block(nfull, nblk)) {
        load_tail(W, nfull * kChunk, n, cur);
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            acc += static_cast<double>(fabsf(cur[j].x));
            acc += static_cast<double>(fabsf(cur[j].y));
            acc += static_cast<double>(fabsf(cur[j].z));
            acc += static_cast<double>(fabsf(cur[j].w));
        }
        if (owns_last(n))
            for (int64_t idx = n & ~static_cast<int64_t>(3); idx < n; ++idx) acc += static_cast<double>(fabsf(W[idx]));
    }
    const double total = block_sum(acc, scratch);
    if (tid == 0) partial[bid] = total;
    if (bid == 0 && tid < kTickets) partial[kMaxPass1 + tid * kTicketStep] = 0.0;
}

__global__ __launch_bounds__(kTernThreads) void abs_sum_kernel(const float* __restrict__ W, int64_t n,
                                                               double* __restrict__ partial) {
    abs_sum_body(W, n, partial, blockIdx.x, gridDim.x);
}

// Delta = (float)((double)f * S1 / n), S1 = fixed-order sum of the pass-1 partials.
__device__ __forceinline__ float delta_from_partials(const double* __restrict__ p1, int nb1, float f,
                                                     int64_t n, double* scratch) {
    double acc = 0.0;
    for (int i = threadIdx.x; i < nb1; i += blockDim.x) acc += p1[i];
    const double s1 = block_sum(acc, scratch);
    return static_cast<float>((static_cast<double>(f) * s1) / static_cast<double>(n));
}

// End of pass 2 of block `slot` out of `slots`: its masked sum and count go to the workspace, and the block that delivers last
// sums all of them in slot order and writes Delta, alpha and nnz, which saves the launch that used to do it (4-5 us).
// The partials are agent-scope atomic stores: they reach memory past the XCD's L2 by themselves, so waiting for them before
// taking the ticket orders them, and the last block reads them by atomic loads that no stale L2 line can serve.  (A release
// fence would write back the whole L2 of the XCD, once per block: 75 us on 2^28 weights.)  One counter for a
// thousand blocks costs 7 us, two levels of them 2.  The tickets are left at zero, for another pass 2 on the same sums.
__device__ __forceinline__ void deliver(TernWorkspace* __restrict__ ws, int slot, int slots, double sum, unsigned long long n,
                                        float delta, float* __restrict__ delta_out, float* __restrict__ alpha_out,
                                        uint64_t* __restrict__ nnz_out, double* scratch, unsigned long long* scratch_u) {
    __shared__ int last;
    unsigned long long* tickets = reinterpret_cast<unsigned long long*>(&ws->p1[kMaxPass1]);
    constexpr int kShared = kTickets - 1;
    if (threadIdx.x == 0) {
        __hip_atomic_store(&ws->p2[slot], sum, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __hip_atomic_store(reinterpret_cast<unsigned long long*>(&ws->cnt[slot]), n, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        const int mine = slot % kShared, of = (slots - mine + kShared - 1) / kShared;
        auto take = [&](int t) {
            return __hip_atomic_fetch_add(tickets + t * kTicketStep, 1ULL, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        };
        last = take(mine) == static_cast<unsigned long long>(of - 1) &&
               take(kShared) == static_cast<unsigned long long>((slots < kShared ? slots : kShared) - 1);
    }
    __syncthreads();
    if (!last) return;
    double acc = 0.0;
    unsigned long long c = 0;
#pragma unroll 4
    for (int i = threadIdx.x; i < slots; i += blockDim.x) {
        acc += __hip_atomic_load(&ws->p2[i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        c += __hip_atomic_load(reinterpret_cast<unsigned long long*>(&ws->cnt[i]), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    const double s = block_sum(acc, scratch);
    const unsigned long long total = block_sum(c, scratch_u);
    if (threadIdx.x == 0) {
        delta_out[0] = delta;
        nnz_out[0] = total;
        alpha_out[0] = total ? static_cast<float>(s / static_cast<double>(total)) : 0.0f;
    }
    if (threadIdx.x < kTickets) tickets[threadIdx.x * kTicketStep] = 0ULL;
}

__device__ __forceinline__ uint32_t quad_or(uint32_t v) {
    // OR across the 4 lanes of a quad (DPP quad_perm [1,0,3,2] then [2,3,0,1]).
    v |= static_cast<uint32_t>(__builtin_amdgcn_update_dpp(0, static_cast<int>(v), 0xB1, 0xF, 0xF, false));
    v |= static_cast<uint32_t>(__builtin_amdgcn_update_dpp(0, static_cast<int>(v), 0x4E, 0xF, 0xF, false));
    return v;
}

// Pass 2 for flat layouts: the packed word index is (flat weight index)/16.
// A wave covers 1024 consecutive weights per step with four fully coalesced
// float4 loads; the four lanes of a quad hold the 16 weights of one output
// word, which is assembled with two DPP ORs and written by the lane whose
// position in the quad equals the load index, so each wave stores 256
// contiguous bytes.
__device__ __forceinline__ void mask_pack_flat_body(
    const float* __restrict__ W, int64_t n, TernWorkspace* __restrict__ ws, int nb1, float f,
    uint32_t* __restrict__ packed, int reverse, int bid, int nblk, int slots, float* __restrict__ delta_out,
    float* __restrict__ alpha_out, uint64_t* __restrict__ nnz_out) {
    const double* __restrict__ p1 = ws->p1;
    __shared__ double scratch[16];
    __shared__ unsigned long long scratch_u[16];
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = tid >> 6;
    const int ql = lane & 3;
    const float delta = delta_from_partials(p1, nb1, f, n, scratch);

    const int64_t nchunks = (n + kChunk - 1) / kChunk;
    const int64_t nfull = n / kChunk;   // chunks that need no bounds test
    const int64_t n4 = n >> 2;          // n % 16 == 0 here
    const int64_t nwords = n >> 4;
    double acc = 0.0;
    uint32_t count = 0;

    auto wave_base = [&](int64_t it) -> int64_t {
        const int64_t c = reverse ? (nchunks - 1 - it) : it;
        return c * kChunk + wave * 1024;   // first weight of this wave's span
    };
    auto load4 = [&](int64_t wbase, float4* v, bool guard) {
        const float4* src = reinterpret_cast<const float4*>(W + wbase);
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            if (guard) {
                const int64_t i4 = (wbase >> 2) + j * 64 + lane;
                v[j] = (i4 < n4) ? src[j * 64 + lane] : make_float4(0.f, 0.f, 0.f, 0.f);
            } else {
                v[j] = src[j * 64 + lane];
            }
        }
    };
    auto process = [&](const float4* v, int64_t wbase, bool guard) {
        uint32_t mine = 0;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const uint32_t f0 = code_field(v[j].x, delta), f1 = code_field(v[j].y, delta);
            const uint32_t f2 = code_field(v[j].z, delta), f3 = code_field(v[j].w, delta);
            // adding +0.0 for the masked-out weights leaves the float64 sum unchanged
            acc += static_cast<double>(f0 ? fabsf(v[j].x) : 0.0f);
            acc += static_cast<double>(f1 ? fabsf(v[j].y) : 0.0f);
            acc += static_cast<double>(f2 ? fabsf(v[j].z) : 0.0f);
            acc += static_cast<double>(f3 ? fabsf(v[j].w) : 0.0f);
            count += (f0 & 1u) + (f1 & 1u) + (f2 & 1u) + (f3 & 1u);
            uint32_t word = ((f0 | (f2 << 2)) << (4 * ql)) | ((f1 | (f3 << 2)) << (16 + 4 * ql));
            word = quad_or(word);
            if (ql == j) mine = word;
        }
        const int64_t widx = (wbase >> 4) + (lane >> 2) + 16 * ql;
        if (!guard || widx < nwords) packed[widx] = mine;
    };

    // iteration `it` maps to chunk it (or nchunks-1-it when walking backwards); a chunk is ragged only
    // if it is the last one in memory order, i.e. it == nchunks-1 forwards or it == 0 backwards
    const bool has_tail = nfull < nchunks;
    const int64_t tail_it = reverse ? 0 : nchunks - 1;
    int64_t it = bid;
    if (has_tail && it == tail_it) {            // only possible for the first iteration of one block
        float4 v[4];
        const int64_t wb = wave_base(it);
        load4(wb, v, true);
        process(v, wb, true);
        it += nblk;
    }
    const int64_t it_end = (has_tail && !reverse) ? nchunks - 1 : nchunks;
    // software pipeline over the full chunks: next loads in flight while this chunk is processed
    float4 cur[4];
    if (it < it_end) load4(wave_base(it), cur, false);
    while (it < it_end) {
        const int64_t nx = it + nblk;
        float4 nxt[4];
        if (nx < it_end) load4(wave_base(nx), nxt, false);
        process(cur, wave_base(it), false);
        if (nx < it_end) {
#pragma unroll
            for (int j = 0; j < 4; ++j) cur[j] = nxt[j];
        }
        it = nx;
    }
    if (has_tail && !reverse && static_cast<int64_t>(bid) == tail_it % nblk && tail_it >= nblk) {
        float4 v[4];
        const int64_t wb = wave_base(tail_it);
        load4(wb, v, true);
        process(v, wb, true);
    }
    const double total = block_sum(acc, scratch);
    const unsigned long long ctotal = block_sum(static_cast<unsigned long long>(count), scratch_u);
    deliver(ws, bid, slots, total, ctotal, delta, delta_out, alpha_out, nnz_out, scratch, scratch_u);
}

__global__ __launch_bounds__(kTernThreads) void mask_pack_flat_kernel(
    const float* __restrict__ W, int64_t n, TernWorkspace* __restrict__ ws, int nb1, float f,
    uint32_t* __restrict__ packed, int reverse, float* __restrict__ delta_out, float* __restrict__ alpha_out,
    uint64_t* __restrict__ nnz_out) {
    mask_pack_flat_body(W, n, ws, nb1, f, packed, reverse, blockIdx.x, gridDim.x, gridDim.x, delta_out, alpha_out, nnz_out);
}

// ---- large flat tensors: codes from ONE stream of W ---------------------------------------------------------
// Both passes of a tensor that no cache holds are bound by the read of W, and Delta is known only after the first.  But it is
// known nearly enough beforehand: a sample gives a band [lo, hi] that holds Delta, a weight outside the band has its code
// whatever Delta turns out to be, and only the words with a weight inside are looked at again.
//   sample    a jittered sample of W: float64 sums of 256 disjoint parts of it
//   band_pack one stream: the pass-1 partials (the same sums, bit for bit, as abs_sum_kernel's), the codes as if Delta were
//             hi, the masked sum and count of the weights above hi, and one bit per word that has a weight inside the band
//   band_fix  Delta; the marked words again, whole, with their weights inside the band added to sum and count.  Where Delta
//             fell outside the band (a sample that misleads, sums that are not finite) it is a whole pass 2 instead: no
//             result depends on the sample.
// 2^28 weights: 368 -> 244 us (6 + 217 + 23); 2^26: 89 -> 62; 2^24: 31.1 -> 29.8, the least that gains.
constexpr int kBandParts = 256;
struct BandState {
    double part[kBandParts];   // sample sums, weights_per_part weights each
    float lo, hi;
};
constexpr int64_t kBandMinWeights = 1LL << 24;
constexpr int kBandSegment = 1024;             // consecutive weights of the sample
inline int64_t band_sample(int64_t n) {        // multiple of 256 segments: 1/64 of the tensor within 2^18 .. 2^22 weights
    int64_t s = n / 64;
    if (s < (1LL << 18)) s = 1LL << 18;
    if (s > (1LL << 22)) s = 1LL << 22;
    return s / (kBandParts * kBandSegment) * (kBandParts * kBandSegment);
}
inline size_t band_bytes(int64_t n) {          // state, then one bit per word, 64 words of a wave and chunk together
    const int64_t chunks = (n + kChunk - 1) / kChunk;
    return sizeof(TernWorkspace) + round_up(sizeof(BandState), 256) + static_cast<size_t>(chunks) * 4 * sizeof(uint64_t);
}

// Block b sums the segments b, b + 256, ... of `segments`; segment g lies at a place of its own in the g-th of `segments`
// equal stretches of W (a fixed place would meet the same columns of every row).
__global__ __launch_bounds__(kTernThreads) void band_sample_kernel(const float* __restrict__ W, int64_t n, int segments,
                                                                   BandState* __restrict__ st) {
    __shared__ double scratch[16];
    const int64_t stretch = n / segments;
    const uint32_t places = static_cast<uint32_t>((stretch - kBandSegment) / 4 + 1 < (1 << 24) ? (stretch - kBandSegment) / 4 + 1
                                                                                               : (1 << 24));
    double acc = 0.0;
#pragma unroll 4
    for (int g = blockIdx.x; g < segments; g += kBandParts) {
        const uint32_t at = __umulhi(static_cast<uint32_t>(g) * 2654435769u, places);
        const float4 v = reinterpret_cast<const float4*>(W + (g * stretch & ~int64_t{3}) + 4 * static_cast<int64_t>(at))[threadIdx.x];
        acc += static_cast<double>(fabsf(v.x)) + static_cast<double>(fabsf(v.y)) + static_cast<double>(fabsf(v.z)) +
               static_cast<double>(fabsf(v.w));
    }
    const double total = block_sum(acc, scratch);
    if (threadIdx.x == 0) st->part[blockIdx.x] = total;
}

// The band: the sample's estimate of Delta plus and minus four standard errors, these from the spread of the parts: a random
// sample misses once in 16000 tensors, and with 5.5 a third more words are read again.
__device__ __forceinline__ void band_of(const BandState* __restrict__ st, int segments, float f, double* scratch, float* lo,
                                        float* hi) {
    const double x = st->part[threadIdx.x];            // kTernThreads == kBandParts
    const double mean = block_sum(x, scratch) / kBandParts;
    const double spread = block_sum((x - mean) * (x - mean), scratch);
    const double scale = static_cast<double>(f) * kBandParts / (static_cast<double>(segments) * kBandSegment);
    const double half = 4.0 * sqrt(spread / (kBandParts * (kBandParts - 1.0))) * scale + 1e-6 * mean * scale;
    const double low = mean * scale - half;
    *lo = low > 0.0 ? static_cast<float>(low) : 0.0f;
    *hi = static_cast<float>(mean * scale + half);
}

// Words of one chunk: lane l of wave w holds float4 number j * 256 + 64 w + l of it (as abs_sum_body reads it), i.e. the quad
// l / 4 holds word 64 j + 16 w + l / 4; lane l stores the word of j = l % 4.
__device__ __forceinline__ int64_t band_word(int64_t chunk, int wave, int lane) {
    return chunk * (kChunk / 16) + (lane & 3) * 64 + wave * 16 + (lane >> 2);
}

__global__ __launch_bounds__(kTernThreads) void band_pack_kernel(const float* __restrict__ W, int64_t n, int segments, float f,
                                                                 TernWorkspace* __restrict__ ws, BandState* __restrict__ st,
                                                                 uint64_t* __restrict__ marks, uint32_t* __restrict__ packed) {
    __shared__ double scratch[16];
    __shared__ unsigned long long scratch_u[16];
    const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid / kWave, ql = lane & 3;
    const int bid = blockIdx.x, nblk = gridDim.x;
    const int64_t nfull = n / kChunk, n4 = n >> 2, nwords = n >> 4;
    auto load4 = [&](int64_t c, float4* v) {
        const float4* src = reinterpret_cast<const float4*>(W + c * kChunk);
#pragma unroll
        for (int j = 0; j < 4; ++j) v[j] = src[j * kTernThreads + tid];
    };
    float4 cur[4];
    int64_t c = bid;
    if (c < nfull) load4(c, cur);
    float lo, hi;
    band_of(st, segments, f, scratch, &lo, &hi);
    if (bid == 0 && tid == 0) {
        st->lo = lo;
        st->hi = hi;
    }
    double all = 0.0, acc = 0.0;
    uint32_t count = 0;                                // per wave: every lane holds the wave's count
    unsigned long long many = 0;
    auto process = [&](const float4* v, int64_t chunk, bool guard) {
        uint32_t mine = 0;
        uint64_t inside = 0;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const float w4[4] = {v[j].x, v[j].y, v[j].z, v[j].w};
            uint32_t fld[4];
            uint64_t near = 0;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const float a = fabsf(w4[e]);
                const bool on = a > hi;
                const double a64 = static_cast<double>(a);
                all += a64;
                acc = fma(a64, on ? 1.0 : 0.0, acc);      // exact product
                const uint64_t above = __ballot(on);
                count += static_cast<uint32_t>(__popcll(above));
                near |= __ballot(a > lo) & ~above;
                fld[e] = on ? ((__float_as_uint(w4[e]) >> 31) << 1 | 1u) : 0u;
            }
            const uint32_t word = quad_or(((fld[0] | (fld[2] << 2)) << (4 * ql)) | ((fld[1] | (fld[3] << 2)) << (16 + 4 * ql)));
            if (ql == j) mine = word;
            near |= near >> 1;
            near |= near >> 2;
            inside |= (near & 0x1111111111111111ULL) << j;
        }
        const int64_t widx = band_word(chunk, wave, lane);
        if (!guard || widx < nwords) __builtin_nontemporal_store(mine, packed + widx);
        if (lane == 0) marks[chunk * 4 + wave] = inside;
    };
    while (c < nfull) {
        const int64_t nx = c + nblk;
        float4 nxt[4];
        if (nx < nfull) load4(nx, nxt);
        process(cur, c, false);
        many += count;
        count = 0;
        if (nx < nfull) {
#pragma unroll
            for (int j = 0; j < 4; ++j) cur[j] = nxt[j];
        }
        c = nx;
    }
    // ragged tail, taken by the block abs_sum_body gives it to
    if (nfull * kChunk < n && bid == tail_block(nfull, nblk)) {
        const float4* src = reinterpret_cast<const float4*>(W);
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int64_t i4 = nfull * (kChunk / 4) + j * kTernThreads + tid;
            cur[j] = i4 < n4 ? src[i4] : make_float4(0.f, 0.f, 0.f, 0.f);      // a zero is outside the band and adds nothing
        }
        process(cur, nfull, true);
        many += count;
    }
    const double total_all = block_sum(all, scratch);
    const double total = block_sum(acc, scratch);
    const unsigned long long ctotal = block_sum(lane == 0 ? many : 0ULL, scratch_u);
    if (tid == 0) {
        ws->p1[bid] = total_all;
        ws->p2[bid] = total;
        ws->cnt[bid] = ctotal;
    }
    if (bid == 0 && tid < kTickets) ws->p1[kMaxPass1 + tid * kTicketStep] = 0.0;
}

// A wave takes `per` marks at a time.  Block b adds its findings to the sums that block b of band_pack_kernel left (nb1 blocks,
// no more than here).
constexpr int kFixBlocks = 1024;
constexpr int kFixList = 4096;                         // 64 marks of 64 words
__global__ __launch_bounds__(kTernThreads) void band_fix_kernel(const float* __restrict__ W, int64_t n, int nb1, int per, float f,
                                                                TernWorkspace* __restrict__ ws, const BandState* __restrict__ st,
                                                                const uint64_t* __restrict__ marks, uint32_t* __restrict__ packed,
                                                                float* __restrict__ delta_out, float* __restrict__ alpha_out,
                                                                uint64_t* __restrict__ nnz_out) {
    __shared__ double scratch[16];
    __shared__ unsigned long long scratch_u[16];
    __shared__ uint16_t list_all[kTernThreads / kWave][kFixList];
    const float lo = st->lo, hi = st->hi;
    const float delta = delta_from_partials(ws->p1, nb1, f, n, scratch);
    if (!(lo <= delta && delta <= hi)) {               // also for a Delta that is no number
        mask_pack_flat_body(W, n, ws, nb1, f, packed, 1, blockIdx.x, gridDim.x, gridDim.x, delta_out, alpha_out, nnz_out);
        return;
    }
    const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave, ql = lane & 3;
    uint16_t* list = list_all[wave];
    const int64_t entries = (n + kChunk - 1) / kChunk * 4;
    const int64_t wave_id = static_cast<int64_t>(blockIdx.x) * (kTernThreads / kWave) + wave;
    const int64_t nwaves = static_cast<int64_t>(gridDim.x) * (kTernThreads / kWave);
    double acc = 0.0;
    uint32_t count = 0;
    for (int64_t e0 = wave_id * per; e0 < entries; e0 += nwaves * per) {
        uint64_t m = lane < per && e0 + lane < entries ? marks[e0 + lane] : 0ULL;
        const int own = __popcll(m);
        int before = own;                              // marked words of the lanes up to this one
#pragma unroll
        for (int off = 1; off < kWave; off <<= 1) {
            const int t = __shfl_up(before, off, kWave);
            if (lane >= off) before += t;
        }
        const int many = __shfl(before, kWave - 1, kWave);
        for (int at = before - own; m; m &= m - 1) list[at++] = static_cast<uint16_t>(lane * 64 + __ffsll(static_cast<unsigned long long>(m)) - 1);
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        // four lanes per word, four words of a quad in flight
        for (int i0 = lane >> 2; i0 < many; i0 += 64) {
            float4 v[4];
            int64_t widx[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                widx[u] = -1;
                if (i0 + 16 * u < many) {
                    const int item = list[i0 + 16 * u];
                    const int64_t entry = e0 + (item >> 6);
                    widx[u] = band_word(entry >> 2, static_cast<int>(entry & 3), item & 63);
                    v[u] = reinterpret_cast<const float4*>(W)[widx[u] * 4 + ql];
                }
            }
#pragma unroll
            for (int u = 0; u < 4; ++u)
                if (widx[u] >= 0) {                    // the same for the four lanes of a quad
                    const float w4[4] = {v[u].x, v[u].y, v[u].z, v[u].w};
                    uint32_t fld[4];
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        const float a = fabsf(w4[e]);
                        fld[e] = code_field(w4[e], delta);
                        if (a > delta && !(a > hi)) {
                            acc += static_cast<double>(a);
                            ++count;
                        }
                    }
                    const uint32_t word =
                        quad_or(((fld[0] | (fld[2] << 2)) << (4 * ql)) | ((fld[1] | (fld[3] << 2)) << (16 + 4 * ql)));
                    if (ql == 0) packed[widx[u]] = word;
                }
        }
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    }
    const bool left = static_cast<int>(blockIdx.x) < nb1;
    const double total = block_sum(acc, scratch) + (left ? ws->p2[blockIdx.x] : 0.0);
    const unsigned long long ctotal =
        block_sum(static_cast<unsigned long long>(count), scratch_u) + (left ? ws->cnt[blockIdx.x] : 0ULL);
    __syncthreads();                                   // the block's slot is read before it is written
    deliver(ws, blockIdx.x, gridDim.x, total, ctotal, delta, delta_out, alpha_out, nnz_out, scratch, scratch_u);
}

// The 16 weights of word j of an output row: filter `row`'s codes k = rs*C + c in the normal copy, input channel `row`'s codes
// k = rs*rows + o in the transposed one.  One division per word, then all sixteen loads are requested (the result: how many
// of them exist; the others read the tensor's first one).  With a 64-bit division and a wait per weight a
// call was (us) 19 instead of 13 for 300 x 200 x 3 x 3, 91 instead of 59 for 3333 x 5008.
// PACED: one load at a time.  Weights that follow one another in a word are taps apart in memory, and a cache line is used by the words
// of several taps, which other waves form at about the same time: that is one sixteenth of the tensor while all waves stand at the
// same weight, and the whole tensor with sixteen loads each, which no L2 holds from about 6 MB on.
__host__ __device__ inline bool paced_words(int64_t n, int RS) {
    // from 16 taps, i.e. half a line, on (us, all at once / paced: 1948x80x5x5 57 / 42, 1622x68x5x5 45 / 39, 4680x19x5x5 36 / 30, 1000x60x7x7 46 /
    // 35; some the other way, 746x189x5x5 60 / 72; below the line 357x29x5x5 10.7 / 14.1; 2000x700x3x3 113 / 203)
    return RS >= 16 && n >= (3 << 19);
}
template <bool TRANSPOSED, bool PACED>
__device__ __forceinline__ uint32_t gather_word(const float* __restrict__ W, int rows, int C, int RS, int row, int j, float (&w)[16]) {
    const uint32_t len = static_cast<uint32_t>(TRANSPOSED ? rows : C), k0 = static_cast<uint32_t>(j) * 16u;
    uint32_t rs = k0 / len, i = k0 - rs * len;
    const int64_t step = TRANSPOSED ? static_cast<int64_t>(C) * RS : RS;
    const int64_t base = static_cast<int64_t>(row) * (TRANSPOSED ? RS : step * C);
    const uint32_t k = len * static_cast<uint32_t>(RS);
    uint32_t real = k > k0 ? k - k0 : 0u;
#pragma unroll
    for (int t = 0; t < 16; ++t) {
        w[t] = W[static_cast<uint32_t>(t) < real ? base + i * step + rs : 0];
        if (PACED && t < 15) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        const bool next = ++i == len;
        i = next ? 0u : i;
        rs += next ? 1u : 0u;
    }
    asm volatile("" : "+v"(real));      // sixteen tests, not kept as sixteen masks: eight blocks a CU instead of seven
    return real;
}
// quotient of a word's number, which is below 2^31 for all but the largest tensors
__device__ __forceinline__ int64_t word_quotient(int64_t id, int d, bool narrow) {
    return narrow ? static_cast<int64_t>(static_cast<uint32_t>(id) / static_cast<uint32_t>(d)) : id / d;
}

// Pass 2 for any layout: grid-stride over the output words of the normal copy (which also carry the
// masked sum and count: every weight belongs to exactly one normal word) and of the transposed copy.
//   normal:     row = filter o,        k   = (r*S+s)*C + c
//   transposed: row = input channel c, k_T = (r*S+s)*rows + o   (threads ordered with c fastest)
template <bool PACED>
__device__ __forceinline__ void mask_pack_gather_body(
    const float* __restrict__ W, int rows, int C, int RS, TernWorkspace* __restrict__ ws, int nb1, float f,
    uint32_t* __restrict__ packed, int wpr, uint32_t* __restrict__ packed_T, int wprT, int bid, int nblk, int slots,
    float* __restrict__ delta_out, float* __restrict__ alpha_out, uint64_t* __restrict__ nnz_out,
    bool only_transposed = false, int slot0 = 0) {
    __shared__ double scratch[16];
    __shared__ unsigned long long scratch_u[16];
    const int64_t n = static_cast<int64_t>(rows) * C * RS;
    const float delta = delta_from_partials(ws->p1, nb1, f, n, scratch);
    const int64_t words_n = only_transposed ? 0 : static_cast<int64_t>(rows) * wpr;
    const int64_t words_t = packed_T ? static_cast<int64_t>(C) * wprT : 0;
    const bool narrow = words_n + words_t < (1LL << 31);
    double acc = 0.0;
    uint32_t count = 0;
    for (int64_t id = static_cast<int64_t>(bid) * blockDim.x + threadIdx.x; id < words_n + words_t;
         id += static_cast<int64_t>(nblk) * blockDim.x) {
        float w[16];
        uint32_t word = 0;
        if (id < words_n) {
            const int64_t o = word_quotient(id, wpr, narrow);
            const uint32_t real = gather_word<false, PACED>(W, rows, C, RS, static_cast<int>(o), static_cast<int>(id - o * wpr), w);
#pragma unroll
            for (int t = 0; t < 16; ++t) {
                const uint32_t fld = static_cast<uint32_t>(t) < real ? code_field(w[t], delta) : 0u;
                // adding +0.0 for the masked-out weights leaves the float64 sum unchanged
                acc += static_cast<double>(fld ? fabsf(w[t]) : 0.0f);
                count += fld & 1u;
                word |= fld << ((t & 1) * 16 + (t >> 1) * 2);
            }
            packed[id] = word;
        } else {
            const int64_t it = id - words_n, j = word_quotient(it, C, narrow);
            const int c = static_cast<int>(it - j * C);
            const uint32_t real = gather_word<true, PACED>(W, rows, C, RS, c, static_cast<int>(j), w);
#pragma unroll
            for (int t = 0; t < 16; ++t)
                word |= (static_cast<uint32_t>(t) < real ? code_field(w[t], delta) : 0u) << ((t & 1) * 16 + (t >> 1) * 2);
            packed_T[static_cast<int64_t>(c) * wprT + j] = word;
        }
    }
    const double total = block_sum(acc, scratch);
    const unsigned long long ctotal = block_sum(static_cast<unsigned long long>(count), scratch_u);
    deliver(ws, slot0 + bid, slots, total, ctotal, delta, delta_out, alpha_out, nnz_out, scratch, scratch_u);
}

template <bool PACED>
__global__ __launch_bounds__(kTernThreads) void mask_pack_gather_kernel(
    const float* __restrict__ W, int rows, int C, int RS, TernWorkspace* __restrict__ ws, int nb1, float f,
    uint32_t* __restrict__ packed, int wpr, uint32_t* __restrict__ packed_T, int wprT, float* __restrict__ delta_out,
    float* __restrict__ alpha_out, uint64_t* __restrict__ nnz_out) {
    mask_pack_gather_body<PACED>(W, rows, C, RS, ws, nb1, f, packed, wpr, packed_T, wprT, blockIdx.x, gridDim.x, gridDim.x, delta_out,
                          alpha_out, nnz_out);
}

// Codes of tensors with rows % 16 == 0 and C % 16 == 0 (filter banks, and matrices that also need the transposed copy),
// staged through LDS: block `bid` owns 16 consecutive filters x CT consecutive channels x all taps.  Its weights are 16
// contiguous runs of CT*R*S floats, read once with float4 loads, the first nine per thread before Delta is known; the 2-bit
// fields go to LDS as bytes in memory order, and the words of both copies are assembled from there, so no thread gathers
// from global memory.  Words written: per filter and tap CT/16 normal words; per channel and tap one transposed word (its
// 16 codes are the block's 16 filters).  Row padding words are written by the blocks with channel tile 0 (normal) and
// filter tile 0 (transposed).
// 16 code bytes of consecutive k -> one word of the packed format (even k in the low half-word).
__device__ __forceinline__ uint32_t word_of_bytes(const uint32_t* d) {
    uint32_t word = 0;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const uint32_t low = (d[i] & 3u) | ((d[i] >> 14) & 0xCu);
        const uint32_t high = ((d[i] >> 8) & 3u) | ((d[i] >> 22) & 0xCu);
        word |= (low | (high << 16)) << (4 * i);
    }
    return word;
}

// Four consecutive weights, four-byte aligned (a filter of odd length starts anywhere).
struct __attribute__((packed, aligned(4))) Weights4 {
    float w[4];
};

constexpr int kTileRows = 16;
constexpr int kTileLdsBytes = 16 * 64 * 25;   // CT <= 64 with R*S <= 25 taps; CT <= 1024 for matrices
__host__ __device__ inline int tile_ct(int C, int RS) {
    if (RS == 1) {
        // matrices: the largest power of two up to 1024 that divides C (runs of up to 4 KB per filter)
        int ct = 16;
        while (ct < 1024 && C % (2 * ct) == 0) ct *= 2;
        return ct;
    }
    return (C % 64 == 0) ? 64 : (C % 32 == 0) ? 32 : 16;
}
__host__ __device__ inline bool tile_ok(int rows, int C, int RS) {
    return RS >= 1 && RS <= 25 && rows % 16 == 0 && C % 16 == 0 &&
           static_cast<int64_t>(rows / 16) * (C / tile_ct(C, RS)) <= kMaxBlocks;
}

__device__ __forceinline__ void mask_pack_tile_body(const float* __restrict__ W, int rows, int C, int RS,
                                                    TernWorkspace* __restrict__ ws, int nb1, float f,
                                                    uint32_t* __restrict__ packed, int wpr, uint32_t* __restrict__ packed_T,
                                                    int wprT, int bid, float* __restrict__ delta_out,
                                                    float* __restrict__ alpha_out, uint64_t* __restrict__ nnz_out) {
    constexpr int U = 9;                           // 64 channels x 9 taps x 16 filters: nine float4 per thread
    __shared__ double scratch[16];
    __shared__ unsigned long long scratch_u[16];
    __shared__ __attribute__((aligned(16))) unsigned char codes[kTileLdsBytes];
    // A transposed word is four bytes of a row that 16-filter neighbours share: the blocks of one XCD (every eighth) take
    // consecutive filter tiles, so that its L2 collects whole lines (2048 x 320 x 3 x 3 with the pass before: 23.8 -> 22.1 us).
    const int CT = tile_ct(C, RS), otiles = rows / kTileRows, tiles = otiles * (C / CT);
    const int xcd = bid & 7, extra = tiles & 7;
    const int tile = xcd * (tiles >> 3) + (xcd < extra ? xcd : extra) + (bid >> 3);
    const int o0 = (tile % otiles) * kTileRows, c0 = (tile / otiles) * CT;
    const int seg = CT * RS, seg4 = seg / 4;       // floats (and code bytes) per filter in this block
    const int tid = threadIdx.x, items = kTileRows * seg4;
    const float* base = W + (static_cast<int64_t>(o0) * C + c0) * RS;
    const int64_t pitch = static_cast<int64_t>(C) * RS;
    const float inv = 1.0f / static_cast<float>(seg4);
    auto row_of = [&](int p) { return static_cast<int>((static_cast<float>(p) + 0.5f) * inv); };      // exact: p < 6400
    float4 v[U];
    auto load = [&](int p0) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int p = p0 + u * kTernThreads;
            if (p < items) {
                const int ol = row_of(p);
                v[u] = reinterpret_cast<const float4*>(base + ol * pitch)[p - ol * seg4];
            }
        }
    };
    load(tid);
    const float delta = delta_from_partials(ws->p1, nb1, f, static_cast<int64_t>(rows) * C * RS, scratch);
    double acc = 0.0;
    uint32_t count = 0;
    for (int p0 = tid;;) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int p = p0 + u * kTernThreads;
            if (p < items) {
                const float w4[4] = {v[u].x, v[u].y, v[u].z, v[u].w};
                uint32_t four = 0;
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const bool on = fabsf(w4[e]) > delta;
                    acc += static_cast<double>(on ? fabsf(w4[e]) : 0.0f);
                    count += on ? 1u : 0u;
                    four |= (on ? (__float_as_uint(w4[e]) >> 31) << 1 | 1u : 0u) << (8 * e);
                }
                reinterpret_cast<uint32_t*>(codes)[p] = four;
            }
        }
        p0 += U * kTernThreads;
        if (p0 - tid >= items) break;
        load(p0);
    }
    __syncthreads();
    // normal copy: word (ol, rs, g) holds channels c0 + 16g .. +15 of tap rs
    const int groups = CT / 16, normal = kTileRows * RS * groups;
    const float invg = 1.0f / static_cast<float>(groups), invrs = 1.0f / static_cast<float>(RS);
    for (int wi = tid; wi < normal; wi += kTernThreads) {
        const int t1 = static_cast<int>((static_cast<float>(wi) + 0.5f) * invg), g = wi - t1 * groups;
        const int ol = static_cast<int>((static_cast<float>(t1) + 0.5f) * invrs), rs = t1 - ol * RS;
        const unsigned char* src = codes + ol * seg + (16 * g) * RS + rs;
        uint32_t word = 0;
        if (RS == 1) {
            const uint4 q = *reinterpret_cast<const uint4*>(src);
            const uint32_t d[4] = {q.x, q.y, q.z, q.w};
            word = word_of_bytes(d);
        } else {
#pragma unroll
            for (int t = 0; t < 16; ++t) word |= static_cast<uint32_t>(src[t * RS]) << ((t & 1) * 16 + (t >> 1) * 2);
        }
        packed[static_cast<int64_t>(o0 + ol) * wpr + (rs * C + c0) / 16 + g] = word;
    }
    if (c0 == 0) {
        const int kw = RS * C / 16, pad = wpr - kw;
        for (int wi = tid; wi < kTileRows * pad; wi += kTernThreads)
            packed[static_cast<int64_t>(o0 + wi / pad) * wpr + kw + wi % pad] = 0u;
    }
    if (packed_T) {
        // transposed copy: word (cl, rs) holds filters o0 .. o0+15; four consecutive (cl, rs) per thread
        for (int it = tid; it < seg4; it += kTernThreads) {
            uint32_t word[4] = {0u, 0u, 0u, 0u};
#pragma unroll
            for (int t = 0; t < kTileRows; ++t) {
                const uint32_t b = reinterpret_cast<const uint32_t*>(codes)[t * seg4 + it];
#pragma unroll
                for (int e = 0; e < 4; ++e) word[e] |= ((b >> (8 * e)) & 3u) << ((t & 1) * 16 + (t >> 1) * 2);
            }
            int cl = static_cast<int>((static_cast<float>(4 * it) + 0.5f) * invrs), rs = 4 * it - cl * RS;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                packed_T[static_cast<int64_t>(c0 + cl) * wprT + (static_cast<int64_t>(rs) * rows + o0) / 16] = word[e];
                const bool next = ++rs == RS;
                rs = next ? 0 : rs;
                cl += next ? 1 : 0;
            }
        }
        if (o0 == 0) {
            const int kw = static_cast<int>(static_cast<int64_t>(RS) * rows / 16), pad = wprT - kw;
            for (int wi = tid; wi < CT * pad; wi += kTernThreads)
                packed_T[static_cast<int64_t>(c0 + wi / pad) * wprT + kw + wi % pad] = 0u;
        }
    }
    const double total = block_sum(acc, scratch);
    const unsigned long long ctotal = block_sum(static_cast<unsigned long long>(count), scratch_u);
    deliver(ws, bid, tiles, total, ctotal, delta, delta_out, alpha_out, nnz_out, scratch, scratch_u);
}

__global__ __launch_bounds__(kTernThreads) void mask_pack_tile_kernel(
    const float* __restrict__ W, int rows, int C, int RS, TernWorkspace* __restrict__ ws, int nb1, float f,
    uint32_t* __restrict__ packed, int wpr, uint32_t* __restrict__ packed_T, int wprT, float* __restrict__ delta_out,
    float* __restrict__ alpha_out, uint64_t* __restrict__ nnz_out) {
    mask_pack_tile_body(W, rows, C, RS, ws, nb1, f, packed, wpr, packed_T, wprT, blockIdx.x, delta_out, alpha_out, nnz_out);
}

// ---- several tensors per launch --------------------------------------------------------------
// The weight tensors of a network are small (at most a few MB): ternarizing them one call at a time is
// bound by launch latency and by kernels too small to fill the chip.  The batch entry point runs the same
// passes once for up to kBatchMax tensors; a block finds its tensor in a table passed by value.
constexpr int kBatchMax = 32;
struct BatchItem {
    const float* W;
    uint32_t* packed;
    uint32_t* packed_T;
    float* delta;
    float* alpha;
    uint64_t* nnz;
    int32_t rows, C, RS, wpr, wprT;
    int32_t nb1, nb2;           // blocks of pass 1 / pass 2 working on this tensor
    int32_t tiled;              // pass 2 through the LDS-staged tile body
    int32_t flat_blocks;        // > 0: flat layout, the first flat_blocks pass-2 blocks stream W, the rest gather the transposed copy
    int32_t first1, first2;     // index of its first block in the pass-1 / pass-2 launch
    // several groups (one Delta, alpha per `rows / groups` filters): the tensor takes no part in the two per-layer
    // launches (nb1 = nb2 = 0) but in the two per-group ones
    int32_t groups;
    int32_t firstg, ngb;        // first block and blocks in the group-statistics launch,
    int32_t firstp, npb;        // in the code-packing launch after it,
    int32_t firstf, nfb;        // in the launch that does both for tensors with one group per filter
};
struct BatchTable {
    BatchItem item[kBatchMax];
    int32_t count;
    float f;
};

// The tensor whose range of blocks in a launch holds `block`: every lane tests one entry (a walk through the table costs a
// scalar-load latency per tensor).  `first` and `blocks` name the launch's members of BatchItem.
__device__ __forceinline__ int batch_find(const BatchTable& tb, int block, int32_t BatchItem::*first, int32_t BatchItem::*blocks) {
    const int lane = threadIdx.x & (kWave - 1);
    bool hit = false;
    if (lane < tb.count) {
        const int local = block - tb.item[lane].*first;
        hit = local >= 0 && local < tb.item[lane].*blocks;
    }
    return __builtin_amdgcn_readfirstlane(static_cast<int>(__ffsll(__ballot(hit))) - 1);
}

__global__ __launch_bounds__(kTernThreads) void batch_abs_sum_kernel(const BatchTable tb, TernWorkspace* __restrict__ ws) {
    const int i = batch_find(tb, blockIdx.x, &BatchItem::first1, &BatchItem::nb1);
    const BatchItem& it = tb.item[i];
    abs_sum_body(it.W, static_cast<int64_t>(it.rows) * it.C * it.RS, ws[i].p1, blockIdx.x - it.first1, it.nb1);
}

template <bool PACED>
__global__ __launch_bounds__(kTernThreads) void batch_mask_pack_kernel(const BatchTable tb, TernWorkspace* __restrict__ ws) {
    const int i = batch_find(tb, blockIdx.x, &BatchItem::first2, &BatchItem::nb2);
    const BatchItem& it = tb.item[i];
    const int local = static_cast<int>(blockIdx.x) - it.first2;
    if (it.tiled)
        mask_pack_tile_body(it.W, it.rows, it.C, it.RS, ws + i, it.nb1, tb.f, it.packed, it.wpr, it.packed_T, it.wprT, local, it.delta,
                            it.alpha, it.nnz);
    else if (local < it.flat_blocks)
        mask_pack_flat_body(it.W, static_cast<int64_t>(it.rows) * it.C, ws + i, it.nb1, tb.f, it.packed, 1, local, it.flat_blocks,
                            it.nb2, it.delta, it.alpha, it.nnz);
    else
        mask_pack_gather_body<PACED>(it.W, it.rows, it.C, it.RS, ws + i, it.nb1, tb.f, it.packed, it.wpr, it.packed_T, it.wprT,
                              local - it.flat_blocks, it.nb2 - it.flat_blocks, it.nb2, it.delta, it.alpha, it.nnz, it.flat_blocks > 0,
                              it.flat_blocks);
}

// One block per group: both passes over the group's contiguous weights.
__device__ __forceinline__ void group_stats_body(const float* __restrict__ W, int64_t n_per_group, float f,
                                                 float* __restrict__ delta, float* __restrict__ alpha,
                                                 uint64_t* __restrict__ nnz, int group) {
    __shared__ double scratch[16];
    __shared__ unsigned long long scratch_u[16];
    const float* seg = W + static_cast<int64_t>(group) * n_per_group;
    double acc = 0.0;
    for (int64_t i = threadIdx.x; i < n_per_group; i += blockDim.x) acc += static_cast<double>(fabsf(seg[i]));
    const double s1 = block_sum(acc, scratch);
    const float d = static_cast<float>((static_cast<double>(f) * s1) / static_cast<double>(n_per_group));
    acc = 0.0;
    uint32_t count = 0;
    for (int64_t i = threadIdx.x; i < n_per_group; i += blockDim.x) {
        const float a = fabsf(seg[i]);
        if (a > d) {
            acc += static_cast<double>(a);
            ++count;
        }
    }
    const double s = block_sum(acc, scratch);
    const unsigned long long total = block_sum(static_cast<unsigned long long>(count), scratch_u);
    if (threadIdx.x == 0) {
        delta[group] = d;
        nnz[group] = total;
        alpha[group] = total ? static_cast<float>(s / static_cast<double>(total)) : 0.0f;
    }
}

__global__ __launch_bounds__(kTernThreads) void group_stats_kernel(
    const float* __restrict__ W, int64_t n_per_group, float f,
    float* __restrict__ delta, float* __restrict__ alpha, uint64_t* __restrict__ nnz) {
    group_stats_body(W, n_per_group, f, delta, alpha, nnz, blockIdx.x);
}

__global__ __launch_bounds__(kTernThreads) void batch_group_stats_kernel(const BatchTable tb) {
    const int i = batch_find(tb, blockIdx.x, &BatchItem::firstg, &BatchItem::ngb);
    const BatchItem& it = tb.item[i];
    group_stats_body(it.W, static_cast<int64_t>(it.rows) * it.C * it.RS / it.groups, tb.f, it.delta, it.alpha, it.nnz,
                     blockIdx.x - it.firstg);
}

// One Delta and alpha per filter, statistics and codes in one launch: a workgroup owns 16 filters, one per wave.  A wave sums
// its filter, which gives Delta, reads it again (from L2: at most 36 KB per wave) for the masked sum, the count and the
// codes, which go to LDS as bytes in the order of W; the words of both copies are then assembled from LDS: a word of the
// normal copy is 16 bytes of one filter, one of the transposed copy the same byte of 16 filters.  Bound by vector
// instructions (about 15 per weight) and by the latency of the reads.  Against one workgroup per filter
// for the statistics and a gathering pass per word (us): ResNet-18, 4800 filters, both copies 91 -> 30; VGG-7 89 -> 35;
// one tensor 8192 x 8192 375 -> 138.
constexpr int kFilterRows = 16;
constexpr int kFilterThreads = kFilterRows * kWave;
constexpr int kFilterMaxK = 9216;                      // 16 x 9216 bytes of LDS
__host__ __device__ inline int filter_pitch(int K) { return (K + 15) / 16 * 16; }
// Rows of taps that no multiple of 16 filters divides make the transposed words straddle workgroups.  A few long filters
// are better shared out over a workgroup each (33 x 7001: 16.2 us as three launches, 18.0 as one).
__host__ inline bool filter_ok(int rows, int64_t K, int RS, bool transposed) {
    return K <= (rows >= 512 ? kFilterMaxK : 4608) && (!transposed || RS == 1 || rows % kFilterRows == 0);
}

__device__ __forceinline__ void filter_pack_body(const float* __restrict__ W, int rows, int C, int RS, float f,
                                                 uint32_t* __restrict__ packed, int wpr, uint32_t* __restrict__ packed_T,
                                                 int wprT, float* __restrict__ delta, float* __restrict__ alpha,
                                                 uint64_t* __restrict__ nnz, int bid, unsigned char* codes) {
    constexpr int U = 6;                            // loads in flight per wave and pass
    const int K = C * RS, pitch = filter_pitch(K);
    const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid / kWave;
    const int o0 = bid * kFilterRows, o = o0 + wave;
    unsigned char* mine = codes + wave * pitch;     // [channel][tap], the order of W
    if (o < rows) {
        const float* seg = W + static_cast<int64_t>(o) * K;
        const Weights4* seg4 = reinterpret_cast<const Weights4*>(seg);
        const int n4 = K / 4;
        double acc = 0.0;
        for (int i = lane; i < n4; i += U * kWave) {
            Weights4 v[U];
#pragma unroll
            for (int u = 0; u < U; ++u)
                if (i + u * kWave < n4) v[u] = seg4[i + u * kWave];
#pragma unroll
            for (int u = 0; u < U; ++u)
                if (i + u * kWave < n4)
#pragma unroll
                    for (int e = 0; e < 4; ++e) acc += static_cast<double>(fabsf(v[u].w[e]));
        }
        if (4 * n4 + lane < K) acc += static_cast<double>(fabsf(seg[4 * n4 + lane]));
        const float d = static_cast<float>((static_cast<double>(f) * wave_sum(acc)) / static_cast<double>(K));
        acc = 0.0;
        uint32_t count = 0;
        auto code = [&](float w) -> uint32_t {
            const bool on = fabsf(w) > d;
            acc += static_cast<double>(on ? fabsf(w) : 0.0f);
            count += on ? 1u : 0u;
            return on ? ((__float_as_uint(w) >> 31) << 1 | 1u) : 0u;
        };
        for (int i = lane; i < n4; i += U * kWave) {
            Weights4 v[U];
#pragma unroll
            for (int u = 0; u < U; ++u)
                if (i + u * kWave < n4) v[u] = seg4[i + u * kWave];
#pragma unroll
            for (int u = 0; u < U; ++u)
                if (i + u * kWave < n4)
                    reinterpret_cast<uint32_t*>(mine)[i + u * kWave] =
                        code(v[u].w[0]) | (code(v[u].w[1]) << 8) | (code(v[u].w[2]) << 16) | (code(v[u].w[3]) << 24);
        }
        if (4 * n4 + lane < K) mine[4 * n4 + lane] = static_cast<unsigned char>(code(seg[4 * n4 + lane]));
        if (K + lane < pitch) mine[K + lane] = 0;
        const double s = wave_sum(acc);
        const unsigned long long total = wave_sum(static_cast<unsigned long long>(count));
        if (lane == 0) {
            delta[o] = d;
            nnz[o] = total;
            alpha[o] = total ? static_cast<float>(s / static_cast<double>(total)) : 0.0f;
        }
        // the normal copy needs nothing of the other waves
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        uint32_t* out = packed + static_cast<int64_t>(o) * wpr;
        if (RS == 1) {
            for (int j = lane; j < wpr; j += kWave) {
                uint32_t word = 0;
                if (16 * j < pitch) {
                    const uint4 b = reinterpret_cast<const uint4*>(mine)[j];
                    const uint32_t q[4] = {b.x, b.y, b.z, b.w};
                    word = word_of_bytes(q);
                }
                out[j] = word;
            }
        } else {
            const float inv = 1.0f / static_cast<float>(C);
            for (int j = lane; j < wpr; j += kWave) {
                uint32_t word = 0;
                if (16 * j < K) {
                    int rs = static_cast<int>((static_cast<float>(16 * j) + 0.5f) * inv);      // exact: below 2^14
                    int c = 16 * j - rs * C;
                    if ((C & 15) == 0) {
                        const unsigned char* src = mine + c * RS + rs;
#pragma unroll
                        for (int t = 0; t < 16; ++t) word |= static_cast<uint32_t>(src[t * RS]) << ((t & 1) * 16 + (t >> 1) * 2);
                    } else {
#pragma unroll
                        for (int t = 0; t < 16; ++t) {
                            if (rs < RS) word |= static_cast<uint32_t>(mine[c * RS + rs]) << ((t & 1) * 16 + (t >> 1) * 2);
                            const bool next = ++c == C;
                            c = next ? 0 : c;
                            rs += next ? 1 : 0;
                        }
                    }
                }
                out[j] = word;
            }
        }
    } else if (packed_T) {
        for (int m = lane; m < pitch / 4; m += kWave) reinterpret_cast<uint32_t*>(mine)[m] = 0u;      // no filter: zero codes
    }
    if (!packed_T) return;
    __syncthreads();
    // transposed copy: word (c, rs) holds filters o0 .. o0+15; four consecutive (c, rs) per thread
    const float inv = 1.0f / static_cast<float>(RS);
    for (int it = tid; 4 * it < K; it += kFilterThreads) {
        uint32_t word[4] = {0u, 0u, 0u, 0u};
#pragma unroll
        for (int t = 0; t < kFilterRows; ++t) {
            const uint32_t b = *reinterpret_cast<const uint32_t*>(codes + t * pitch + 4 * it);
#pragma unroll
            for (int e = 0; e < 4; ++e) word[e] |= ((b >> (8 * e)) & 3u) << ((t & 1) * 16 + (t >> 1) * 2);
        }
        int c = static_cast<int>((static_cast<float>(4 * it) + 0.5f) * inv);
        int rs = 4 * it - c * RS;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            if (c < C) packed_T[static_cast<int64_t>(c) * wprT + (static_cast<int64_t>(rs) * rows + o0) / 16] = word[e];
            const bool next = ++rs == RS;
            rs = next ? 0 : rs;
            c += next ? 1 : 0;
        }
    }
    if (bid == 0) {
        const int kw = static_cast<int>((static_cast<int64_t>(RS) * rows + 15) / 16), pad = wprT - kw;
        for (int wi = tid; wi < C * pad; wi += kFilterThreads)
            packed_T[static_cast<int64_t>(wi / pad) * wprT + kw + wi % pad] = 0u;
    }
}

__global__ __launch_bounds__(kFilterThreads) void filter_pack_kernel(
    const float* __restrict__ W, int rows, int C, int RS, float f, uint32_t* __restrict__ packed, int wpr,
    uint32_t* __restrict__ packed_T, int wprT, float* __restrict__ delta, float* __restrict__ alpha, uint64_t* __restrict__ nnz) {
    extern __shared__ __attribute__((aligned(16))) unsigned char filter_codes[];
    filter_pack_body(W, rows, C, RS, f, packed, wpr, packed_T, wprT, delta, alpha, nnz, blockIdx.x, filter_codes);
}

__global__ __launch_bounds__(kFilterThreads) void batch_filter_pack_kernel(const BatchTable tb) {
    extern __shared__ __attribute__((aligned(16))) unsigned char filter_codes[];
    const int i = batch_find(tb, blockIdx.x, &BatchItem::firstf, &BatchItem::nfb);
    const BatchItem& it = tb.item[i];
    filter_pack_body(it.W, it.rows, it.C, it.RS, tb.f, it.packed, it.wpr, it.packed_T, it.wprT, it.delta, it.alpha, it.nnz,
                     blockIdx.x - it.firstf, filter_codes);
}

// ---- sign binarization of the binary-weight comparison (Sec. 3) ------------------------------------------
// alpha of one group per block (float64 sum in a fixed order); used for several groups, where a group is small.
__global__ __launch_bounds__(kTernThreads) void group_abs_mean_kernel(const float* __restrict__ W, int64_t n_per_group,
                                                                      float* __restrict__ alpha) {
    __shared__ double scratch[16];
    const float* seg = W + static_cast<int64_t>(blockIdx.x) * n_per_group;
    double acc = 0.0;
    for (int64_t i = threadIdx.x; i < n_per_group; i += blockDim.x) acc += static_cast<double>(fabsf(seg[i]));
    const double s1 = block_sum(acc, scratch);
    if (threadIdx.x == 0) alpha[blockIdx.x] = static_cast<float>(s1 / static_cast<double>(n_per_group));
}

// alpha of a whole tensor from the pass-1 partial sums of abs_sum_kernel (one block).
__global__ __launch_bounds__(kTernThreads) void abs_mean_finalize_kernel(const double* __restrict__ p1, int nb1, int64_t n,
                                                                         float* __restrict__ alpha) {
    __shared__ double scratch[16];
    double acc = 0.0;
    for (int i = threadIdx.x; i < nb1; i += blockDim.x) acc += p1[i];
    const double s1 = block_sum(acc, scratch);
    if (threadIdx.x == 0) alpha[0] = static_cast<float>(s1 / static_cast<double>(n));
}

// 1-bit sign codes of a matrix whose rows need no padding (K % 128 == 0): a wave takes 64 consecutive weights
// per step, lane l reading the weight whose code lands in bit l of the two output words (even k first, then
// odd k, per word), so that the wave's ballot is the pair of words.
__global__ __launch_bounds__(256) void sign_pack_flat_kernel(const float* __restrict__ W, int64_t npairs,
                                                             uint64_t* __restrict__ out) {
    const int lane = threadIdx.x & 63;
    const int64_t wave = (static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x) >> 6;
    const int64_t nwaves = (static_cast<int64_t>(gridDim.x) * blockDim.x) >> 6;
    const int l = lane & 31;
    const int koff = (lane >> 5) * 32 + (l < 16 ? 2 * l : 2 * (l - 16) + 1);
    for (int64_t p = wave; p < npairs; p += nwaves) {
        const unsigned long long m = __ballot(W[p * 64 + koff] < 0.0f);
        if (lane == 0) out[p] = m;
    }
}

// 1-bit sign codes, one thread per output word (32 weights): k = (r*S+s)*C + c of filter `row`.
__global__ __launch_bounds__(256) void sign_pack_kernel(const float* __restrict__ W, int rows, int C, int RS,
                                                        uint32_t* __restrict__ out, int wpr) {
    const int64_t id = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
    if (id >= static_cast<int64_t>(rows) * wpr) return;
    const int row = static_cast<int>(id / wpr), j = static_cast<int>(id % wpr);
    const int64_t K = static_cast<int64_t>(RS) * C;
    uint32_t word = 0;
#pragma unroll 8
    for (int t = 0; t < 32; ++t) {
        const int64_t k = static_cast<int64_t>(j) * 32 + t;
        if (k < K) {
            const int rs = static_cast<int>(k / C);
            const int c = static_cast<int>(k - static_cast<int64_t>(rs) * C);
            const float w = W[(static_cast<int64_t>(row) * C + c) * RS + rs];
            word |= (w < 0.0f ? 1u : 0u) << ((t & 1) * 16 + (t >> 1));
        }
    }
    out[id] = word;
}

// Codes for any layout.  One thread per output word.
//   normal:     out row = filter o,        k   = (r*S+s)*C + c
//   transposed: out row = input channel c, k_T = (r*S+s)*rows + o
// Threads are ordered so that neighbouring threads read neighbouring source
// weights where the layout allows it.
__device__ __forceinline__ void pack_gather_body(
    const float* __restrict__ W, int rows, int C, int RS, const float* __restrict__ delta,
    int rows_per_group, uint32_t* __restrict__ out, int wpr, int transposed, int64_t id) {
    const int64_t words = static_cast<int64_t>(transposed ? C : rows) * wpr;
    if (id >= words) return;
    const bool narrow = words < (1LL << 31);
    float w[16];
    uint32_t word = 0;
    if (transposed) {
        const int64_t j = word_quotient(id, C, narrow);         // input channel, fastest across threads
        const int c = static_cast<int>(id - j * C);
        const uint32_t real = gather_word<true, false>(W, rows, C, RS, c, static_cast<int>(j), w);
        // group of the word's first filter, and the filter's place in it
        const uint32_t per_group = static_cast<uint32_t>(rows_per_group), filters = static_cast<uint32_t>(rows);
        const uint32_t o0 = static_cast<uint32_t>(j) * 16u % filters;
        uint32_t g = o0 / per_group, r = o0 - g * per_group, left = filters - o0;
        float d[16];
#pragma unroll
        for (int t = 0; t < 16; ++t) {
            d[t] = delta[g];
            const bool wrap = --left == 0u, next = ++r == per_group;
            r = wrap || next ? 0u : r;
            g = wrap ? 0u : g + (next ? 1u : 0u);
            left = wrap ? filters : left;
        }
#pragma unroll
        for (int t = 0; t < 16; ++t)
            word |= (static_cast<uint32_t>(t) < real ? code_field(w[t], d[t]) : 0u) << ((t & 1) * 16 + (t >> 1) * 2);
        out[static_cast<int64_t>(c) * wpr + j] = word;
        return;
    }
    const int64_t o = word_quotient(id, wpr, narrow);
    const uint32_t real = gather_word<false, false>(W, rows, C, RS, static_cast<int>(o), static_cast<int>(id - o * wpr), w);
    const float d = delta[static_cast<int>(o) / rows_per_group];
#pragma unroll
    for (int t = 0; t < 16; ++t) word |= (static_cast<uint32_t>(t) < real ? code_field(w[t], d) : 0u) << ((t & 1) * 16 + (t >> 1) * 2);
    out[id] = word;
}

__global__ __launch_bounds__(256) void pack_gather_kernel(
    const float* __restrict__ W, int rows, int C, int RS, const float* __restrict__ delta,
    int rows_per_group, uint32_t* __restrict__ out, int wpr, int transposed) {
    pack_gather_body(W, rows, C, RS, delta, rows_per_group, out, wpr, transposed,
                     static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x);
}

// Per-group tensors of a multi-tensor call: the words of the normal copy, then those of the transposed copy.
__global__ __launch_bounds__(256) void batch_pack_gather_kernel(const BatchTable tb) {
    const int i = batch_find(tb, blockIdx.x, &BatchItem::firstp, &BatchItem::npb);
    const BatchItem& it = tb.item[i];
    const int64_t id = static_cast<int64_t>(blockIdx.x - it.firstp) * blockDim.x + threadIdx.x;
    const int64_t words_n = static_cast<int64_t>(it.rows) * it.wpr;
    const int rpg = it.rows / it.groups;
    if (id < words_n)
        pack_gather_body(it.W, it.rows, it.C, it.RS, it.delta, rpg, it.packed, it.wpr, 0, id);
    else if (it.packed_T)
        pack_gather_body(it.W, it.rows, it.C, it.RS, it.delta, rpg, it.packed_T, it.wprT, 1, id - words_n);
}

__global__ __launch_bounds__(256) void unpack_i8_kernel(const uint32_t* __restrict__ packed, int rows,
                                                        int64_t K, int wpr, int8_t* __restrict__ codes) {
    const int64_t id = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
    if (id >= static_cast<int64_t>(rows) * K) return;
    const int64_t row = id / K, k = id % K;
    const uint32_t word = packed[row * wpr + (k >> 4)];
    const int t = static_cast<int>(k & 15);
    const uint32_t fld = (word >> ((t & 1) * 16 + (t >> 1) * 2)) & 3u;
    codes[id] = (fld & 1u) ? ((fld & 2u) ? -1 : 1) : 0;
}

}  // namespace twn

using namespace twn;

extern "C" size_t twn_ternarize_workspace_bytes(const twn_weight_desc* wd, int32_t groups) {
    if (!wd || groups < 1) return 0;
    const int64_t K = static_cast<int64_t>(wd->R) * wd->S * wd->C, n = K * wd->rows;
    // more than the least the call takes: without the room for marks a large flat tensor is read twice
    if (groups == 1 && wd->R == 1 && wd->S == 1 && K % 128 == 0 && n >= kBandMinWeights) return band_bytes(n);
    return sizeof(TernWorkspace);
}

// Host-side argument checks shared by twn_ternarize and twn_ternarize_static (no GPU call).
static int32_t ternarize_check(const float* W, const twn_weight_desc* wd, int32_t groups, float delta_factor,
                               const uint32_t* packed, const uint32_t* packed_T, const float* delta,
                               const float* alpha, const uint64_t* nnz) {
    if (!W || !wd || !packed || !delta || !alpha || !nnz) return TWN_ERR_NULL;
    if (wd->rows <= 0 || wd->C <= 0 || wd->R <= 0 || wd->S <= 0) return TWN_ERR_SHAPE;
    if (groups < 1 || wd->rows % groups != 0) return TWN_ERR_SHAPE;
    if (!(delta_factor > 0.0f) || delta_factor > 1.0f) return TWN_ERR_SHAPE;
    const int64_t RS = static_cast<int64_t>(wd->R) * wd->S;
    const int64_t K = RS * wd->C;
    const int64_t KT = RS * wd->rows;
    const int64_t n = K * wd->rows;
    if (RS > (1 << 15) || K >= (1LL << 31) || KT >= (1LL << 31) || n >= (1LL << 40)) return TWN_ERR_SHAPE;
    if (!aligned(W, 16) || !aligned(packed, 16) || (packed_T && !aligned(packed_T, 16))) return TWN_ERR_ALIGN;
    return TWN_OK;
}

// Blocks of pass 1 for a tensor of n weights (two persistent blocks per CU measured best with the prefetch);
// the parameter update that leaves pass-1 sums behind uses the same partition.
static int pass1_blocks(int64_t n) {
    const int64_t nchunks = (n + kChunk - 1) / kChunk;
    int want = env_int(Env::TERN_BLOCKS, 512);
    if (want < 1) want = 1;
    if (want > kMaxPass1) want = kMaxPass1;
    return static_cast<int>(nchunks < want ? nchunks : want);
}

// LDS of a workgroup.  Long filters in more workgroups than CUs run one workgroup per CU (more than half of the 160 KB):
// two at once would share a CU from the start while others finish early (ResNet-18's 21 tensors 34 -> 30 us).
static int filter_lds(int K, int64_t blocks) {
    const int need = kFilterRows * filter_pitch(K);
    return K > 2048 && blocks > 256 && need < 84 * 1024 ? 84 * 1024 : need;
}

// The dynamic-LDS limit of the per-filter kernels is raised once.
static bool filter_lds_allowed() {
    static std::once_flag once;
    static bool allowed = false;
    std::call_once(once, [] {
        const int bytes = kFilterRows * kFilterMaxK;
        allowed = hipFuncSetAttribute(reinterpret_cast<const void*>(filter_pack_kernel),
                                      hipFuncAttributeMaxDynamicSharedMemorySize, bytes) == hipSuccess &&
                  hipFuncSetAttribute(reinterpret_cast<const void*>(batch_filter_pack_kernel),
                                      hipFuncAttributeMaxDynamicSharedMemorySize, bytes) == hipSuccess;
    });
    return allowed;
}

// Launches of one ternarization; `workspace` is device memory of at least sizeof(TernWorkspace) bytes, either
// the caller's (twn_ternarize) or the library's own per-device array (twn_ternarize_static).
static int32_t ternarize_impl(const float* W, const twn_weight_desc* wd, int32_t groups,
                              float delta_factor, uint32_t* packed, uint32_t* packed_T,
                              float* delta, float* alpha, uint64_t* nnz,
                              void* workspace, size_t workspace_bytes, void* stream, bool presummed = false) {
    const int32_t rc = ternarize_check(W, wd, groups, delta_factor, packed, packed_T, delta, alpha, nnz);
    if (rc != TWN_OK) return rc;
    if (presummed && groups != 1) return TWN_ERR_UNSUPPORTED;
    const int64_t RS = static_cast<int64_t>(wd->R) * wd->S;
    const int64_t K = RS * wd->C;
    const int64_t KT = RS * wd->rows;
    const int64_t n = K * wd->rows;
    if (!workspace || workspace_bytes < sizeof(TernWorkspace) || !aligned(workspace, 8)) return TWN_ERR_WORKSPACE;

    hipStream_t st = as_stream(stream);
    const int wpr = static_cast<int>(twn_packed_words_per_row(K));
    const int wprT = static_cast<int>(twn_packed_words_per_row(KT));
    const int rows_per_group = wd->rows / groups;

    if (groups == 1) {
        TernWorkspace* ws = static_cast<TernWorkspace*>(workspace);
        const int nb = pass1_blocks(n);
        // matrices stream through the flat kernel; when the transposed copy is wanted too, the tile kernel
        // writes both from one read of W instead of a second, gathering pass
        const bool flat = (RS == 1) && (K % 128 == 0) && !(packed_T && tile_ok(wd->rows, wd->C, 1));
        // (TWN_TERN_REVERSE asks for the second pass by name)
        const bool band = flat && !presummed && n >= kBandMinWeights && workspace_bytes >= band_bytes(n) &&
                          !env_set(Env::TERN_REVERSE);
        if (!presummed && !band) abs_sum_kernel<<<nb, kTernThreads, 0, st>>>(W, n, ws->p1);
        if (flat) {
            if (band) {
                BandState* state = reinterpret_cast<BandState*>(ws + 1);
                uint64_t* marks = reinterpret_cast<uint64_t*>(reinterpret_cast<unsigned char*>(state) +
                                                              round_up(sizeof(BandState), 256));
                const int segments = static_cast<int>(band_sample(n) / kBandSegment);
                band_sample_kernel<<<kBandParts, kTernThreads, 0, st>>>(W, n, segments, state);
                band_pack_kernel<<<nb, kTernThreads, 0, st>>>(W, n, segments, delta_factor, ws, state, marks, packed);
                const int blocks = nb > kFixBlocks ? nb : kFixBlocks;
                const int64_t per = ((n + kChunk - 1) / kChunk * 4 + blocks * 4 - 1) / (blocks * 4);
                band_fix_kernel<<<blocks, kTernThreads, 0, st>>>(W, n, nb, static_cast<int>(per < kWave ? per : kWave), delta_factor,
                                                                 ws, state, marks, packed, delta, alpha, nnz);
            } else {
                const int reverse = env_int(Env::TERN_REVERSE, 1);
                mask_pack_flat_kernel<<<nb, kTernThreads, 0, st>>>(W, n, ws, nb, delta_factor, packed, reverse, delta, alpha, nnz);
            }
            if (packed_T) {
                const int64_t words = static_cast<int64_t>(wd->C) * wprT;
                pack_gather_kernel<<<static_cast<unsigned>((words + 255) / 256), 256, 0, st>>>(
                    W, wd->rows, wd->C, static_cast<int>(RS), delta, rows_per_group, packed_T, wprT, 1);
            }
        } else {
            const int64_t words = static_cast<int64_t>(wd->rows) * wpr +
                                  (packed_T ? static_cast<int64_t>(wd->C) * wprT : 0);
            int64_t nb2 = (words + kTernThreads - 1) / kTernThreads;
            if (nb2 > kMaxBlocks) nb2 = kMaxBlocks;
            if (tile_ok(wd->rows, wd->C, static_cast<int>(RS))) {
                nb2 = static_cast<int64_t>(wd->rows / kTileRows) * (wd->C / tile_ct(wd->C, static_cast<int>(RS)));
                mask_pack_tile_kernel<<<static_cast<unsigned>(nb2), kTernThreads, 0, st>>>(
                    W, wd->rows, wd->C, static_cast<int>(RS), ws, nb, delta_factor, packed, wpr, packed_T, wprT, delta, alpha, nnz);
            } else
                (paced_words(n, static_cast<int>(RS)) ? mask_pack_gather_kernel<true> : mask_pack_gather_kernel<false>)<<<
                    static_cast<unsigned>(nb2), kTernThreads, 0, st>>>(
                    W, wd->rows, wd->C, static_cast<int>(RS), ws, nb, delta_factor, packed, wpr, packed_T, wprT, delta, alpha, nnz);
        }
    } else if (groups == wd->rows && filter_ok(wd->rows, K, static_cast<int>(RS), packed_T != nullptr)) {
        if (!filter_lds_allowed()) return TWN_ERR_HIP;
        filter_pack_kernel<<<static_cast<unsigned>((wd->rows + kFilterRows - 1) / kFilterRows), kFilterThreads,
                             filter_lds(static_cast<int>(K), (wd->rows + kFilterRows - 1) / kFilterRows), st>>>(
            W, wd->rows, wd->C, static_cast<int>(RS), delta_factor, packed, wpr, packed_T, wprT, delta, alpha, nnz);
    } else {
        group_stats_kernel<<<groups, kTernThreads, 0, st>>>(W, n / groups, delta_factor, delta, alpha, nnz);
        const int64_t words = static_cast<int64_t>(wd->rows) * wpr;
        pack_gather_kernel<<<static_cast<unsigned>((words + 255) / 256), 256, 0, st>>>(
            W, wd->rows, wd->C, static_cast<int>(RS), delta, rows_per_group, packed, wpr, 0);
        if (packed_T) {
            const int64_t wordsT = static_cast<int64_t>(wd->C) * wprT;
            pack_gather_kernel<<<static_cast<unsigned>((wordsT + 255) / 256), 256, 0, st>>>(
                W, wd->rows, wd->C, static_cast<int>(RS), delta, rows_per_group, packed_T, wprT, 1);
        }
    }
    return launch_status();
}

extern "C" int32_t twn_ternarize(const float* W, const twn_weight_desc* wd, int32_t groups,
                                 float delta_factor, uint32_t* packed, uint32_t* packed_T,
                                 float* delta, float* alpha, uint64_t* nnz,
                                 void* workspace, size_t workspace_bytes, void* stream) {
    return ternarize_impl(W, wd, groups, delta_factor, packed, packed_T, delta, alpha, nnz, workspace, workspace_bytes,
                          stream);
}

// ---- parameter update fused with pass 1 of the next ternarization (Alg. 1 step 10; Sec. 2.4; Table 1) --------
// One read of W, V, dW and one write of W, V per weight (20 bytes); the float64 sum of |W| after the update is
// accumulated chunk by chunk and element by element exactly as abs_sum_body does it, so that the partial sums
// (and with them Delta of the ternarization that follows) are bit-identical to a separate pass over the updated
// tensor, which would cost 4 more bytes per weight.
__global__ __launch_bounds__(kTernThreads) void sgd_update_kernel(float* __restrict__ W, float* __restrict__ V,
                                                                  const float* __restrict__ dW, int64_t n, float lr,
                                                                  float momentum, float wd, double* __restrict__ partial) {
    __shared__ double scratch[16];
    const int tid = threadIdx.x;
    const int bid = blockIdx.x, nblk = gridDim.x;
    const int64_t nfull = n / kChunk;
    double acc = 0.0;
    auto load4 = [&](const float* p, int64_t c, float4* v) {
        const float4* src = reinterpret_cast<const float4*>(p + c * kChunk);
#pragma unroll
        for (int j = 0; j < 4; ++j) v[j] = src[j * kTernThreads + tid];
    };
    auto update = [&](float& w, float& v, float g) {
        g = fmaf(wd, w, g);
        v = fmaf(momentum, v, g);
        w = fmaf(-lr, v, w);
        acc += static_cast<double>(fabsf(w));
    };
    int64_t c = bid;
    float4 w4[4], v4[4], g4[4];
    if (c < nfull) {
        load4(W, c, w4);
        load4(V, c, v4);
        load4(dW, c, g4);
    }
    while (c < nfull) {
        const int64_t nx = c + nblk;
        float4 wn[4], vn[4], gn[4];
        if (nx < nfull) {
            load4(W, nx, wn);
            load4(V, nx, vn);
            load4(dW, nx, gn);
        }
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            update(w4[j].x, v4[j].x, g4[j].x);
            update(w4[j].y, v4[j].y, g4[j].y);
            update(w4[j].z, v4[j].z, g4[j].z);
            update(w4[j].w, v4[j].w, g4[j].w);
        }
        float4* wdst = reinterpret_cast<float4*>(W + c * kChunk);
        float4* vdst = reinterpret_cast<float4*>(V + c * kChunk);
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            wdst[j * kTernThreads + tid] = w4[j];
            vdst[j * kTernThreads + tid] = v4[j];
        }
        if (nx < nfull) {
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                w4[j] = wn[j];
                v4[j] = vn[j];
                g4[j] = gn[j];
            }
        }
        c = nx;
    }
    // ragged tail (at most one chunk), taken by the block abs_sum_body gives it to, in its element order
    if (nfull * kChunk < n && bid == tail_block(nfull, nblk)) {
        const int64_t base = nfull * kChunk;
        load_tail(W, base, n, w4);
        load_tail(V, base, n, v4);
        load_tail(dW, base, n, g4);
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int64_t idx = base + static_cast<int64_t>(j * kTernThreads + tid) * 4;
            if (idx + 3 < n) {
                update(w4[j].x, v4[j].x, g4[j].x);
                update(w4[j].y, v4[j].y, g4[j].y);
                update(w4[j].z, v4[j].z, g4[j].z);
                update(w4[j].w, v4[j].w, g4[j].w);
                *reinterpret_cast<float4*>(W + idx) = w4[j];
                *reinterpret_cast<float4*>(V + idx) = v4[j];
            }
        }
        if (owns_last(n))
            for (int64_t idx = n & ~static_cast<int64_t>(3); idx < n; ++idx) {
                float w = W[idx], v = V[idx];
                update(w, v, dW[idx]);
                W[idx] = w;
                V[idx] = v;
            }
    }
    const double total = block_sum(acc, scratch);
    if (partial && tid == 0) partial[bid] = total;
    if (partial && bid == 0 && tid < kTickets) partial[kMaxPass1 + tid * kTicketStep] = 0.0;       // as pass 1 leaves them
}

extern "C" int32_t twn_sgd_update(float* W, float* V, const float* dW, int64_t n, float lr, float momentum,
                                  float weight_decay, void* tern_workspace, size_t workspace_bytes, void* stream) {
    if (!W || !V || !dW) return TWN_ERR_NULL;
    if (n <= 0 || n >= (1LL << 40)) return TWN_ERR_SHAPE;
    if (!(lr == lr) || !(momentum == momentum) || !(weight_decay == weight_decay)) return TWN_ERR_SHAPE;
    if (!aligned(W, 16) || !aligned(V, 16) || !aligned(dW, 16)) return TWN_ERR_ALIGN;
    if (tern_workspace && (workspace_bytes < sizeof(TernWorkspace) || !aligned(tern_workspace, 8))) return TWN_ERR_WORKSPACE;
    TernWorkspace* ws = static_cast<TernWorkspace*>(tern_workspace);
    sgd_update_kernel<<<pass1_blocks(n), kTernThreads, 0, as_stream(stream)>>>(W, V, dW, n, lr, momentum, weight_decay,
                                                                              ws ? ws->p1 : nullptr);
    return launch_status();
}

extern "C" int32_t twn_ternarize_presummed(const float* W, const twn_weight_desc* wd, float delta_factor,
                                           uint32_t* packed, uint32_t* packed_T, float* delta, float* alpha,
                                           uint64_t* nnz, void* workspace, size_t workspace_bytes, void* stream) {
    return ternarize_impl(W, wd, 1, delta_factor, packed, packed_T, delta, alpha, nnz, workspace, workspace_bytes, stream,
                          true);
}

extern "C" size_t twn_binarize_workspace_bytes(const twn_weight_desc* wd, int32_t groups) {
    (void)groups;
    if (!wd) return 0;
    return sizeof(TernWorkspace);
}

extern "C" int32_t twn_binarize(const float* W, const twn_weight_desc* wd, int32_t groups, uint32_t* packed1,
                                float* alpha, void* workspace, size_t workspace_bytes, void* stream) {
    if (!W || !wd || !packed1 || !alpha) return TWN_ERR_NULL;
    if (wd->rows <= 0 || wd->C <= 0 || wd->R <= 0 || wd->S <= 0) return TWN_ERR_SHAPE;
    if (groups < 1 || wd->rows % groups != 0) return TWN_ERR_SHAPE;
    const int64_t RS = static_cast<int64_t>(wd->R) * wd->S;
    const int64_t K = RS * wd->C;
    const int64_t n = K * wd->rows;
    if (RS > (1 << 15) || K >= (1LL << 31) || n >= (1LL << 40)) return TWN_ERR_SHAPE;
    if (!aligned(W, 16) || !aligned(packed1, 16)) return TWN_ERR_ALIGN;
    if (!workspace || workspace_bytes < sizeof(TernWorkspace) || !aligned(workspace, 8)) return TWN_ERR_WORKSPACE;
    hipStream_t st = as_stream(stream);
    if (groups == 1) {
        TernWorkspace* ws = static_cast<TernWorkspace*>(workspace);
        const int nb = pass1_blocks(n);
        abs_sum_kernel<<<nb, kTernThreads, 0, st>>>(W, n, ws->p1);
        abs_mean_finalize_kernel<<<1, kTernThreads, 0, st>>>(ws->p1, nb, n, alpha);
    } else {
        group_abs_mean_kernel<<<groups, kTernThreads, 0, st>>>(W, n / groups, alpha);
    }
    const int wpr = static_cast<int>(twn_packed1_words_per_row(K));
    const int64_t words = static_cast<int64_t>(wd->rows) * wpr;
    if (RS == 1 && K % 128 == 0) {
        const int64_t npairs = n / 64;
        const int64_t blocks = (npairs + 3) / 4 < 4096 ? (npairs + 3) / 4 : 4096;
        sign_pack_flat_kernel<<<static_cast<unsigned>(blocks), 256, 0, st>>>(W, npairs, reinterpret_cast<uint64_t*>(packed1));
    } else {
        sign_pack_kernel<<<static_cast<unsigned>((words + 255) / 256), 256, 0, st>>>(W, wd->rows, wd->C,
                                                                                      static_cast<int>(RS), packed1, wpr);
    }
    return launch_status();
}

// ---- the entry point that allocates nothing -------------------------------------------------------------
// The per-block partial sums of twn_ternarize live in a file-scope device array instead of a caller
// workspace.  Every GPU the library runs on holds its own copy of the array at its own address: the
// address is looked up once per device (with that device current) and only that pointer is ever handed
// to kernels.  Nothing in the array has to start at zero: every partial a pass reads was written by the
// pass before it in the same call.
namespace twn {
constexpr int kStaticMaxDevices = 64;
static __device__ __align__(256) unsigned char scratch[sizeof(TernWorkspace)];
static std::mutex g_scratch_mutex;
static void* g_scratch_ptr[kStaticMaxDevices];      // per device: address of `scratch` there, null until looked up
}  // namespace twn

extern "C" size_t twn_ternarize_static_scratch_bytes(void) { return sizeof(TernWorkspace); }

extern "C" int32_t twn_ternarize_static(const float* W, const twn_weight_desc* wd, int32_t groups,
                                        float delta_factor, uint32_t* packed, uint32_t* packed_T,
                                        float* delta, float* alpha, uint64_t* nnz, void* stream) {
    // every check that needs no GPU comes first; tensors beyond the 2^40 weights the fixed array is specified
    // for are rejected here with TWN_ERR_SHAPE
    const int32_t rc = ternarize_check(W, wd, groups, delta_factor, packed, packed_T, delta, alpha, nnz);
    if (rc != TWN_OK) return rc;
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess) return TWN_ERR_HIP;
    if (dev < 0 || dev >= kStaticMaxDevices) return TWN_ERR_UNSUPPORTED;
    void* ptr = nullptr;
    {
        std::lock_guard<std::mutex> lock(g_scratch_mutex);
        if (!g_scratch_ptr[dev]) {
            void* p = nullptr;
            if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || !p) return TWN_ERR_HIP;
            g_scratch_ptr[dev] = p;
        }
        ptr = g_scratch_ptr[dev];
    }
    return ternarize_impl(W, wd, groups, delta_factor, packed, packed_T, delta, alpha, nnz, ptr, sizeof(TernWorkspace),
                          stream);
}

extern "C" size_t twn_ternarize_batch_workspace_bytes(int32_t count) {
    if (count < 1 || count > kBatchMax) return 0;
    return static_cast<size_t>(count) * sizeof(TernWorkspace);
}

extern "C" int32_t twn_ternarize_batch(const twn_ternarize_item* items, int32_t count, float delta_factor,
                                       void* workspace, size_t workspace_bytes, void* stream) {
    if (!items) return TWN_ERR_NULL;
    if (count < 1 || count > kBatchMax) return TWN_ERR_SHAPE;
    if (!(delta_factor > 0.0f) || delta_factor > 1.0f) return TWN_ERR_SHAPE;
    if (!workspace || workspace_bytes < static_cast<size_t>(count) * sizeof(TernWorkspace) || !aligned(workspace, 8))
        return TWN_ERR_WORKSPACE;
    BatchTable tb{};
    tb.count = count;
    tb.f = delta_factor;
    int64_t total_n = 0;
    for (int i = 0; i < count; ++i) {
        const twn_ternarize_item& in = items[i];
        if (!in.W || !in.packed || !in.delta || !in.alpha || !in.nnz) return TWN_ERR_NULL;
        const twn_weight_desc& wd = in.wd;
        if (wd.rows <= 0 || wd.C <= 0 || wd.R <= 0 || wd.S <= 0) return TWN_ERR_SHAPE;
        const int64_t RS = static_cast<int64_t>(wd.R) * wd.S;
        const int64_t K = RS * wd.C, KT = RS * wd.rows, n = K * wd.rows;
        if (RS > (1 << 15) || K >= (1LL << 31) || KT >= (1LL << 31) || n >= (1LL << 40)) return TWN_ERR_SHAPE;
        if (!aligned(in.W, 16) || !aligned(in.packed, 16) || (in.packed_T && !aligned(in.packed_T, 16))) return TWN_ERR_ALIGN;
        if (in.groups < 1 || wd.rows % in.groups != 0) return TWN_ERR_SHAPE;
        if (in.groups == 1) total_n += n;
    }
    if (total_n == 0) total_n = 1;      // only per-group tensors
    // blocks are shared out in proportion to the tensor sizes: about 1024 per pass in total
    int first1 = 0, first2 = 0;
    int64_t firstg = 0, firstp = 0;
    int filter_k = 0;
    for (int i = 0; i < count; ++i) {
        const twn_ternarize_item& in = items[i];
        const twn_weight_desc& wd = in.wd;
        const int64_t RS = static_cast<int64_t>(wd.R) * wd.S;
        const int64_t K = RS * wd.C, KT = RS * wd.rows, n = K * wd.rows;
        BatchItem& it = tb.item[i];
        it.W = in.W; it.packed = in.packed; it.packed_T = in.packed_T;
        it.delta = in.delta; it.alpha = in.alpha; it.nnz = in.nnz;
        it.rows = wd.rows; it.C = wd.C; it.RS = static_cast<int32_t>(RS);
        it.wpr = static_cast<int32_t>(twn_packed_words_per_row(K));
        it.wprT = static_cast<int32_t>(twn_packed_words_per_row(KT));
        it.groups = in.groups;
        it.firstg = it.firstp = it.firstf = 0;
        it.ngb = it.npb = it.nfb = 0;
        if (in.groups > 1) {
            it.nb1 = it.nb2 = it.first1 = it.first2 = 0;
            it.tiled = it.flat_blocks = 0;
            if (in.groups == wd.rows && filter_ok(wd.rows, K, static_cast<int>(RS), in.packed_T != nullptr)) {
                it.nfb = (wd.rows + kFilterRows - 1) / kFilterRows;      // placed below
                if (K > filter_k) filter_k = static_cast<int>(K);
                continue;
            }
            // one block per group for the statistics, one thread per output word for the codes
            const int64_t words = static_cast<int64_t>(wd.rows) * it.wpr + (in.packed_T ? static_cast<int64_t>(wd.C) * it.wprT : 0);
            it.firstg = static_cast<int32_t>(firstg);
            it.firstp = static_cast<int32_t>(firstp);
            it.ngb = in.groups;
            it.npb = static_cast<int32_t>((words + 255) / 256);
            firstg += it.ngb;
            firstp += it.npb;
            if (firstg >= (1LL << 30) || firstp >= (1LL << 30)) return TWN_ERR_SHAPE;
            continue;
        }
        int64_t share = (1024 * n + total_n - 1) / total_n;
        if (share < 1) share = 1;
        const int64_t nchunks = (n + kChunk - 1) / kChunk;
        it.nb1 = static_cast<int32_t>(nchunks < share ? nchunks : share);
        const int64_t words = static_cast<int64_t>(wd.rows) * it.wpr + (in.packed_T ? static_cast<int64_t>(wd.C) * it.wprT : 0);
        int64_t nb2 = (words + kTernThreads - 1) / kTernThreads;
        if (nb2 > 4 * share) nb2 = 4 * share;
        if (nb2 > kMaxBlocks) nb2 = kMaxBlocks;
        if (it.nb1 > kMaxPass1) it.nb1 = kMaxPass1;
        const bool flat = (RS == 1) && (K % 128 == 0) && !(in.packed_T && tile_ok(wd.rows, wd.C, 1));
        it.tiled = (!flat && tile_ok(wd.rows, wd.C, static_cast<int>(RS))) ? 1 : 0;
        if (it.tiled) nb2 = static_cast<int64_t>(wd.rows / kTileRows) * (wd.C / tile_ct(wd.C, static_cast<int>(RS)));
        it.flat_blocks = 0;
        if (flat) {
            // flat layout: the normal copy is written while W streams by; only the transposed copy gathers
            it.flat_blocks = it.nb1;
            int64_t nbT = in.packed_T ? (static_cast<int64_t>(wd.C) * it.wprT + kTernThreads - 1) / kTernThreads : 0;
            if (nbT > 4 * share) nbT = 4 * share;
            if (nbT > kMaxBlocks - it.flat_blocks) nbT = kMaxBlocks - it.flat_blocks;
            nb2 = it.flat_blocks + nbT;
        }
        it.nb2 = static_cast<int32_t>(nb2);
        it.first1 = first1;
        first1 += it.nb1;
    }
    // A block that takes long ends the launch late if it starts late: tiles of filters larger than 3x3 first, then untiled tensors, whose
    // gathering blocks are chains of latencies (within one that streams they follow), then tiles by the weights they hold.  us with both
    // copies, as listed / untiled tensors first / so: VGG-7, whose classifier of 10 gathers, 36.8 / 34.0 / 32.1; VGG-16 46.2 / 46.2 / 43.7;
    // 192x64x3x3, 1024x64x5x5, 64x64x5x5 and four others 21.3 / 23.5 / 21.7.
    auto order = [](const BatchItem& it) { return !it.tiled ? 1 : it.RS > 9 ? 0 : tile_ct(it.C, it.RS) * it.RS > 64 * 9 ? 2 : 3; };
    for (int turn = 0; turn < 4; ++turn)
        for (int i = 0; i < count; ++i)
            if (tb.item[i].nb2 > 0 && order(tb.item[i]) == turn) {
                tb.item[i].first2 = first2;
                first2 += tb.item[i].nb2;
            }
    // longest filters first: a long one that starts late ends the launch late
    int64_t firstf = 0;
    for (int64_t below = kFilterMaxK + 1; filter_k > 0 && below > 0;) {
        int64_t longest = 0;
        for (int i = 0; i < count; ++i) {
            const int64_t K = static_cast<int64_t>(tb.item[i].C) * tb.item[i].RS;
            if (tb.item[i].nfb > 0 && K < below && K > longest) longest = K;
        }
        for (int i = 0; i < count && longest > 0; ++i)
            if (tb.item[i].nfb > 0 && static_cast<int64_t>(tb.item[i].C) * tb.item[i].RS == longest) {
                tb.item[i].firstf = static_cast<int32_t>(firstf);
                firstf += tb.item[i].nfb;
            }
        if (firstf >= (1LL << 22)) return TWN_ERR_SHAPE;        // grid below 2^32 threads
        below = longest;
    }
    hipStream_t st = as_stream(stream);
    TernWorkspace* ws = static_cast<TernWorkspace*>(workspace);
    if (first1 > 0) {
        batch_abs_sum_kernel<<<first1, kTernThreads, 0, st>>>(tb, ws);
        // paced words: also for the smaller tensors of such a call
        bool paced = false;
        for (int i = 0; i < count; ++i) {
            const BatchItem& it = tb.item[i];
            paced = paced || (it.nb2 > 0 && !it.tiled && paced_words(static_cast<int64_t>(it.rows) * it.C * it.RS, it.RS));
        }
        (paced ? batch_mask_pack_kernel<true> : batch_mask_pack_kernel<false>)<<<first2, kTernThreads, 0, st>>>(tb, ws);
    }
    if (firstf > 0) {
        if (!filter_lds_allowed()) return TWN_ERR_HIP;
        batch_filter_pack_kernel<<<static_cast<unsigned>(firstf), kFilterThreads, filter_lds(filter_k, firstf), st>>>(tb);
    }
    if (firstg > 0) {
        batch_group_stats_kernel<<<static_cast<unsigned>(firstg), kTernThreads, 0, st>>>(tb);
        batch_pack_gather_kernel<<<static_cast<unsigned>(firstp), 256, 0, st>>>(tb);
    }
    return launch_status();
}

extern "C" int32_t twn_unpack_i8(const uint32_t* packed, int32_t rows, int64_t K, int8_t* codes, void* stream) {
    if (!packed || !codes) return TWN_ERR_NULL;
    if (rows <= 0 || K <= 0 || K >= (1LL << 31)) return TWN_ERR_SHAPE;
    if (!aligned(packed, 16)) return TWN_ERR_ALIGN;
    const int64_t total = static_cast<int64_t>(rows) * K;
    unpack_i8_kernel<<<static_cast<unsigned>((total + 255) / 256), 256, 0, as_stream(stream)>>>(
        packed, rows, K, static_cast<int>(twn_packed_words_per_row(K)), codes);
    return launch_status();
}
