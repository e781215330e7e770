// Shared device/host helpers for the gfx950 kernels of the TWN hot path.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <atomic>

#include "twn.h"

namespace twn {

constexpr int kWave = 64;

inline hipStream_t as_stream(void* s) { return reinterpret_cast<hipStream_t>(s); }

inline int32_t launch_status() {
    return hipGetLastError() == hipSuccess ? TWN_OK : TWN_ERR_HIP;
}

inline bool aligned(const void* p, size_t a) { return (reinterpret_cast<uintptr_t>(p) & (a - 1)) == 0; }

inline size_t round_up(size_t v, size_t a) { return (v + a - 1) / a * a; }

// 64-wide slabs of a reduction of length k.  The sum is unsigned: two terms of alpha*dY double a K that may be just below
// 2^30, and k + 63 would pass the largest int.
__host__ __device__ inline int k_slabs(int32_t k) { return static_cast<int>((static_cast<uint32_t>(k) + 63u) >> 6); }

// Environment overrides for launch-shape sweeps, TWN_<name> (unset = built-in choice).  One value per name: a workspace
// query and the launch after it ask at different places and have to agree.  It is stamped with the generation that
// twn_reload_env advances: a dispatch asks for up to ten of them, and a locked search by name cost it about a microsecond.
#define TWN_ENV_NAMES(X) \
    X(BUFLOAD) X(C64) X(C64_OCC) X(DX_CLASSES) X(DX_CLASS_BATCH) X(DX_CLASS_MIN_PIXELS) X(F32_SPLITK) X(FIRST) \
    X(FIRST_OCC) X(FIRST_STAGGER) X(FIRST_THROUGH) X(FWD_PAIR) X(SMALL) X(STREAM) X(STREAM_KS) X(STREAM_OCC) \
    X(STREAM_PC) X(STREAM_PC_STAGES) X(TERN_BLOCKS) X(TERN_REVERSE) X(TILE) X(WG_BLOCKS) X(WG_KS) \
    X(WG_ROWS_SPLITS) X(WG_TAPS) X(WG_XCD)
enum class Env : int {
#define TWN_ENV_ENUM(n) n,
    TWN_ENV_NAMES(TWN_ENV_ENUM)
#undef TWN_ENV_ENUM
    kCount
};
extern std::atomic<uint64_t> g_env[static_cast<int>(Env::kCount)];      // generation << 33 | is set << 32 | value
extern std::atomic<uint32_t> g_env_generation;      // starts at 1
uint64_t env_read(Env name, uint32_t generation);
inline uint64_t env_value(Env name) {
    const uint32_t gen = g_env_generation.load(std::memory_order_relaxed);
    const uint64_t v = g_env[static_cast<int>(name)].load(std::memory_order_relaxed);
    return (v >> 33) == gen ? v : env_read(name, gen);
}
inline bool env_set(Env name) { return (env_value(name) >> 32) & 1u; }
inline int env_int(Env name, int fallback) {
    const uint64_t v = env_value(name);
    return ((v >> 32) & 1u) ? static_cast<int>(static_cast<uint32_t>(v)) : fallback;
}

// ---- wave / block reductions in a fixed order (bit-identical run to run) ----
__device__ __forceinline__ double wave_sum(double v) {
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, kWave);
    return v;
}

__device__ __forceinline__ unsigned long long wave_sum(unsigned long long v) {
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, kWave);
    return v;
}

// Block-wide sum for blocks of up to 16 waves; every thread gets the result.
// `scratch` must hold 16 values and is reusable after the call returns.
template <typename T>
__device__ __forceinline__ T block_sum(T v, T* scratch) {
    const int lane = threadIdx.x & (kWave - 1);
    const int wave = threadIdx.x / kWave;
    const int nwaves = (blockDim.x + kWave - 1) / kWave;
    v = wave_sum(v);
    __syncthreads();
    if (lane == 0) scratch[wave] = v;
    __syncthreads();
    T total = scratch[0];
    for (int w = 1; w < nwaves; ++w) total += scratch[w];
    return total;
}

// float -> bf16 bits, round to nearest even (finite inputs).
__device__ __forceinline__ uint16_t f32_to_bf16(float f) {
    uint32_t u = __float_as_uint(f);
    u += 0x7FFFu + ((u >> 16) & 1u);
    return static_cast<uint16_t>(u >> 16);
}

// Two floats -> two bf16 in one register (low half = a), round to nearest even: one v_cvt_pk_bf16_f32.
__device__ __forceinline__ uint32_t pack_bf16x2(float a, float b) {
    typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
    typedef float f32x2_t __attribute__((ext_vector_type(2)));
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(f32x2_t{a, b}, bf16x2_t));
}

__device__ __forceinline__ float bf16_to_f32(uint16_t b) {
    return __uint_as_float(static_cast<uint32_t>(b) << 16);
}

// A float as three bf16 terms whose sum is the float: 3 x 8 significant bits, each term takes what the ones before leave.
constexpr int kAlphaTerms = 3;
__device__ __forceinline__ void alpha_terms(float v, uint16_t* t) {
#pragma unroll
    for (int k = 0; k < kAlphaTerms; ++k) {
        t[k] = f32_to_bf16(v);
        v -= bf16_to_f32(t[k]);
    }
}

// Two bf16 values times two float32 factors, each product as two bf16 terms: hi = bf16(v), lo = bf16(v - hi).
struct Bf16Terms {
    uint32_t hi, lo;
};
__device__ __forceinline__ Bf16Terms split_scaled_bf16x2(uint32_t x, float a0, float a1) {
    const float v0 = __uint_as_float(x << 16) * a0, v1 = __uint_as_float(x & 0xFFFF0000u) * a1;
    const uint32_t hi = pack_bf16x2(v0, v1);
    return Bf16Terms{hi, pack_bf16x2(v0 - __uint_as_float(hi << 16), v1 - __uint_as_float(hi & 0xFFFF0000u))};
}

// 2-bit field of the packed format: bit0 = non-zero, bit1 = negative.
__device__ __forceinline__ uint32_t code_field(float w, float delta) {
    const uint32_t nz = fabsf(w) > delta ? 1u : 0u;
    const uint32_t neg = (w < 0.0f) ? nz : 0u;
    return nz | (neg << 1);
}

}  // namespace twn
