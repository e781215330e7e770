// Host-only helpers of the C ABI: status strings, packed-format sizes, env overrides.
#include <cstdlib>
#include <mutex>

#include "twn_common.h"

namespace twn {

// The TWN_* overrides are read from the environment once each and remembered: launches do not call getenv
// (which is neither free nor safe against a concurrent setenv).  twn_reload_env forgets what was read.
std::atomic<uint64_t> g_env[static_cast<int>(Env::kCount)] = {};
std::atomic<uint32_t> g_env_generation{1};

uint64_t env_read(Env name, uint32_t generation) {
#define TWN_ENV_STRING(n) "TWN_" #n,
    static const char* const names[] = {TWN_ENV_NAMES(TWN_ENV_STRING)};
#undef TWN_ENV_STRING
    static std::mutex mutex;
    std::lock_guard<std::mutex> lock(mutex);
    std::atomic<uint64_t>& kept = g_env[static_cast<int>(name)];
    uint64_t seen = kept.load(std::memory_order_relaxed);
    if ((seen >> 33) == generation) return seen;        // another thread has read it meanwhile
    const char* v = std::getenv(names[static_cast<int>(name)]);
    const bool set = v && *v;
    seen = (static_cast<uint64_t>(generation) << 33) | (static_cast<uint64_t>(set) << 32) |
           static_cast<uint32_t>(set ? std::atoi(v) : 0);
    kept.store(seen, std::memory_order_relaxed);
    return seen;
}

}  // namespace twn

extern "C" void twn_reload_env(void) {
    // a generation fits 31 bits in the stamp; 0 stands for "never read"
    uint32_t g = twn::g_env_generation.load(std::memory_order_relaxed);
    while (!twn::g_env_generation.compare_exchange_weak(g, g == 0x7FFFFFFFu ? 1u : g + 1u, std::memory_order_relaxed)) {
    }
}

extern "C" const char* twn_status_str(int32_t status) {
    switch (status) {
        case TWN_OK: return "ok";
        case TWN_ERR_NULL: return "null pointer";
        case TWN_ERR_SHAPE: return "bad shape or size";
        case TWN_ERR_ALIGN: return "misaligned pointer or leading dimension";
        case TWN_ERR_UNSUPPORTED: return "unsupported dtype, variant or option";
        case TWN_ERR_WORKSPACE: return "workspace missing or too small";
        case TWN_ERR_HIP: return "HIP launch failed";
        default: return "unknown status";
    }
}

extern "C" int32_t twn_abi_version(void) { return 2; }

extern "C" int64_t twn_packed_words_per_row(int64_t K) {
    if (K <= 0) return 0;
    return 8 * ((K + 127) / 128);
}

extern "C" int64_t twn_packed1_words_per_row(int64_t K) {
    if (K <= 0) return 0;
    return 4 * ((K + 127) / 128);
}

extern "C" size_t twn_packed_bytes(int32_t rows, int64_t K) {
    if (rows <= 0 || K <= 0) return 0;
    return static_cast<size_t>(rows) * static_cast<size_t>(twn_packed_words_per_row(K)) * 4u;
}
