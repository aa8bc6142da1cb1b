// The tags of launches that merge their pieces themselves.  Plain host code, no HIP.
#pragma once

#include <atomic>
#include <chrono>
#include <cstdint>
#include <random>

namespace cusa {

// Where a process's tags start: 64 random bits, mixed with the clock.  Called under the C interface, which no exception may leave: where the
// machine has no random numbers to give, the clock and an address (both through SplitMix64's finalizer; Steele, Lea and Flood, OOPSLA 2014) have to do.
template <typename Source>
uint64_t tag_start() noexcept {
    static const char here = 0;
    uint64_t x = (uint64_t)std::chrono::steady_clock::now().time_since_epoch().count() ^ (uint64_t)std::chrono::system_clock::now().time_since_epoch().count() << 20 ^
                 (uint64_t)(uintptr_t)&here;
    x = (x ^ x >> 30) * 0xBF58476D1CE4E5B9ull;
    x = (x ^ x >> 27) * 0x94D049BB133111EBull;
    x ^= x >> 31;
    try {
        Source source;
        x ^= (uint64_t)source() << 32 | source();
    } catch (...) {
    }
    return x;
}

// A tag that no other call of this or an earlier process is likely to have had: steps by an odd constant, which come back to a
// value after 2^64 of them.  (0 means no tag.)
inline uint64_t new_tag() noexcept {
    static std::atomic<uint64_t> state{tag_start<std::random_device>()};
    const uint64_t t = state.fetch_add(0x9E3779B97F4A7C15ull, std::memory_order_relaxed);
    return t ? t : 1;
}

}  // namespace cusa
