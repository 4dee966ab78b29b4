// A number per call by which its split partials are marked as written: no
// other call holds it and no leftover memory does.
#pragma once

#include <stdint.h>
#include <sys/random.h>
#include <time.h>
#include <unistd.h>

#include <atomic>

namespace sangam {

// Where a process starts: the kernel's entropy, else its id and the time.
// (std::random_device throws where it finds no source.)
inline uint64_t nonce_seed() noexcept {
    uint64_t x = 0;
    if (getentropy(&x, sizeof x) == 0) return x;
    timespec t{};
    clock_gettime(CLOCK_REALTIME, &t);
    return (uint64_t(getpid()) << 40) ^ (uint64_t(t.tv_sec) * 1000000000u + uint64_t(t.tv_nsec));
}

// A mixed counter; never 0.
inline uint64_t next_nonce() noexcept {
    static const uint64_t seed = nonce_seed();
    static std::atomic<uint64_t> calls{0};
    for (;;) {
        uint64_t x = seed + calls.fetch_add(1, std::memory_order_relaxed) * 0x9E3779B97F4A7C15ull;
        x = (x ^ (x >> 30)) * 0xBF58476D1CE4E5B9ull;  // splitmix64 (Steele, Lea, Flood, 2014), a bijection
        x = (x ^ (x >> 27)) * 0x94D049BB133111EBull;
        x ^= x >> 31;
        if (x) return x;
    }
}

}  // namespace sangam
