// Splitting a grid over launches.
#pragma once

#include <cstdint>

namespace lsl {

// A launch counts its threads in 32 bits; half of that range per launch.
constexpr uint64_t kLaunchThreads = 1ull << 31;

inline uint64_t launch_blocks(uint32_t threads) { return kLaunchThreads / threads; }

// launches that for_launches makes
inline uint64_t launch_count(uint64_t blocks, uint32_t threads) {
    return (blocks + launch_blocks(threads) - 1) / launch_blocks(threads);
}

// Calls f(first block, number of blocks) for each launch of a grid of `blocks`
// workgroups of `threads` threads.
template <typename F>
void for_launches(uint64_t blocks, uint32_t threads, F&& f) {
    const uint64_t per = launch_blocks(threads);
    for (uint64_t b = 0; b < blocks; b += per)
        f(b, (uint32_t)(blocks - b < per ? blocks - b : per));
}

}  // namespace lsl
