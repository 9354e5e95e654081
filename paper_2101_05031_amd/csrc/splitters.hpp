// Which segments the chaining of contours stops at (contours.hip) whatever
// their neighbours are, and how many splitters a call can have.
#pragma once

#include <algorithm>
#include <cstdint>

namespace lsl {

constexpr uint32_t kSplit = 8;         // about one segment in this many

// Half of them by a multiple of the golden ratio: indices a constant stride
// apart, as along a wall (one segment per row), are then picked evenly for most
// strides, but hardly ever for some (near Fibonacci numbers of segments per
// row: up to every row of 2048 missed with 2584), and a walk of that length is one
// lane's serial chain of gathers.  The other half by a mixed hash, which no
// stride evades: at most 181 steps between picks over 2048 rows of any stride up
// to 2^17 (counted from one start each).  One open chain per row's place, 2048 rows, 610 and 2584 segments per
// row: 985 -> 450 us and 2591 -> 761 us; 612 and 2586, which the first rule alone
// serves well, 381 -> 389 and 678 -> 697 us (the mixed hash alone: 407 and 715).
constexpr bool split_pick(uint32_t s) {
    uint32_t h = s * 2654435761u;
    const bool even = h < 0xffffffffu / (2 * kSplit);
    h ^= h >> 16;
    h *= 2654435761u;
    h ^= h >> 13;
    h *= 2654435761u;
    return even || h < 0xffffffffu / (2 * kSplit);
}

// At most this many splitters: half of the segments are smaller than both
// neighbours, split_pick takes at most t / 8 + 4 of the first t segments for
// every t up to 2^30 (counted), and an open chain starts on a border edge.
inline uint32_t poly_splitters(uint64_t total, int32_t nk, int32_t W, int32_t H) {
    const uint64_t border = 2 * (uint64_t)nk * ((uint64_t)W + (uint64_t)H);
    return (uint32_t)std::min<uint64_t>(total,
                                        total / 2 + total / kSplit + total / 64 + 1024 + border);
}

}  // namespace lsl
