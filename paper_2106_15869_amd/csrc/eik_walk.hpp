// How dense kernels cover a grid.
//
// Flat passes: node i and then every flat_step(blocks)-th one, in 64 bits: the
// step past the last of nearly 2^31 nodes comes out negative in 32.
//
// The local pass: walks of `steps` planes along the
// outer axis, walk k starting at plane k * steps.  Plane numbers are 64-bit: an
// outer extent may lie just below 2^31, where a 32-bit step past the last walk
// comes out negative.  (constexpr: host and device.)
#pragma once

#include <stdint.h>

namespace eik {

constexpr int kFlatBlock = 256;  // lanes per workgroup

constexpr int flat_blocks(int64_t n) {
    const int64_t b = (n + kFlatBlock - 1) / kFlatBlock;
    return b < 1 ? 1 : b < (1 << 20) ? static_cast<int>(b) : 1 << 20;
}
constexpr int64_t flat_step(int64_t blocks) { return blocks * kFlatBlock; }

struct Walk {
    int64_t begin, end;  // planes
};

constexpr int64_t walk_count(int64_t outer, int steps) { return (outer + steps - 1) / steps; }

constexpr Walk walk_of(int64_t k, int64_t outer, int steps) {
    const int64_t begin = k * steps, end = begin + steps;
    return Walk{begin, end < outer ? end : outer};
}

// Planes per walk: the two values at its ends are read by the next walk too, so
// long walks, but at least half a million lanes (four waves for each of the
// 1024 SIMDs twice over).
constexpr int walk_steps(int64_t n) {
    const int64_t s = n >> 19;
    return s < 1 ? 1 : s < 16 ? static_cast<int>(s) : 16;
}

// Blocks along the walks (grid.y), each of which takes every such walk.
constexpr int walk_blocks(int64_t outer, int steps) {
    const int64_t k = walk_count(outer, steps);
    return k < 65535 ? static_cast<int>(k) : 65535;
}

}  // namespace eik
