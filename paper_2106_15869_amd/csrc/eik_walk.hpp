// How dense kernels cover a grid.
//
// Flat passes: node i and then every flat_step(blocks)-th one, in 64 bits: the
// step past the last of nearly 2^31 nodes comes out negative in 32.
//
// The local pass: walks of `steps` planes along the outer axis, walk k starting
// at plane k * steps; lane l takes node l % plane of walk l / plane.  Plane
// numbers are unsigned: the end of a walk may lie past 2^31.  (constexpr: host
// and device.)
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
    uint32_t begin, end;  // planes
};

constexpr int64_t walk_count(int64_t outer, int steps) { return (outer + steps - 1) / steps; }

constexpr Walk walk_of(uint32_t k, uint32_t outer, int steps) {
    const uint32_t begin = k * static_cast<uint32_t>(steps), end = begin + static_cast<uint32_t>(steps);
    return Walk{begin, end < outer ? end : outer};
}

// Planes per walk: the two values at its ends are read by the next walk too, so
// long walks, but at least half a million lanes (four waves for each of the
// 1024 SIMDs twice over).  Measured at 16 M nodes, 1 / 4 / 16 planes: 10485 x 40 x
// 40 float 91, 66, 63 us, 65280 x 257 double 125, 101, 110; 200 x 333 x 250 float on
// inputs not read before 83.3 us at 8, 81.6 at 16.  With fewer than sixteen nodes
// a plane the lanes of a wave read as many lines as they walk: two planes (16 M x 1
// float 75 us at 1, 62 at 2, 136 at 8; 2 M x 8 double 109 at 1 and 2, 121 at 8).
constexpr int walk_steps(int64_t n, int64_t plane) {
    const int64_t s = n >> 19, most = plane < 16 ? 2 : 16;
    return s < 1 ? 1 : static_cast<int>(s < most ? s : most);
}

// A lane per node of a plane and walk, numbered through: the lanes of a wave may
// lie in different walks, so planes of any size fill it.  No more than the
// grid has nodes (31 bits).
constexpr int64_t walk_lanes(int64_t plane, int64_t outer, int steps) { return plane * walk_count(outer, steps); }

}  // namespace eik
