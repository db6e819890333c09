// Flat passes cover every node once and the dense local pass's walks every plane
// once, and both stay in the grid, also where it has nearly 2^31 nodes.
#include <cstdio>
#include <initializer_list>

#include "../../paper_2106_15869_amd/csrc/eik_walk.hpp"

using namespace eik;

static int fails = 0;

static void covers(int64_t plane, int64_t outer) {
    const int steps = walk_steps(plane * outer, plane);
    const int64_t walks = walk_count(outer, steps);
    int64_t planes = 0;
    bool in = walk_lanes(plane, outer, steps) <= plane * outer;
    for (int64_t k = 0; k < walks; ++k) {
        const Walk w = walk_of(static_cast<uint32_t>(k), static_cast<uint32_t>(outer), steps);
        in &= w.begin == planes && w.begin < w.end && w.end <= outer;
        planes += w.end - w.begin;
    }
    // the last lane is the last node of the last walk
    const int64_t last = walk_lanes(plane, outer, steps) - 1;
    in &= last / plane == walks - 1 && last % plane == plane - 1;
    if (!in || planes != outer) {
        std::printf("plane %lld outer %lld: in %d planes %lld\n", (long long)plane, (long long)outer, in,
                    (long long)planes);
        ++fails;
    }
}

static void flat(int64_t n) {
    const int64_t lanes = flat_step(flat_blocks(n));
    int64_t nodes = 0;
    bool in = true;
    // a lane's nodes are its number and what follows at the step; the lanes
    // differ only in how many there are
    for (int64_t lane : {int64_t(0), (n - 1) % lanes, lanes - 1}) {
        int64_t c = 0;
        for (int64_t i = lane; i < n; i += lanes) in &= i >= 0 && ++c > 0;
        in &= c == (lane < n ? (n - 1 - lane) / lanes + 1 : 0);
        nodes += c;
    }
    if (!in || nodes == 0) std::printf("flat %lld\n", (long long)n), ++fails;
}

int main() {
    const int64_t top = (int64_t(1) << 31) - 1;
    for (int64_t outer : {top, top - 1})
        covers(1, outer);
    for (int64_t plane : {1, 2, 16, 33, 255, 257, 4096})
        for (int64_t outer : {1, 2, 15, 16, 17, 1000, 65535, 65536, 65537}) covers(plane, outer);
    for (int64_t n : {int64_t(1), int64_t(255), int64_t(257), int64_t(1) << 28, (int64_t(1) << 28) + 1, top, top - 300})
        flat(n);
    covers(2, top / 2);
    covers(top, 1);
    std::printf(fails ? "failed\n" : "clean\n");
    return fails != 0;
}
