// Flat passes cover every node once and the dense local pass's walks every plane
// once, and both stay in the grid, also where it has nearly 2^31 nodes.
#include <cstdio>
#include <initializer_list>

#include "../../paper_2106_15869_amd/csrc/eik_walk.hpp"

using namespace eik;

static int fails = 0;

static void covers(int64_t plane, int64_t outer) {
    const int steps = walk_steps(plane * outer);
    const int64_t walks = walk_count(outer, steps);
    const int blocks = walk_blocks(outer, steps);
    int64_t planes = 0, taken = 0;
    bool in = true;
    for (int64_t b = 0; b < blocks; ++b)
        for (int64_t k = b; k < walks; k += blocks) {
            const Walk w = walk_of(k, outer, steps);
            in &= w.begin >= 0 && w.begin < w.end && w.end <= outer && w.begin == k * steps;
            planes += w.end - w.begin;
            ++taken;
        }
    if (!in || planes != outer || taken != walks) {
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
    for (int64_t outer : {top, top - 1, top - 15, top - 16, top - 65535 * 16, top - 65535 * 16 - 1, top / 2})
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
