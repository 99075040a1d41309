// Checks of the block kernels' planning on the host.
#include <cstdio>
#include <cstdlib>
#include <vector>

#include "lb_block_table.h"

using namespace lbk;

// The plan made from the counts that a context keeps is the one made by cutting the
// active lattices anew, and the table it stands for fits what the context reserves.
static int kept_counts() {
    unsigned s = 5;
    auto rnd = [&](int lo, int hi) {
        s = s * 1664525u + 1013904223u;
        return lo + (int)((s >> 8) % (unsigned)(hi - lo + 1));
    };
    for (int pass = 0; pass < 400; ++pass) {
        const bool vdw = pass % 2;
        std::vector<lb_geometry> G;
        std::vector<BlockCounts> counts;
        for (int n = rnd(1, 30); n > 0; --n) {
            lb_geometry g{rnd(3, pass % 7 ? 400 : 4000), rnd(5, 140), 0, 0, 0, 0};
            if (n % 8) {
                g.tube_len = rnd(1, g.nx);
                g.x_in = rnd(0, g.nx - g.tube_len);
                g.tube_h = rnd(3, g.ny - 2);
                g.y0 = rnd(1, g.ny - 1 - g.tube_h);
            }
            G.push_back(g);
            counts.push_back(count_blocks(g, vdw));
        }
        for (int k = 0; k < 10; ++k) {
            std::vector<int> active(G.size());
            for (int& a : active) a = rnd(0, 3) > 0;
            const size_t room = block_capacity(counts, vdw);
            const BlockPlan a = plan_block_tiles(counts, active, vdw, room), b = plan_block_tiles(G, active, vdw);
            const size_t n =
                build_blocks(G, active, a.K, block_rx(a.shape), block_ry(a.shape, vdw), block_align(a.shape, vdw), nullptr);
            if (a.shape != b.shape || a.K != b.K || a.tiles != n || n > room) {
                std::printf("plan from counts: shape %d K %d, %zu tiles, %zu cut\n", a.shape, a.K, a.tiles, n);
                return 1;
            }
        }
    }
    return 0;
}

// `model nx ny x_in tube_len tube_h y0`: the plan of that lattice and the tiles of the
// column in the middle of its tube.
static int print_plan(char** v) {
    const bool vdw = v[1][0] == 'v';
    const lb_geometry g{std::atoi(v[2]), std::atoi(v[3]), std::atoi(v[4]), std::atoi(v[5]), std::atoi(v[6]), std::atoi(v[7])};
    const BlockPlan p = plan_block_tiles(std::vector<lb_geometry>{g}, {1}, vdw);
    std::vector<BlockDev> t;
    build_blocks({g}, {1}, p.K, block_rx(p.shape), block_ry(p.shape, vdw), block_align(p.shape, vdw), &t);
    int column = 0;
    const int x = g.x_in + g.tube_len / 2;
    for (const BlockDev& b : t) column += b.xs <= x && x < b.xe;
    std::printf("%d %d %d\n", p.shape, p.K, column);
    return 0;
}

int main(int argc, char** argv) { return argc == 8 ? print_plan(argv) : kept_counts(); }
