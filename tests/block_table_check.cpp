// Checks of the block kernels' tile table on the host: every fluid node is the
// output of exactly one tile, and every tile's region holds what its steps read.
#include <cstdio>
#include <cstdlib>
#include <vector>

#include "lb_block_table.h"

static bool solid(const lb_geometry& g, int x, int y) {
    x = ((x % g.nx) + g.nx) % g.nx;
    y = ((y % g.ny) + g.ny) % g.ny;
    return g.tube_len > 0 && x >= g.x_in && x < g.x_in + g.tube_len && (y < g.y0 || y >= g.y0 + g.tube_h);
}

static int bad(const char* what, const lb_geometry& g, int K, int rx, int ry) {
    std::printf("%s: %dx%d tube %d+%d rows %d+%d, K=%d region %dx%d\n", what, g.nx, g.ny, g.x_in, g.tube_len, g.y0,
                g.tube_h, K, rx, ry);
    return 1;
}

static int check(const lb_geometry& g, int K, int rx, int ry, int align) {
    const int halo = 2 * K;
    std::vector<lbk::BlockDev> t;
    const size_t n = lbk::build_blocks({g, g}, {0, 1}, K, rx, ry, align, &t);
    if (n != t.size() || n != lbk::build_blocks({g, g}, {0, 1}, K, rx, ry, align, nullptr))
        return bad("count differs", g, K, rx, ry);
    std::vector<int> hit((size_t)g.nx * g.ny, 0);
    for (const lbk::BlockDev& b : t) {
        if (b.cap != 1) return bad("retired capillary listed", g, K, rx, ry);
        if (b.xs < 0 || b.xe > g.nx || b.xs >= b.xe || b.ya < 0 || b.yb > g.ny || b.ya >= b.yb)
            return bad("tile out of the lattice", g, K, rx, ry);
        for (int y = b.ya; y < b.yb; ++y)
            for (int x = b.xs; x < b.xe; ++x) {
                if (solid(g, x, y)) return bad("solid output", g, K, rx, ry);
                ++hit[(size_t)y * g.nx + x];
            }
        if (b.xe + halo > b.xs - halo + rx) return bad("region too narrow", g, K, rx, ry);
        // what the tile can depend on: nodes joined to it by fluid nodes within the
        // halo; each of their rows, and the solid rows next to them, are in the region
        const int x0 = b.xs - halo, x1 = b.xe + halo, y0 = b.ya - halo, y1 = b.yb + halo, w = x1 - x0, h = y1 - y0;
        std::vector<char> seen((size_t)w * h, 0);
        std::vector<int> todo;
        for (int y = b.ya; y < b.yb; ++y)
            for (int x = b.xs; x < b.xe; ++x) {
                seen[(size_t)(y - y0) * w + x - x0] = 1;
                todo.push_back((y - y0) * w + x - x0);
            }
        while (!todo.empty()) {
            const int k = todo.back();
            todo.pop_back();
            const int x = k % w + x0, y = k / w + y0;
            if (y < b.yr || y >= b.yr + ry) return bad("region too low", g, K, rx, ry);
            if (solid(g, x, y)) continue;
            for (int dy = -1; dy <= 1; ++dy)
                for (int dx = -1; dx <= 1; ++dx) {
                    const int xx = x + dx, yy = y + dy;
                    if (xx < x0 || xx >= x1 || yy < y0 || yy >= y1 || seen[(size_t)(yy - y0) * w + xx - x0]) continue;
                    seen[(size_t)(yy - y0) * w + xx - x0] = 1;
                    todo.push_back((yy - y0) * w + xx - x0);
                }
        }
    }
    for (int y = 0; y < g.ny; ++y)
        for (int x = 0; x < g.nx; ++x)
            if (hit[(size_t)y * g.nx + x] != (solid(g, x, y) ? 0 : 1)) return bad("not covered once", g, K, rx, ry);
    return 0;
}

int main() {
    const int regions[][3] = {{32, 32, 1}, {32, 24, 1}, {64, 24, 1}, {64, 32, 16}};
    const lb_geometry fixed[] = {{256, 64, 128, 128, 20, 22}, {131, 41, 0, 131, 39, 1}, {700, 42, 175, 350, 40, 1},
                                 {1024, 128, 256, 768, 40, 44}, {5, 3, 0, 0, 0, 0}, {3, 22, 0, 3, 20, 1},
                                 {520, 41, 100, 300, 11, 15}, {300, 300, 60, 240, 298, 1}};
    int n = 0;
    unsigned s = 1;
    auto rnd = [&](int lo, int hi) {
        s = s * 1664525u + 1013904223u;
        return lo + (int)((s >> 8) % (unsigned)(hi - lo + 1));
    };
    for (const auto& r : regions)
        for (int K = 1; 4 * K < std::min(r[0], r[1]); ++K) {
            for (const lb_geometry& g : fixed) {
                if (check(g, K, r[0], r[1], r[2])) return 1;
                ++n;
            }
            for (int k = 0; k < 150; ++k) {
                lb_geometry g{rnd(3, 400), rnd(5, 140), 0, 0, 0, 0};
                if (k % 8) {
                    g.tube_len = rnd(1, g.nx);
                    g.x_in = rnd(0, g.nx - g.tube_len);
                    g.tube_h = rnd(3, g.ny - 2);
                    g.y0 = rnd(1, g.ny - 1 - g.tube_h);
                }
                if (check(g, K, r[0], r[1], r[2])) return 1;
                ++n;
            }
        }
    // small lattices take a small shape and several steps, large ones the large shape
    const lb_geometry big{3000, 700, 700, 2000, 500, 100};
    for (int vdw = 0; vdw < 2; ++vdw) {
        const lbk::BlockPlan a = lbk::plan_block_tiles({fixed[0]}, {1}, vdw), b = lbk::plan_block_tiles({big}, {1}, vdw);
        if (a.shape == 1 || a.K < 4 || b.shape != 1 || b.K < 2) return bad("plan", big, a.K, a.shape, b.shape);
        if (lbk::plan_block_tiles({big}, {0}, vdw).tiles != 0) return bad("plan of no capillary", big, 0, 0, 0);
    }
    std::printf("block table: %d cases\n", n);
    return 0;
}
