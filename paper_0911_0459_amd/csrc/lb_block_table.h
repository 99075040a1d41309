// Tile table of the multi-step block kernels: the output nodes and the region of
// each workgroup.  Host code only, so that it also builds without HIP.
#pragma once
#include <algorithm>
#include <array>
#include <cstdint>
#include <vector>

#include "lbcap.h"

namespace lbk {

// Output nodes [xs, xe) x [ya, yb) of capillary cap; the workgroup's region
// starts at row yr and at column xs - 2 K.
struct BlockDev {
    int cap;
    int xs, xe;
    int ya, yb;
    int yr;
};

// Tiles for regions of rx x ry nodes advanced K steps per launch (rx, ry > 4 K);
// returns their number and lists them if out is given.  A step reaches two nodes,
// so a tile needs 2 K nodes around it, taken periodically; tiles lie in the tube's
// channel or in the reservoir, never in both.  Where every column a tile can read
// lies in the tube, the region ends one wall row outside the channel: nothing
// behind the wall can reach the tile, so a channel that fits the region between
// its walls needs no halo rows at all.  Tiles are of balanced height, and of
// balanced width or, with align > 1, cut at multiples of align columns.  Listed
// column by column, so that neighbouring tiles are close in the table.
inline size_t build_blocks(const std::vector<lb_geometry>& G, const std::vector<int>& active, int K, int rx, int ry,
                           int align, std::vector<BlockDev>* out) {
    const int halo = 2 * K, wmax = rx - 2 * halo, hmax = ry - 2 * halo;
    size_t count = 0;
    if (out) out->clear();
    for (size_t k = 0; k < G.size(); ++k) {
        if (!active[k]) continue;
        const lb_geometry& g = G[k];
        const bool tube = g.tube_len > 0;
        const int x0 = tube ? g.x_in : g.nx, x1 = tube ? g.x_in + g.tube_len : g.nx;
        // n tiles over the H rows from y0; the first and the last one `extra` rows
        // taller than an equal share
        auto column = [&](int xs, int xe, int y0, int H, int n, int extra, bool walled) {
            count += n;
            if (!out) return;
            const long long inner = H - 2 * extra;
            int ya = y0;
            for (int j = 0; j < n; ++j) {
                const int yb = j == n - 1 ? y0 + H : y0 + extra + (int)(inner * (j + 1) / n);
                out->push_back(BlockDev{(int)k, xs, xe, ya, yb, walled && j == 0 ? ya - 1 : ya - halo});
                ya = yb;
            }
        };
        auto section = [&](int c0, int c1, bool in_tube) {
            const int w = c1 - c0, n = (w + wmax - 1) / wmax;
            for (int i = 0, xs = c0, xe; xs < c1; ++i, xs = xe) {
                xe = align > 1 ? std::min(c1, (xs + wmax) / align * align) : c0 + (int)((long long)w * (i + 1) / n);
                const int H = g.tube_h;
                if (!in_tube) {
                    column(xs, xe, 0, g.ny, (g.ny + hmax - 1) / hmax, 0, false);
                } else if (g.tube_len < g.nx && (xs - halo < g.x_in || xe + halo > x1)) {
                    column(xs, xe, g.y0, H, (H + hmax - 1) / hmax, 0, false);
                } else {
                    // rows a tile can hold next to one wall: hmax and what the missing halo leaves
                    const int extra = halo - 1, one = hmax + extra;
                    if (H <= ry - 2)
                        column(xs, xe, g.y0, H, 1, 0, true);
                    else if (H <= 2 * one)
                        column(xs, xe, g.y0, H, 2, 0, true);
                    else
                        column(xs, xe, g.y0, H, 2 + (H - 2 * one + hmax - 1) / hmax, extra, true);
                }
            }
        };
        section(0, x0, false);
        section(x0, x1, true);
        section(x1, g.nx, false);
    }
    return count;
}

// How a context's lattices are cut: a shape (0: 32 x 32 nodes, one node per
// thread; 1: 64 columns, two nodes per thread, 24 rows for the binary model, 32
// for van der Waals: what two workgroups per CU leave in LDS; 2: 32 x 24 nodes) and K.
struct BlockPlan {
    int shape, K;
    size_t tiles;
};

constexpr int BLOCK_SHAPES = 3;
inline int block_rx(int shape) { return shape == 1 ? 64 : 32; }
inline int block_ry(int shape, bool vdw) { return shape == 2 || (shape == 1 && !vdw) ? 24 : 32; }
// Columns the tiles are cut at.  A lattice beyond the caches is bound by the lines
// its tiles share: whole 64-byte sectors measured 71.9 against 74.0 us per step
// (vdW 16384 x 1024, K = 4).  The binary tiles (52 columns at K = 3, 56 at K = 2) would
// lose more columns, down to 48, than that gains (the 256-capillary sweep: 422 against
// 374 us).
inline int block_align(int shape, bool vdw) { return shape == 1 && vdw ? 16 : 1; }

// What a launch of shape `shape` costs at K steps, kmin <= K <= kmax (see plan_block_tiles).
struct BlockCost {
    int shape, kmin, kmax;
    double launch, launch_k, tile, tile_k;
};
constexpr BlockCost BLOCK_COST_BINARY[BLOCK_SHAPES] = {
    {0, 2, 6, 2.8, 1.64, 2.57, 0.44}, {1, 2, 3, 4.4, 2.07, 3.95, 0.46}, {2, 2, 5, 2.5, 1.47, 2.02, 0.30}};
constexpr BlockCost BLOCK_COST_VDW[BLOCK_SHAPES] = {
    {0, 2, 6, 2.84, 1.10, 2.85, 0.06}, {1, 2, 4, 3.64, 1.83, 4.79, 0.23}, {2, 2, 5, 2.66, 0.99, 2.09, 0.05}};
inline const BlockCost* block_costs(bool vdw) { return vdw ? BLOCK_COST_VDW : BLOCK_COST_BINARY; }

// Every plan has a place: shape i at K steps is place 6 i + K - kmin.
constexpr int BLOCK_PLANS = 6 * BLOCK_SHAPES;
using BlockCounts = std::array<unsigned, BLOCK_PLANS>;

// Tiles that each plan cuts a lattice into.
inline BlockCounts count_blocks(const lb_geometry& g, bool vdw) {
    BlockCounts n{};
    for (int i = 0; i < BLOCK_SHAPES; ++i) {
        const BlockCost& c = block_costs(vdw)[i];
        for (int K = c.kmin; K <= c.kmax; ++K)
            n[6 * i + K - c.kmin] = (unsigned)build_blocks({g}, {1}, K, block_rx(c.shape), block_ry(c.shape, vdw),
                                                           block_align(c.shape, vdw), nullptr);
    }
    return n;
}

// The cheapest plan.  A launch costs its own latency, which grows with K, and so much
// for every further tile of a CU: whole rounds of 256 tiles up to the second (the 5 x
// 512 x 64 batch of the binary model: 250 tiles at K = 3 3.05 us a step, 290 at K = 4
// 3.63), a continuous flow of tiles beyond.  The coefficients are fits (us) to
// lattices of 5e3 to 7e6 nodes; they hold to 6 - 8 % (rms), and the plan they choose
// was the best of the 11 or 12 measured ones on 27 of 30 lattices (2 %, 7 % and 15 %
// off on the others).  The 24-row shape has fewer wavefronts to take through each step
// while CUs are idle (binary 131 x 41 1.97 us a step against 2.08, 256 x 64 1.97
// against 2.06); a small K when halos cost throughput (binary 4096 x 256: 8.2 us at
// K = 2, 10.6 at K = 4), the large shape, with fewer halo nodes, from about a million
// nodes (binary 8192 x 1024: 79 against 102 us).
//
// counts: count_blocks of each capillary, kept by the caller, who plans again whenever
// one retires (counting all plans of 256 capillaries takes the host 1 to 3 ms, summing them 1 us).
// Plans of more than `most` tiles are left out.
inline BlockPlan plan_block_tiles(const std::vector<BlockCounts>& counts, const std::vector<int>& active, bool vdw,
                                  size_t most = SIZE_MAX) {
    std::array<size_t, BLOCK_PLANS> total{};
    for (size_t k = 0; k < counts.size(); ++k)
        for (int i = 0; i < BLOCK_PLANS && active[k]; ++i) total[i] += counts[k][i];
    BlockPlan best{0, 0, 0};
    double cheapest = 0.0;
    for (int i = 0; i < BLOCK_SHAPES; ++i) {
        const BlockCost& c = block_costs(vdw)[i];
        for (int K = c.kmin; K <= c.kmax; ++K) {
            const size_t n = total[6 * i + K - c.kmin];
            if (n > most) continue;
            const double over = n <= 512 ? (n > 256 ? 1.0 : 0.0) : n / 256.0 - 0.5;
            const double us = (c.launch + c.launch_k * K + (c.tile + c.tile_k * K) * over) / K;
            if (best.K == 0 || us < cheapest) {
                best = BlockPlan{c.shape, K, n};
                cheapest = us;
            }
        }
    }
    return best;
}

// Tiles that a context reserves room for: those of the plan for all its capillaries,
// which also fits whatever set of them is active, and the finest plan up to 65,536.
// (The finest plan of a large context would take 0.5 bytes a node, and is no plan for
// one: over random parts of 256 and 1024 capillaries of the sweep no plan is left out
// that would have been taken.)
inline size_t block_capacity(const std::vector<BlockCounts>& counts, bool vdw) {
    size_t finest = 0;
    for (const BlockCounts& n : counts) finest += *std::max_element(n.begin(), n.end());
    const std::vector<int> all(counts.size(), 1);
    return std::max(plan_block_tiles(counts, all, vdw).tiles, std::min<size_t>(finest, 65536));
}

inline BlockPlan plan_block_tiles(const std::vector<lb_geometry>& G, const std::vector<int>& active, bool vdw) {
    std::vector<BlockCounts> counts;
    for (const lb_geometry& g : G) counts.push_back(count_blocks(g, vdw));
    return plan_block_tiles(counts, active, vdw);
}

}  // namespace lbk
