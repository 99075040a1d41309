// Multi-step block kernels of lbcap: K time steps of one tile of nodes per launch
// (schedule 4 of the van der Waals model, schedule 6 of the binary model).
//
// A workgroup owns a tile and a halo of 2 K nodes around it (a step reaches two
// nodes): it loads the region once, runs K steps with the neighbours' populations
// exchanged through LDS, each step on two nodes less all round, and stores the
// tile.
//
// The arithmetic per node and step is that of the row sweeps (the same functions
// on the same FP32 values: what a step leaves in LDS for the next one is rounded
// exactly as it would be stored), so the fields do not depend on K, on the tiling
// or on how steps are grouped into launches, and are bitwise those of lb_wide_vdw
// and lb_wmom_bin, which take the single steps of large contexts.
//
// Per step two phases, each ended by an LDS-only barrier; with m = 2 (steps left
// after this one), on nodes up to a distance from the tile:
//   pull     populations of the neighbours from LDS, moments (binary: u, the
//            stencils of phi and A)                                   up to m + 1
//   collide  (binary: and the phi update), new populations into LDS   up to m
// The pull of one step and the collide of the previous one are a barrier apart,
// so one copy of the populations is enough; phi is read in both phases and
// written in the second one, so it has two.
//
// What bounds it.  A small lattice is a chain of latencies: one node's arithmetic
// and two barriers (1.0 us a step for van der Waals, 1.5 us for the binary model)
// and a K-th of 2.6 us for the launch, the loads and the stores (the fits of
// lb_block_table.h, 24-row shape).  The row sweeps, marching a few dozen workgroups
// through their rows at about 2 us a row, left most CUs idle: vdW 256 x 64 10.1 -> 1.5
// us per step, binary 1024 x 128 46.2 -> 2.5 us, binary 4096 x 256 47.1 -> 8.4 us.  A
// large one is bound by the vector ALU, all its cycles (vdW 16384 x 1024 at K = 4: 157 M
// wavefront instructions a launch; the 256-capillary sweep at K = 3: 631 M; halo nodes
// are a third to a half of the work): the state crosses HBM once per launch instead of
// every step, and the sweep runs at 346 instead of 495 us per step.  On vdW 16384 x 1024
// K = 4 measured 68 us (K = 3: 79, K = 2: 103; two steps per row sweep, schedule 5: 96).
// Two nodes per thread in the 64-column shape: one row per wavefront (scalar row
// data, no lane masks for the rows) and both nodes' neighbours at constant distances
// from two address registers keep it to 80 (binary) and 58 registers, two workgroups
// per CU, so that one's loads and stores run under the other's arithmetic.
//
// Every wavefront of a workgroup waits for the one at the wall, so its ghosts and
// bounce-back sources are picked among values already read instead of read under a
// branch for each direction (the sweep 382 -> 345 us, binary 1024 x 128 3.3 -> 2.7 us
// at that step),
// and wavefronts without solid neighbours run code compiled for none (vdW
// 16384 x 1024 70.7 -> 68.6 us).
#pragma once
#include <algorithm>
#include <type_traits>

#include "lb_barrier.h"
#include "lb_block_table.h"
#include "lb_wmom.h"

namespace lbk {

struct BlockArgs {
    const CapDev* caps;
    const BlockDev* blocks;
    int nblocks;
    float* arena0;
    float* arena1;
    int cur;                 // capillary k reads arena (cur ^ par_k), writes the other
    int halo;                // 2 K of the table
    int steps;               // steps of this launch, at most K
};

// Region of RX x RY nodes of one workgroup: RP rows of threads, node j of a thread
// RP rows above its node j - 1.
template <int RX_, int RY_, int RP_>
struct BlockShape {
    static constexpr int RX = RX_, RY = RY_, RP = RP_;
    static constexpr int N = RX * RY;                    // nodes of the region
    static constexpr int NPT = (RY + RP - 1) / RP;       // nodes per thread
    static constexpr int NT = (RX * RP + SW - 1) / SW * SW;   // threads (whole wavefronts)
    static constexpr int WAVES = (2048 / NT) * (NT / SW) / 4 < 8 ? (2048 / NT) * (NT / SW) / 4 : 8;
    static constexpr int JS = RP * RX;                   // words from a thread's node to its next one
    static constexpr int PAD = RX + 1;                   // LDS words before the first plane (see BlockAt)
    // planes within reach of one address register: a DS instruction's constant is 16 bits
    static constexpr int REACH = std::min((65536 / 4 - 1 - PAD - (NPT - 1) * JS - PAD) / N, 8);
};

// What a thread knows of one of its nodes, fixed for the launch.
struct BlockNode {
    int voff;       // byte offset in a plane
    int dist;       // distance from the tile (Chebyshev; 0 and less inside)
    unsigned sm;    // solid-neighbour bits
    bool fluid;
    bool walls;     // some node of the wavefront has such neighbours
};

constexpr int BLOCK_NOWHERE = 1 << 20;   // distance of a node that takes no part

template <typename S>
__device__ __forceinline__ void block_nodes(const Geo& g, const BlockDev& b, const BlockArgs& a, int rb,
                                            BlockNode (&n)[S::NPT]) {
    const int rx = threadIdx.x % S::RX;
    // with 64 columns a wavefront is one row: its row data is scalar
    const int r0 = S::RX == SW ? __builtin_amdgcn_readfirstlane(threadIdx.x / S::RX) : threadIdx.x / S::RX;
    const int x = b.xs - a.halo + rx;
    // -halo <= x < nx + RX and the same for y: at most one turn of the lattice, unless
    // it is smaller than the region
    const bool small = g.nx < S::RX || g.ny < S::RY;
    const LaneCols L = lane_cols_of(g, small ? wrap_mod(x, g.nx) : (x < 0 ? x + g.nx : (x >= g.nx ? x - g.nx : x)));
    const int dx = max(b.xs - x, x - b.xe + 1);
    const bool rim = rx == 0 || rx == S::RX - 1;
#pragma unroll
    for (int j = 0; j < S::NPT; ++j) {
        const int ry = r0 + j * S::RP, y = b.yr + ry;
        const RowInfo r = row_info(g, small ? wrap_mod(y, g.ny) : y);
        n[j].voff = L.b0 + r.y0 * rb;
        n[j].dist = max(dx, max(b.ya - y, y - b.yb + 1));
        // the region's rim is only read: its neighbours are not in the region (a rim
        // row that is nearer lies behind a wall)
        if (rim || ry == 0 || ry >= S::RY - 1) n[j].dist = max(n[j].dist, 2 * a.steps);
        if (r0 >= S::RP || ry >= S::RY) n[j].dist = BLOCK_NOWHERE;
        n[j].sm = r.any ? solid_bits(L, r) : 0u;
        n[j].fluid = !(L.t0 && r.w0);
        n[j].walls = __builtin_amdgcn_ballot_w64(n[j].sm != 0u) != 0;
    }
}

// The value, opaque to the optimiser: what is computed from it is not carried in
// registers over the steps of a launch.
template <typename T>
__device__ __forceinline__ T per_step(T v) {
    asm volatile("" : "+v"(v));
    return v;
}

// Workgroups go to the 8 XCDs round-robin: each XCD takes a contiguous run of the
// table, so that neighbouring tiles share an L2.  -1 past the end.
__device__ __forceinline__ int block_index(int n) {
    const int per = (n + 7) >> 3;
    const int i = (int)(blockIdx.x & 7) * per + (int)(blockIdx.x >> 3);
    return (int)(blockIdx.x >> 3) < per && i < n ? i : -1;
}

// The planes of a region in LDS, plane k of node `at` at word PAD + k N + at: every
// neighbour of every plane of every node of a thread lies at a non-negative constant
// distance from its first node's word.  A DS instruction's constant reaches 64 KB, so
// the planes from REACH on get an address register of their own.  Both are made once
// per launch, as byte addresses, and are opaque to the optimiser, which would else
// carry sums of them in further registers.
template <typename S>
struct BlockAt {
    int lo, hi;
    __device__ __forceinline__ explicit BlockAt(int at) : lo(per_step(4 * at)), hi(per_step(4 * (at + S::REACH * S::N))) {}
    // plane `plane` of node j, `off` words further
    __device__ __forceinline__ float& ref(float* lds, int j, int plane, int off) const {
        char* b = reinterpret_cast<char*>(lds);
        return plane < S::REACH
                   ? *reinterpret_cast<float*>(b + 4 * (S::PAD + plane * S::N + j * S::JS + off) + lo)
                   : *reinterpret_cast<float*>(b + 4 * (S::PAD + (plane - S::REACH) * S::N + j * S::JS + off) + hi);
    }
    // the neighbour (dx, dy)
    __device__ __forceinline__ float& at(float* lds, int j, int plane, int dx = 0, int dy = 0) const {
        return ref(lds, j, plane, dy * S::RX + dx);
    }
};

// Populations 1..8 of the node at `at` of a region of RX columns, streamed from the
// neighbours' (plane i - 1 of F) or by bounce-back; f[0] is the node's own.  A
// wavefront without boundary nodes reads at offsets fixed at compile time.
template <bool WALLS, typename S>
__device__ __forceinline__ void block_pull(float* lds, const BlockAt<S>& k, int j, unsigned sm, float f0,
                                           float (&f)[9]) {
    f[0] = f0;
#pragma unroll
    for (int i = 1; i < 9; ++i)
        if constexpr (WALLS) {
            const bool bb = (sm >> opp_(i)) & 1u;
            f[i] = *reinterpret_cast<float*>(
                reinterpret_cast<char*>(lds) + 4 * (S::PAD + j * S::JS) + k.lo +
                4 * (bb ? (opp_(i) - 1) * S::N : (i - 1) * S::N - ey_(i) * S::RX - ex_(i)));
        } else {
            f[i] = k.at(lds, j, i - 1, -ex_(i), -ey_(i));
        }
}

// Calls body(sm, std::bool_constant) with the solid-neighbour bits of a node; a
// wavefront without such neighbours runs code compiled for none.
template <typename F>
__device__ __forceinline__ void block_node(const BlockNode& n, F body) {
    if (n.walls)
        body(per_step(n.sm), std::true_type{});
    else
        body(0u, std::false_type{});
}

// ---- van der Waals model ---------------------------------------------------------
template <typename S, typename CT, bool FORCE>
__global__ void __launch_bounds__(S::NT, S::WAVES) lb_block_vdw(BlockArgs a) {
    const int bi = block_index(a.nblocks);
    if (bi < 0) return;
    const BlockDev b = a.blocks[bi];
    const CapDev c = a.caps[b.cap];
    const Geo g = geo_of(c);
    const int P = (int)c.plane;
    const int sb = a.cur ^ c.par;
    const Planes fs = planes_of((sb ? a.arena1 : a.arena0) + c.off_f, 9, P, c.pitch);
    const Planes fd = planes_of((sb ? a.arena0 : a.arena1) + c.off_f, 9, P, c.pitch);

    constexpr int NPT = S::NPT, QP = 8;
    // planes 0..7: shifted populations 1..8; QP: drho
    __shared__ float lds[S::PAD + 9 * S::N];

    BlockNode n[NPT];
    block_nodes<S>(g, b, a, fs.rb, n);
    const BlockAt<S> k(threadIdx.x);
    const float G2 = 2.f * c.G;

    float f0[NPT];
    {
        float f[NPT][9];
#pragma unroll
        for (int j = 0; j < NPT; ++j)
            if (n[j].dist <= 2 * a.steps) {
#pragma unroll
                for (int i = 0; i < 9; ++i) f[j][i] = ld(fs, n[j].voff, i * fs.pb);
            }
#pragma unroll
        for (int j = 0; j < NPT; ++j) {
            if (n[j].dist <= 2 * a.steps) {
                f0[j] = f[j][0];
#pragma unroll
                for (int i = 1; i < 9; ++i) k.at(lds, j, i - 1) = f[j][i];
                if (!n[j].fluid) k.at(lds, j, QP) = 0.f;
            }
            if (!n[j].fluid) n[j].dist = BLOCK_NOWHERE;   // nothing more to do there
        }
    }
    for (int left = a.steps - 1; left >= 0; --left) {
        lds_barrier();
        Mom<float> mom[NPT];
#pragma unroll
        for (int j = 0; j < NPT; ++j)
            if (n[j].dist <= 2 * left + 1)
                block_node(n[j], [&](unsigned sm, auto walls) {
                    float p[9];
                    block_pull<walls.value>(lds, k, j, sm, f0[j], p);
                    mom[j] = moments_of(p, sm != 0u);
                    k.at(lds, j, QP) = mom[j].drho;
                });
        lds_barrier();
#pragma unroll
        for (int j = 0; j < NPT; ++j)
            if (n[j].dist <= 2 * left) {
                float dxf, dyf, lapf;
                CT o[9];
                auto collide = [&](unsigned sm, auto) {
                    const float* q0 = &k.at(lds, j, QP);
                    stencil3(q0 - S::RX, q0, q0 + S::RX, 0, sm, G2, dxf, dyf, lapf);
                    vdw_node_collide<CT, FORCE>(c, mom[j], sm, dxf, dyf, lapf, o);
                };
                // (with a force one code for all nodes: the sums with it would not be
                // contracted alike in the two)
                if constexpr (FORCE)
                    collide(per_step(n[j].sm), std::true_type{});
                else
                    block_node(n[j], collide);
                if (left > 0) {
                    f0[j] = (float)o[0];
#pragma unroll
                    for (int i = 1; i < 9; ++i) k.at(lds, j, i - 1) = (float)o[i];
                } else {
#pragma unroll
                    for (int i = 0; i < 9; ++i) st(fd, (float)o[i], n[j].voff, i * fd.pb);
                }
            }
    }
}

// ---- binary model, moment storage ------------------------------------------------
// Reads the state and phi (written by the step before), writes the state `steps`
// steps later and phi one step after it.
template <typename S, typename CT, typename ST, bool FORCE>
__global__ void __launch_bounds__(S::NT, S::WAVES) lb_block_bin(BlockArgs a) {
    const int bi = block_index(a.nblocks);
    if (bi < 0) return;
    const BlockDev b = a.blocks[bi];
    const CapDev c = a.caps[b.cap];
    const Geo g = geo_of(c);
    const int P = (int)c.plane;
    const int sb = a.cur ^ c.par;
    const Planes ms = planes_of((sb ? a.arena1 : a.arena0) + c.off_f, NMOM, P, c.pitch);
    const Planes ps = planes_of((sb ? a.arena1 : a.arena0) + c.off_phi, 1, P, c.pitch);
    const Planes md = planes_of((sb ? a.arena0 : a.arena1) + c.off_f, NMOM, P, c.pitch);
    const Planes pd = planes_of((sb ? a.arena0 : a.arena1) + c.off_phi, 1, P, c.pitch);

    constexpr int NPT = S::NPT, UX = 8, UY = 9, AM = 10, PH = 11;
    // planes 0..7: populations 1..8; UX, UY, AM: ux, uy, A; PH, PH + 1: phi of this
    // step and of the next one in turn
    __shared__ float lds[S::PAD + 13 * S::N];

    BlockNode n[NPT];
    block_nodes<S>(g, b, a, ms.rb, n);
    const BlockAt<S> k(threadIdx.x);
    const float G2 = 2.f * c.G;
    const float kap = c.kappa, Gam = c.Gamma;

    int q[NPT];         // phi in fixed point
    float f0[NPT];
    // kp: this step's phi is plane PH, kn: the next one's is
    BlockAt<S> kp = k, kn = k;
    kn.hi = per_step(k.hi + 4 * S::N);
    static_assert(S::REACH <= PH, "phi is reached from hi");
    // the populations and phi of node j for its neighbours
    auto exchange = [&](int j, const float (&m)[NMOM], const BlockAt<S>& phi) {
        float f[9];
        pops_of_stored(m, f);
        f0[j] = f[0];
#pragma unroll
        for (int i = 1; i < 9; ++i) k.at(lds, j, i - 1) = f[i];
        phi.at(lds, j, PH) = phi_of_fixed(phi_bits(q[j]));
    };
    {
        float m[NPT][NMOM];
#pragma unroll
        for (int j = 0; j < NPT; ++j)
            if (n[j].dist <= 2 * a.steps) {
#pragma unroll
                for (int i = 0; i < NMOM; ++i) m[j][i] = ld(ms, n[j].voff, i * ms.pb);
                q[j] = __builtin_bit_cast(int, ld(ps, n[j].voff, 0));
            }
#pragma unroll
        for (int j = 0; j < NPT; ++j) {
            if (n[j].dist <= 2 * a.steps) {
                if (n[j].fluid) {
                    exchange(j, m[j], kp);
                } else {
#pragma unroll
                    for (int i = UX; i <= PH + 1; ++i) k.at(lds, j, i) = 0.f;
                }
            }
            if (!n[j].fluid) n[j].dist = BLOCK_NOWHERE;   // nothing more to do there
        }
    }
    for (int left = a.steps - 1; left >= 0; --left) {
        lds_barrier();
        Mom<float> mom[NPT];
        float dxf[NPT], dyf[NPT], lapf[NPT];
#pragma unroll
        for (int j = 0; j < NPT; ++j)
            if (n[j].dist <= 2 * left + 1) {
                float p[9];
                block_node(n[j], [&](unsigned sm, auto walls) { block_pull<walls.value>(lds, k, j, sm, f0[j], p); });
                const unsigned sm = per_step(n[j].sm);
                mom[j] = moments_of(p, sm != 0u);
                const float Fb = sm != 0u ? 0.f : c.Fx;
                const float inv_rho = recip(c.rho_ref + mom[j].drho);
                const float ux = (mom[j].jx + 0.5f * Fb) * inv_rho, uy = mom[j].jy * inv_rho;
                stencil3(&kp.at(lds, j, PH, 0, -1), &kp.at(lds, j, PH), &kp.at(lds, j, PH, 0, 1), 0, sm, G2, dxf[j],
                         dyf[j], lapf[j]);
                const float ph = kp.at(lds, j, PH);
                const float gmu = Gam * (mu_bulk(c, ph) - kap * lapf[j]);
                k.at(lds, j, UX) = ux;
                k.at(lds, j, UY) = uy;
                k.at(lds, j, AM) = gmu - 0.5f * ph * (ux * ux + uy * uy);
            }
        lds_barrier();
#pragma unroll
        for (int j = 0; j < NPT; ++j)
            if (n[j].dist <= 2 * left) {
                const unsigned sm = per_step(n[j].sm);
                const float phi = kp.at(lds, j, PH);
                const float uxf = k.at(lds, j, UX), uyf = k.at(lds, j, UY);
                const PostState<CT> s8 =
                    bin_node_state<CT, ST, FORCE>(c, mom[j], sm, phi, dxf[j], dyf[j], lapf[j], uxf, uyf);
                const float m[NMOM] = {(float)s8.drho, (float)third(s8.jx), (float)third(s8.jy), (float)s8.b,
                                       (float)s8.d, (float)s8.pxx, (float)s8.pxy};
                __builtin_amdgcn_sched_barrier(0);
                const float dphi = phi_delta(sm, phi, uxf, uyf, k.at(lds, j, AM),
                                             [&](int i, float& am, float& pp, float& x, float& y) {
                                                 am = k.at(lds, j, AM, -ex_(i), -ey_(i));
                                                 pp = kp.at(lds, j, PH, -ex_(i), -ey_(i));
                                                 x = k.at(lds, j, UX, -ex_(i), -ey_(i));
                                                 y = k.at(lds, j, UY, -ex_(i), -ey_(i));
                                             });
                q[j] += fixed_of_phi(dphi);
                if (left > 0) {
                    exchange(j, m, kn);
                } else {
#pragma unroll
                    for (int i = 0; i < NMOM; ++i) st(md, m[i], n[j].voff, i * md.pb);
                    st(pd, phi_bits(q[j]), n[j].voff, 0);
                }
            }
        const int h = kp.hi;
        kp.hi = per_step(kn.hi);
        kn.hi = per_step(h);
    }
}

}  // namespace lbk
