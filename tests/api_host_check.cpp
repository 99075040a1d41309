// Checks of the library's host logic on a HIP runtime of host memory (host_hip.h):
// the name of one check is the argument.
#include <cstdio>

#include "lb_api.hip"

#include "host_hip.h"

#define EXPECT(x)                                                     \
    do {                                                              \
        if (!(x)) {                                                   \
            std::printf("%s:%d: %s\n", __FILE__, __LINE__, #x);     \
            return 1;                                                 \
        }                                                             \
    } while (0)

static lb_params params(lb_model m) {
    lb_params p{};
    p.model = m;
    p.kappa = m == LB_VDW ? 0.02 : 0.04;
    p.a = 9.0 / 49.0, p.b = 2.0 / 21.0, p.T = 0.56;
    p.A = p.B = 0.04, p.Gamma = 1.0;
    p.nu_l = p.nu_g = 0.2;
    p.theta_deg = std::nan("");
    p.q_mid = std::nan("");
    return p;
}

// n capillaries of one model
static lb_ctx* context(lb_model m, const std::vector<lb_geometry>& g) {
    std::vector<lb_params> p(g.size(), params(m));
    std::vector<std::vector<double>> q;
    std::vector<const double*> qp;
    for (const lb_geometry& x : g) q.emplace_back((size_t)x.nx * x.ny, m == LB_VDW ? 3.0 : 0.5);
    for (const auto& x : q) qp.push_back(x.data());
    lb_ctx* c = nullptr;
    return lb_batch_init(&c, (int)g.size(), p.data(), g.data(), qp.data(), nullptr) == LB_OK ? c : nullptr;
}

static const lb_geometry SMALL{256, 64, 128, 128, 20, 22};

// An executable graph is destroyed only after the stream has been waited for.
static int graphs_outlive_their_replays() {
    for (lb_model m : {LB_VDW, LB_BINARY}) {
        lb_ctx* c = context(m, {SMALL, SMALL});
        EXPECT(c);
        EXPECT(lb_step(c, 200) == LB_OK && rt.replays > 0 && rt.pending);
        EXPECT(lb_batch_retire(c, 1) == LB_OK);
        EXPECT(rt.destroyed_pending == 0);
        EXPECT(lb_step(c, 200) == LB_OK && rt.pending);
        lb_launch_config cfg;
        EXPECT(lb_get_launch_config(c, &cfg) == LB_OK);
        cfg.graph_steps = 0;
        EXPECT(lb_set_launch_config(c, &cfg) == LB_OK);
        EXPECT(rt.destroyed_pending == 0);
        lb_free(c);
        EXPECT(rt.destroyed_pending == 0);
    }
    return 0;
}

// A table upload that fails leaves a context that refuses to step, until the call
// that set it is repeated.
static int failed_tables_do_not_step() {
    for (lb_model m : {LB_VDW, LB_BINARY}) {
        lb_ctx* c = context(m, {SMALL, SMALL});
        EXPECT(c);
        lb_launch_config own, strips;
        EXPECT(lb_get_launch_config(c, &own) == LB_OK);
        strips = own;
        strips.schedule = 3;
        for (int copy = 0; copy < 3; ++copy) {   // a descriptor, the tiles, the tables of the block kernels
            EXPECT(lb_step(c, 3) == LB_OK);
            auto broken = [&]() -> bool {
                const long t = lb_time(c);
                return lb_step(c, 5) == LB_ESTATE && lb_time(c) == t && lb_check(c) == LB_ESTATE;
            };
            rt.skip_copies = copy, rt.fail_copies = 1;
            EXPECT(lb_batch_retire(c, 0) == LB_EDEVICE && broken());
            EXPECT(lb_batch_retire(c, 0) == LB_OK && lb_step(c, 5) == LB_OK && lb_check(c) == LB_OK);
            rt.skip_copies = copy, rt.fail_copies = 1;
            EXPECT(lb_batch_revive(c, 0) == LB_EDEVICE && broken());
            EXPECT(lb_batch_revive(c, 0) == LB_OK);
        }
        for (int copy = 0; copy < (m == LB_BINARY ? 3 : 2); ++copy) {   // (descriptors of a changed storage)
            EXPECT(lb_set_launch_config(c, &strips) == LB_OK);
            rt.skip_copies = copy, rt.fail_copies = 1;
            EXPECT(lb_set_launch_config(c, &own) == LB_EDEVICE);
            EXPECT(lb_step(c, 5) == LB_ESTATE);
            rt.launches.clear();
            EXPECT(lb_set_launch_config(c, &own) == LB_OK);
            EXPECT(rt.count("lb_convert") == 0 && c->d_caps[1].mstore == (m == LB_BINARY));
            EXPECT(lb_step(c, 1) == LB_OK && rt.count("lb_block") == 1);
        }
        std::vector<char> image(lb_checkpoint_bytes(c));
        EXPECT(lb_save(c, image.data(), image.size()) == LB_OK);
        const int copies = m == LB_BINARY ? 7 : 5;   // populations (and phi) of two, descriptors, tiles, table
        for (int copy = 0; copy < copies; ++copy) {
            rt.skip_copies = copy, rt.fail_copies = 1;
            EXPECT(lb_load(c, image.data(), image.size()) == LB_EDEVICE && lb_step(c, 5) == LB_ESTATE);
            EXPECT(lb_load(c, image.data(), image.size()) == LB_OK && lb_step(c, 1) == LB_OK);
        }
        lb_free(c);
    }
    return 0;
}

// A context allocates no device memory beyond its state: none with a caller's
// d_state, and none when capillaries retire, return or load, or launch
// configurations change, whatever the plan becomes.
static int no_device_memory_beside_the_state() {
    unsigned s = 1;
    auto rnd = [&](int lo, int hi) {
        s = s * 1664525u + 1013904223u;
        return lo + (int)((s >> 8) % (unsigned)(hi - lo + 1));
    };
    for (int pass = 0; pass < 30; ++pass) {
        const lb_model m = pass % 2 ? LB_VDW : LB_BINARY;
        std::vector<lb_geometry> g;
        for (int n = rnd(2, 24); n > 0; --n) {
            const int ny = rnd(20, 120), nx = rnd(60, 900), h = rnd(8, ny - 4), len = rnd(20, nx - 20);
            g.push_back({nx, ny, rnd(1, nx - len), len, h, rnd(1, ny - 1 - h)});
        }
        lb_ctx* c = context(m, g);
        EXPECT(c);
        const int before = rt.mallocs;
        std::vector<char> image(lb_checkpoint_bytes(c));
        EXPECT(lb_save(c, image.data(), image.size()) == LB_OK);
        lb_launch_config cfg, strips;
        EXPECT(lb_get_launch_config(c, &cfg) == LB_OK);
        strips = cfg;
        strips.schedule = 5;
        for (int k = 0; k < 40; ++k) {
            const int cap = rnd(0, (int)g.size() - 1);
            EXPECT((rnd(0, 2) ? lb_batch_retire(c, cap) : lb_batch_revive(c, cap)) == LB_OK);
            if (k % 10 == 5) {
                EXPECT(lb_set_launch_config(c, &strips) == LB_OK && lb_set_launch_config(c, &cfg) == LB_OK);
                EXPECT(lb_load(c, image.data(), image.size()) == LB_OK);
            }
            EXPECT(lb_step(c, 1) == LB_OK);
        }
        EXPECT(rt.mallocs == before);
        lb_free(c);

        // in the caller's memory, which is not touched past its end
        const lb_params p = params(m);
        const size_t bytes = lb_state_bytes(&p, &g[0]);
        char* mem = (char*)std::aligned_alloc(4096, (bytes + 8191) / 4096 * 4096);
        std::memset(mem + bytes, 0x5a, 4096);
        const std::vector<double> q((size_t)g[0].nx * g[0].ny, m == LB_VDW ? 3.0 : 0.5);
        EXPECT(lb_init(&c, &p, &g[0], q.data(), mem, bytes, nullptr) == LB_OK);
        EXPECT(lb_step(c, 9) == LB_OK && rt.mallocs == before);
        lb_free(c);
        for (int k = 0; k < 4096; ++k) EXPECT(mem[bytes + k] == 0x5a);
        std::free(mem);
    }
    return 0;
}

// The single-step tiles are, in order, those with a fluid node.
static int tiles_with_fluid() {
    unsigned s = 3;
    auto rnd = [&](int lo, int hi) {
        s = s * 1664525u + 1013904223u;
        return lo + (int)((s >> 8) % (unsigned)(hi - lo + 1));
    };
    for (int pass = 0; pass < 2000; ++pass) {
        lb_geometry g{rnd(3, 400), rnd(5, 90), 0, 0, 0, 0};
        if (pass % 8) {
            g.tube_len = rnd(1, g.nx), g.x_in = rnd(0, g.nx - g.tube_len);
            g.tube_h = rnd(3, g.ny - 2), g.y0 = rnd(1, g.ny - 1 - g.tube_h);
        }
        const int rows = 1 << rnd(0, 3);
        std::vector<TileDev> t;
        build_tiles({g, g}, {0, 1}, rows, t);
        size_t at = 0;
        for (int y0 = 0; y0 < g.ny; y0 += rows)
            for (int x0 = 0; x0 < g.nx; x0 += TILE_W) {
                bool fluid = false;
                const int h = std::min(rows, g.ny - y0);
                for (int y = y0; y < y0 + h; ++y)
                    for (int x = x0; x < std::min(x0 + TILE_W, g.nx); ++x) fluid = fluid || !solid_at(g, x, y);
                if (!fluid) continue;
                EXPECT(at < t.size() && t[at].cap == 1 && t[at].x0 == x0 && t[at].y0 == y0 && t[at].rows == h);
                ++at;
            }
        EXPECT(at == t.size() && (int)at == count_tiles(g, rows));
    }
    return 0;
}

// Single steps of large contexts go by the row sweep, all others by the tiles; what
// is large is counted over the active capillaries.
static int single_steps_of_large_contexts() {
    const lb_geometry part{1500, 500, 100, 1000, 200, 150}, large{3000, 1500, 700, 1000, 1400, 50};
    for (lb_model m : {LB_VDW, LB_BINARY}) {
        const char* rows = m == LB_VDW ? "lb_wide_vdw" : "lb_wmom_bin";
        lb_ctx* c = context(m, {large, part});
        EXPECT(c);
        lb_launch_config cfg;
        EXPECT(lb_get_launch_config(c, &cfg) == LB_OK);
        cfg.graph_steps = 0;
        EXPECT(lb_set_launch_config(c, &cfg) == LB_OK);
        const int K = c->block_k;
        auto launches = [&](long steps, int tiles, int sweeps) {
            rt.launches.clear();
            return lb_step(c, steps) == LB_OK && rt.count("lb_block") == tiles && rt.count(rows) == sweeps &&
                   (int)rt.launches.size() == tiles + sweeps;
        };
        EXPECT(launches(1, 0, 1));
        // K steps, and (binary) the last one of the call
        EXPECT(m == LB_VDW ? launches(K, 1, 0) && launches(K + 1, 1, 1) : launches(K + 1, 1, 1) && launches(K + 2, 1, 2));
        EXPECT(lb_batch_retire(c, 0) == LB_OK);   // 0.45 M nodes are left
        EXPECT(launches(1, 1, 0));
        EXPECT(lb_batch_revive(c, 0) == LB_OK && launches(1, 0, 1));
        lb_free(c);
    }
    return 0;
}

// A run replays graphs as soon as it holds the steps of one, and every graph of a
// call is captured before the first launch.
static int graphs_are_replayed() {
    const lb_geometry large{3000, 1500, 700, 1000, 1400, 50}, mid{1024, 128, 256, 768, 40, 44};
    for (lb_model m : {LB_VDW, LB_BINARY})
        for (const lb_geometry& g : {SMALL, mid, large})
            for (int graph_steps : {6, 30, 64})
                for (int every : {0, 16, 63, 64, 65, 100}) {
                    lb_ctx* c = context(m, {g});
                    EXPECT(c);
                    lb_launch_config cfg;
                    EXPECT(lb_get_launch_config(c, &cfg) == LB_OK);
                    cfg.graph_steps = graph_steps;
                    EXPECT(lb_set_launch_config(c, &cfg) == LB_OK && lb_step(c, 5) == LB_OK);
                    (void)hipStreamSynchronize(c->stream);
                    const int K = c->block_k, held = graph_steps / K * K;   // steps of a graph
                    EXPECT(K > 1);
                    const HostRuntime before = rt;
                    rt.launches.clear();
                    EXPECT(lb_batch_step(c, 400, every) == LB_OK && lb_time(c) == 405);
                    EXPECT(rt.late_captures == before.late_captures);
                    long want = 0;
                    for (long t = 5; t < 405;) {
                        const long n = every ? std::min(405 - t, every - t % every) : 400;
                        want += held ? (n - (m == LB_BINARY)) / held : 0;
                        t += n;
                    }
                    EXPECT(rt.replays - before.replays == want);
                    EXPECT(want > 0 ? rt.captures > before.captures : rt.captures == before.captures);
                    lb_free(c);
                }
    return 0;
}

// The tuner times whole launches only, at least trial_steps steps of each candidate.
static int tuner_times_whole_launches() {
    const lb_geometry mid{1024, 128, 256, 768, 40, 44}, wide{2600, 560, 500, 1900, 440, 50};
    for (lb_model m : {LB_VDW, LB_BINARY})
        for (const lb_geometry& g : {SMALL, mid, wide})
            for (int trial : {2, 3, 5, 10, 128}) {
                lb_ctx* c = context(m, {g});
                EXPECT(c);
                const int K = c->block_k;
                rt.launches.clear();
                lb_launch_config best;
                double us;
                EXPECT(lb_autotune(c, trial, &best, &us) == LB_OK && lb_time(c) == 0);
                int steps = 0;
                for (const Launched& l : rt.launches)
                    if (l.kernel.find("lb_block") != std::string::npos) {
                        EXPECT(l.block.steps == K && l.block.halo == 2 * K);
                        steps += l.block.steps;
                    }
                EXPECT(steps >= trial + 2);
                if (m == LB_VDW) EXPECT(rt.count("lb_wide_vdw") == 0);   // (an odd step of schedule 5)
                lb_free(c);
            }
    return 0;
}

// Read-outs pass through memory that is coherent by its flags, and the events that the
// host waits for in between release to the system.
static int read_outs_are_coherent() {
    lb_ctx* c = context(LB_BINARY, {SMALL});
    EXPECT(c);
    rt.event_flags.clear();
    std::vector<double> q((size_t)SMALL.nx * SMALL.ny);
    EXPECT(lb_moments(c, q.data(), nullptr, nullptr, nullptr) == LB_OK);
    int n = 0;
    EXPECT(lb_batch_l_history(c, 0, nullptr, nullptr, 0, &n) == LB_OK);
    EXPECT(rt.pinned_flags.size() == 1 && rt.event_flags.size() == 2);
    EXPECT((rt.pinned_flags[0] & hipHostMallocCoherent) && (rt.pinned_flags[0] & hipHostMallocMapped) &&
           (rt.pinned_flags[0] & hipHostMallocPortable) && !(rt.pinned_flags[0] & hipHostMallocNonCoherent));
    for (unsigned f : rt.event_flags) EXPECT((f & hipEventReleaseToSystem) && (f & hipEventDisableTiming));
    lb_free(c);
    return 0;
}

// Under a caller's capture a call is direct launches, evenly many for an even number
// of steps; one that steps graph_steps at a time is refused.
static int captured_calls_can_be_replayed() {
    const lb_geometry mid{1024, 128, 256, 768, 40, 44}, large{3000, 1500, 700, 1000, 1400, 50};
    for (lb_model m : {LB_VDW, LB_BINARY})
        for (const lb_geometry& g : {SMALL, mid, large})
            for (int schedule : {m == LB_VDW ? 4 : 6, 3, 5})
                for (int every : {0, 7})
                    for (long n = 1; n < 70; ++n) {
                        static lb_ctx* c = nullptr;
                        static lb_launch_config cfg;
                        if (n == 1) {
                            lb_free(c);
                            c = context(m, {g});
                            EXPECT(c && lb_get_launch_config(c, &cfg) == LB_OK);
                            cfg.schedule = schedule;
                            EXPECT(lb_set_launch_config(c, &cfg) == LB_OK);
                            EXPECT(lb_step(c, 200) == LB_OK);   // (its graphs are there)
                        }
                        const long t = lb_time(c);
                        const int cur = c->cur, replays = rt.replays;
                        hipGraph_t graph;
                        EXPECT(hipStreamBeginCapture(c->stream, hipStreamCaptureModeThreadLocal) == hipSuccess);
                        rt.launches.clear();
                        const lb_status s = lb_batch_step(c, n, every);
                        EXPECT(rt.capturing && rt.replays == replays);
                        EXPECT(hipStreamEndCapture(c->stream, &graph) == hipSuccess && hipGraphDestroy(graph) == hipSuccess);
                        if (!every && n >= cfg.graph_steps) {
                            EXPECT(s == LB_EDEVICE && rt.launches.empty() && lb_time(c) == t);
                            continue;
                        }
                        EXPECT(s == LB_OK && lb_time(c) == t + n);
                        int steps = 0, launches = 0;
                        for (const Launched& l : rt.launches) {
                            if (l.kernel.find("lb_interface") != std::string::npos ||
                                l.kernel.find("lb_health") != std::string::npos)
                                continue;
                            ++launches;
                            const bool two = l.kernel.find("lb_wide2") != std::string::npos;
                            steps += l.kernel.find("lb_block") != std::string::npos ? l.block.steps : 1 + two;
                        }
                        EXPECT(steps == n && launches % 2 == n % 2 && (c->cur ^ cur) == n % 2);
                    }
    return 0;
}

// The tiles of a context of billions of nodes go to launches of fewer than 2^32 threads,
// each tile once.
static int large_tables_in_several_launches() {
    for (lb_model m : {LB_VDW, LB_BINARY})
        for (int shape = 0; shape < BLOCK_SHAPES; ++shape) {
            lb_ctx* c = context(m, {SMALL});
            EXPECT(c);
            c->block_shape = shape;
            for (int n : {1, BLOCK_SLICE, BLOCK_SLICE + 1, 6000000}) {
                c->nblocks = n;   // (the kernels do not run)
                rt.launches.clear();
                enqueue_block(c, c->block_k);
                EXPECT(hipGetLastError() == hipSuccess);
                const BlockDev* at = c->d_blocks;
                for (const Launched& l : rt.launches) {
                    EXPECT(l.block.blocks == at && l.block.steps == c->block_k);
                    at += l.block.nblocks;
                }
                EXPECT(at == c->d_blocks + n);
            }
            lb_free(c);
        }
    return 0;
}

int main(int argc, char** argv) {
    const struct {
        const char* name;
        int (*run)();
    } checks[] = {
        {"graphs_outlive_their_replays", graphs_outlive_their_replays},
        {"failed_tables_do_not_step", failed_tables_do_not_step},
        {"single_steps_of_large_contexts", single_steps_of_large_contexts},
        {"graphs_are_replayed", graphs_are_replayed},
        {"tuner_times_whole_launches", tuner_times_whole_launches},
        {"read_outs_are_coherent", read_outs_are_coherent},
        {"captured_calls_can_be_replayed", captured_calls_can_be_replayed},
        {"large_tables_in_several_launches", large_tables_in_several_launches},
        {"tiles_with_fluid", tiles_with_fluid},
        {"no_device_memory_beside_the_state", no_device_memory_beside_the_state},
    };
    for (const auto& k : checks)
        if (argc == 2 && std::string(argv[1]) == k.name) return k.run();
    std::printf("no such check\n");
    return 2;
}
