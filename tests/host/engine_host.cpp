// Scheduling of the host engine, checked without a GPU (fake_device.h): each
// check prints its name and whether it held; the exit status counts failures.
#include "engine.cpp"

#include "fake_device.h"

// Heap allocations so far (no exception may cross the C interface, and a
// polling step makes none).
static long allocations = 0;
void *operator new(size_t n)
{
    ++allocations;
    if (void *p = std::malloc(n ? n : 1)) return p;
    throw std::bad_alloc();
}
void *operator new(size_t n, const std::nothrow_t &) noexcept
{
    ++allocations;
    return std::malloc(n ? n : 1);
}
void operator delete(void *p) noexcept { std::free(p); }
void operator delete(void *p, size_t) noexcept { std::free(p); }

namespace {

int failures = 0;

void check(bool ok, const char *what)
{
    std::printf("%s: %s\n", ok ? "ok" : "FAILED", what);
    std::fflush(stdout);
    failures += !ok;
}

void fresh_device()
{
    dev = Device();
    g_taken[0] = 0;
}

// A context of one density on an n^3 grid with p = 0 on top.
struct Context {
    std::vector<double> rho, rhs, p;
    std::vector<char> ws;
    pcg_ctx_t *c = nullptr;
    int status = 0;

    Context(int nx, int ny, int nz, pcg_opts_t o, size_t spare = 0)
    {
        const pcg_grid_t g = { nx, ny, nz, 1.0 };
        const size_t n = (size_t)nx * ny * nz;
        rho.assign(n, 1.0);
        rhs.assign(n, 1.0);
        p.assign(n, 0.0);
        pcg_bc_t bc{};
        bc.kind[5] = PCG_BC_DIRICHLET;
        size_t need = 0;
        pcg_workspace_bytes(&g, &o, &need);
        ws.resize(need + spare + 256);
        void *at = (void *)(((uintptr_t)ws.data() + 255) / 256 * 256);
        status = pcg_setup(&c, &g, rho.data(), nullptr, &bc, &o, at, need + spare, nullptr);
        dev.count_from_zero();
    }
    ~Context() { pcg_destroy(c); }
    pcg_stats_t solve(double tol, int maxit, int flags = 0)
    {
        pcg_stats_t st{};
        dev.count_from_zero();
        status = pcg_solve_ex(c, rhs.data(), p.data(), tol, maxit, flags, &st);
        return st;
    }
};

// A resident FP32 + refinement solve looks at its state after a few trips,
// whatever reduction is asked of one, and after the first where the solve
// may end there.
void refinement_trips()
{
    fresh_device();
    pcg_opts_t o{};
    o.precision = PCG_PREC_FP32_IR;
    {
        Context c(33, 31, 29, o);
        const pcg_stats_t st = c.solve(1e-11, 1000000);
        check(c.status == PCG_OK && st.outer_iters == 4 && dev.resident <= 5 && dev.waits <= 2,
              "refinement: one wait where the tolerance needs three trips");
    }
    dev.trips = 1;
    for (double inner : { 0.9, 0.99, 0.9999999, 1.0 - 0x1p-53 }) {
        o.inner_tol = inner;
        Context c(33, 31, 29, o);
        c.solve(1e-11, 1000000);
        check(c.status == PCG_OK && dev.resident <= 6, "refinement: few trips queued for an inner_tol near 1");
        c.solve(1e-300, 1000000);
        check(c.status == PCG_OK && dev.resident <= 6, "refinement: few trips queued for a tolerance out of reach");
    }
    o.inner_tol = 0.0;
    Context c(33, 31, 29, o);
    c.solve(1e-11, 1000000, PCG_WARM_START);
    check(c.status == PCG_OK && dev.resident <= 1 && dev.waits == 1,
          "refinement: a warm start is looked at after its first trip");
    dev.trips = 3;
    const pcg_stats_t st = c.solve(1e-11, 5);
    check(c.status == PCG_MAXIT && st.iters == 5 && dev.resident <= 1 && dev.waits == 1,
          "refinement: so is a solve of few iterations");
}

// A solve whose workgroups do not get to run side by side, or whose launch is
// refused, ends on the tile passes with the same status and iterations, and
// so do the later ones of the context and every member of a batch.
void left_the_chip()
{
    for (int prec : { PCG_PREC_FP64, PCG_PREC_FP32_IR })
        for (int refused : { 0, 1 })
            for (int maxit : { 1000000, 40 }) {
                fresh_device();
                pcg_opts_t o{};
                o.precision = prec;
                Context c(33, 31, 29, o);
                const pcg_stats_t a = c.solve(1e-11, maxit);
                const int sa = c.status;
                check(sa == (maxit == 40 ? PCG_MAXIT : PCG_OK) && dev.resident > 0, "on the chip");
                int32_t wgs = -1, cells = -1;
                check(pcg_resident_form(c.c, &wgs, &cells) == PCG_OK && wgs > 1 && wgs <= dev.cus && cells > 0,
                      "resident form: reported");
                pcg_set_timing(c.c, 1);
                check(pcg_resident_form(c.c, &wgs, &cells) == PCG_OK && wgs == 0 && cells == 0,
                      "resident form: not for timed solves");
                pcg_set_timing(c.c, 0);
                (refused ? dev.refused : dev.timeouts) = 1;
                const pcg_stats_t b = c.solve(1e-11, maxit);
                check(pcg_resident_form(c.c, &wgs, &cells) == PCG_OK && wgs == 0 && cells == 0,
                      "resident form: none after leaving the chip");
                check(c.status == sa && b.iters == a.iters && b.outer_iters == a.outer_iters,
                      "left the chip: the tile passes solve it");
                const pcg_stats_t d = c.solve(1e-11, maxit);
                check(c.status == sa && d.iters == a.iters && dev.resident == 0 && dev.graphs > 0,
                      "left the chip: the next solve is theirs too");
            }
    // contexts created soon after do not try, later ones do (nor do time-outs
    // that the test hook asked for count)
    for (int kind : { 0, 1, 2 })
    for (int ago : { 0, 9, 11 }) {
        fresh_device();
        Context a(33, 31, 29, pcg_opts_t{});
        if (kind == 2) pcg_set_resident_limits(a.c, 0, 0);
        (kind == 0 ? dev.refused : dev.timeouts) = 1;
        a.solve(1e-8, 1000000);
        check((g_taken[0] != 0) == (kind < 2), "left the chip: noted for the device");
        if (kind < 2) g_taken[0] -= std::chrono::duration_cast<Clock::duration>(std::chrono::seconds(ago)).count();
        Context b(33, 31, 29, pcg_opts_t{});
        b.solve(1e-8, 1000000);
        check(a.status == PCG_OK && b.status == PCG_OK && (dev.resident > 0) == (ago > 10 || kind == 2),
              "left the chip: contexts created soon after");
    }
    for (int refused : { 0, 1 }) {
        fresh_device();
        pcg_opts_t o{};
        o.precision = PCG_PREC_FP32_IR;
        const pcg_grid_t g = { 17, 19, 21, 1.0 };
        const size_t n = (size_t)g.nx * g.ny * g.nz;
        std::vector<double> rho(n, 1.0), rhs(n, 1.0), p(n);
        std::vector<char> mem((16u << 20) + 256);
        pcg_bc_t bc{};
        bc.kind[5] = PCG_BC_DIRICHLET;
        pcg_batch_t *b = nullptr;
        pcg_batch_create(&b, (void *)(((uintptr_t)mem.data() + 255) / 256 * 256), 16u << 20, 8, &o, nullptr);
        int32_t slot[5], active = 1, steps = 0;
        auto admit = [&](int i) {
            return pcg_batch_admit(b, &g, rho.data(), nullptr, &bc, rhs.data(), p.data(), 1e-11, 1000000, 0,
                                   &slot[i]);
        };
        bool ok = true;
        for (int i = 0; i < 4; ++i) ok = ok && admit(i) == PCG_OK;
        ok = ok && pcg_batch_step(b, 1, &active) == PCG_OK && dev.resident > 0;
        (refused ? dev.refused : dev.timeouts) = 1;
        ok = ok && pcg_batch_step(b, 1, &active) == PCG_OK && active == 4;
        ok = ok && admit(4) == PCG_OK;
        while (ok && active && steps++ < 100) ok = pcg_batch_step(b, 1, &active) == PCG_OK;
        for (int i = 0; i < 5; ++i) {
            pcg_stats_t st;
            ok = ok && pcg_batch_poll(b, slot[i], &st) == PCG_OK && st.iters == 300 && st.outer_iters == 4;
        }
        check(ok && !active, "left the chip: every member of a batch ends");
        pcg_batch_destroy(b);
    }
}

// A step of several replays takes a batch's solves through their trips (and
// to the checks behind the last), not only to the end of the next one.
void several_replays()
{
    for (int prec : { PCG_PREC_FP64, PCG_PREC_FP32_IR })
        for (int top : { PCG_BC_DIRICHLET, PCG_BC_NEUMANN })
            for (int flags : { 0, (int)PCG_TWO_SWEEPS }) {
                fresh_device();
                // ten replays, or three trips of five: the first step of
                // eight ends within a loop
                dev.iters = prec == PCG_PREC_FP64 ? 300 : 150;
                pcg_opts_t o{};
                o.precision = prec;
                const pcg_grid_t g = { 17, 19, 21, 1.0 };
                const size_t n = (size_t)g.nx * g.ny * g.nz;
                std::vector<double> rho(n, 1.0), rhs(n, 1.0), p(n);
                std::vector<char> mem((16u << 20) + 256);
                pcg_bc_t bc{};
                bc.kind[5] = top;
                pcg_batch_t *b = nullptr;
                pcg_batch_create(&b, (void *)(((uintptr_t)mem.data() + 255) / 256 * 256), 16u << 20, 8, &o,
                                 nullptr);
                int32_t slot, active = 1, steps = 0;
                bool ok = true;
                for (int i = 0; i < 4; ++i)
                    ok = ok && pcg_batch_admit(b, &g, rho.data(), nullptr, &bc, rhs.data(), p.data(), 1e-11,
                                               1000000, flags, &slot) == PCG_OK;
                recorded.reserve(4096);   // (the stand-in's own list)
                const long before = allocations;
                while (ok && active && steps++ < 100) ok = pcg_batch_step(b, 8, &active) == PCG_OK;
                check(allocations == before, "a polling step allocates nothing");
                check(ok && steps <= 2 + (top == PCG_BC_NEUMANN), "several replays a step");
                pcg_batch_destroy(b);
            }
}

// The columns of the kernels around a solve: every cell in one lane's span of
// planes, most lanes of a full launch with a column, and launches that the
// runtime takes (fewer than 2^32 threads) up to the largest grid.
void columns()
{
    bool once = true, busy = true, fits = true;
    for (int P : { 1, 2, 6, 15, 16, 25, 63, 255, 256, 257, 300, 1000, 1023, 1024, 1025, 1300, 5000 })
        for (int nz : { 1, 2, 3, 4, 5, 7, 64, 333, 2049 }) {
            std::vector<int> seen((size_t)P * nz, 0);
            const int64_t T = col_tiles(P, nz);
            int64_t with = 0;
            for (int64_t t = 0; t < T; ++t)
                for (int l = 0; l < kBlock; ++l) {
                    const ColumnSpan c = col_span((uint32_t)t, (uint32_t)l, P, nz);
                    with += c.k1 > c.k0;
                    for (int k = c.k0; k < c.k1; ++k)
                        if (c.q < 0 || c.q >= P || k < 0 || k >= nz) once = false;
                        else ++seen[(size_t)k * P + c.q];
                }
            for (int v : seen) once = once && v == 1;
            if (T > 4) busy = busy && with >= 0.75 * T * kBlock;
        }
    for (int64_t P : { 1ll, 3ll, 31ll, 63ll, 1023ll, 1024ll, 65537ll, 178956970ll }) {
        const int nz = (int)std::min<int64_t>(INT32_MAX, ((int64_t(1) << 31) - 1) / P);
        const int64_t b = col_blocks(P, nz), T = col_tiles(P, nz);
        fits = fits && b >= 1 && b <= T && b * kBlock <= 0xffffffffll && T <= INT32_MAX &&
               (T + b) * kBlock / kBlock < 0x100000000ll;
        const ColumnSpan c = col_span((uint32_t)(T - 1), 0, (int)P, nz);
        fits = fits && c.q < P && c.k0 >= 0 && c.k0 < c.k1 && c.k1 <= nz;
    }
    check(once, "columns: every cell once");
    check(busy, "columns: three quarters of the lanes have one");
    check(fits, "columns: launches of the largest grids");
}

// Tile heights: a table that the caller installed is taken at its word; the
// built-in one (installed again, too) leaves room for more even heights.
void tile_rules()
{
    fresh_device();
    for (int prec : { PCG_PREC_FP64, PCG_PREC_FP32_IR })
        for (int flags : { (int)PCG_FLAT_TILES, (int)PCG_PLANE_TILES, (int)PCG_NARROW_TILES }) {
            const int table = flags == PCG_FLAT_TILES ? 0 : flags == PCG_PLANE_TILES ? 2 : 3;
            const int nx = table == 3 ? 131 : 132;
            pcg_opts_t o{};
            o.precision = prec;
            o.flags = flags;
            auto geometry = [&] {
                Context c(nx, 90, 97, o, 48 << 10);
                return c.c->eng.slots[0].geo;
            };
            const int table_tz = rule_for((int64_t)nx * 90 * 97, prec, false, table == 0 ? 0 : table == 3 ? 1 : 2).tz;
            const int before = geometry().tz;
            check(before != table_tz, "tile rules: the built-in height is replaced");
            int64_t mc[64];
            int32_t tz[64], gr[64], n = 0;
            pcg_get_tile_rules(prec, table, 64, mc, tz, gr, &n);
            const int64_t all[1] = { INT64_MAX };
            const int32_t own_tz[1] = { 17 }, own_grid[1] = { 256 };
            pcg_set_tile_rules(prec, table, 1, all, own_tz, own_grid);
            check(geometry().tz == 17, "tile rules: an installed height stands");
            pcg_set_tile_rules(prec, table, n, mc, tz, gr);
            check(geometry().tz == before, "tile rules: the built-in ones again");
        }
}

// The resident plan: every cell in one brick, no brick without cells, and
// each bound that the kernel relies on (threads, LDS, rows beside a brick, the
// reciprocal that divides by the row length, exchange words, workgroups).
void bricks()
{
    fresh_device();
    bool cover = true, bounds = true, some = false, none = true, exact = true;
    std::vector<ResidentShape> shapes(64);
    for (int prec : { PCG_PREC_FP64, PCG_PREC_FP32_IR }) {
        const int ns = resident_shapes(prec, shapes.data(), 64);
        const size_t es = prec == PCG_PREC_FP32_IR ? 4 : 8;
        for (const bool batch : { false, true }) {
            std::vector<int> cap;
            for (int i = 0; i < ns; ++i) cap.push_back(dev.cus * (batch ? shapes[i].batch : 1));
            for (const bool faces : { false, true })
                for (int nx : { 1, 2, 3, 24, 33, 97, 128, 255, 320, 511, 512, 513, 1000, 1536, 2560, 3071, 3072, 3073 })
                    for (int ny : { 1, 2, 3, 7, 29, 64, 101, 128, 500 })
                        for (int nz : { 1, 2, 5, 8, 9, 45, 96, 150, 2000 }) {
                            const pcg_grid_t g = { nx, ny, nz, 1.0 };
                            const ResidentPlan p =
                                resident_plan(g, prec, pcg_opts_t{}, batch, faces, shapes.data(), cap.data(), ns);
                            if (p.shape < 0) continue;
                            some = true;
                            const ResidentShape &sh = shapes[p.shape];
                            std::vector<int> seen((size_t)ny * nz, 0);
                            for (int b = 0; b < p.bricks(); ++b) {
                                const int j0 = b % p.rnby * p.rby, k0 = b / p.rnby * sh.planes;
                                const int by = std::min(p.rby, ny - j0), bz = std::min(sh.planes, nz - k0);
                                cover = cover && by >= 1 && bz >= 1;
                                for (int k = k0; k < k0 + bz; ++k)
                                    for (int j = j0; j < j0 + by; ++j) ++seen[(size_t)k * ny + j];
                            }
                            for (int v : seen) cover = cover && v == 1;
                            const int halo = res_halo(sh.cols * sh.planes) * kResThreads;
                            const size_t row = nx + 2, plane = (p.rby + 2) * row;
                            // the last row beside a brick, its cell's x + 1 neighbour
                            const size_t last = (sh.planes - 1) * plane + (p.rby + 1) * row + nx + 1;
                            bounds = bounds && p.rbz == sh.planes && sh.faces == faces &&
                                     (int64_t)nx * p.rby <= (int64_t)sh.cols * kResThreads &&
                                     (last + 1) * es <= p.lds && p.lds <= kResLds / (batch ? sh.batch : 1) &&
                                     2 * sh.planes * nx <= halo && halo <= 4096 && nx <= 4096 &&
                                     (size_t)p.bricks() * kResWords * 8 <= es * nx * ny * nz &&
                                     p.bricks() <= cap[p.shape];
                        }
            for (const pcg_grid_t g : { pcg_grid_t{ 1, 1, INT32_MAX, 1.0 }, pcg_grid_t{ 3072, 1, 699050, 1.0 },
                                        pcg_grid_t{ 1, 178956970, 12, 1.0 }, pcg_grid_t{ 512, 512, 512, 1.0 } })
                none = none && resident_plan(g, prec, pcg_opts_t{}, batch, false, shapes.data(), cap.data(), ns).shape < 0;
        }
    }
    for (uint32_t nx = 2; nx <= 4096; ++nx) {
        const uint32_t inv = ((1u << 24) + nx - 1u) / nx;
        for (uint32_t m = 0; m < 4096; ++m) exact = exact && (uint32_t)(((uint64_t)(m << 8) * inv) >> 32) == m / nx;
    }
    check(some && cover, "bricks: every cell in one");
    check(bounds, "bricks: within the kernel's bounds");
    check(none, "bricks: grids too large have none");
    check(exact, "bricks: the row of a value beside one");
}

}  // namespace

int main()
{
    bricks();
    tile_rules();
    columns();
    refinement_trips();
    left_the_chip();
    several_replays();
    std::printf("%d failed\n", failures);
    return failures != 0;
}
