// Scheduling of the host engine, checked without a GPU (fake_device.h): each
// check prints its name and whether it held; the exit status counts failures.
#include "engine.cpp"

#include "fake_device.h"

namespace {

int failures = 0;

void check(bool ok, const char *what)
{
    std::printf("%s: %s\n", ok ? "ok" : "FAILED", what);
    std::fflush(stdout);
    failures += !ok;
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
    dev = Device();
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

}  // namespace

int main()
{
    refinement_trips();
    std::printf("%d failed\n", failures);
    return failures != 0;
}
