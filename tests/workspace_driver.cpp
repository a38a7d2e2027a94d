// Drives the solver's workspaces and the device memory accounting on a
// host-side runtime (hip_host.h); the launches are counted, not run.
#include "hip_host.h"

#include "wcl_api.hip"
#include "wcl_solver.hip"

static int n_eo = 0, n_inv = 0;
int launch_eo_fields(const Geom&, int, const void*, const void*, const void*, double, double, void*, void*, void*,
                     size_t, int*, hipStream_t) {
    ++n_eo;
    return WCL_OK;
}
int launch_site_inverse(const Geom&, const void*, double, double, void*, void*, void*, int*, hipStream_t) {
    ++n_inv;
    return WCL_OK;
}

struct Fixture {
    wcl_ctx ctx{};
    Fixture(size_t budget = (size_t)-1 / 2) { ctx.budget = budget; }
    wcl_lattice* lattice(int L) {
        wcl_lattice* lat = nullptr;
        const int d[4] = {L, L, L, L};
        wcl_create_lattice(&ctx, d, nullptr, &lat);
        return lat;
    }
};

// A workspace serves several lattices.  When it cannot be grown for a larger
// one, what it held is gone: the smaller one's fields are built again, also
// where its buffers come back at the addresses that they had.
static int rebuilt_after_failed_growth() {
    const char* name = "rebuilt-after-failed-growth";
    Fixture fx;
    Workspace* ws = wcl_workspace_new(&fx.ctx);
    wcl_lattice *a = fx.lattice(4), *b = fx.lattice(8);
    EoFields f, f2;
    HOST_CHECK(name, eo_fields(a, ws, 0.1, 1.0, WCL_F32, true, nullptr, &f) == WCL_OK && n_eo == 1);
    HOST_CHECK(name, eo_fields(a, ws, 0.1, 1.0, WCL_F32, true, nullptr, &f) == WCL_OK && n_eo == 1);   // kept
    void *inv[3], *inv2[3];
    HOST_CHECK(name, site_inverse(a, ws, 0.1, 1.0, nullptr, inv) == WCL_OK && n_inv == 1);
    HOST_CHECK(name, site_inverse(a, ws, 0.1, 1.0, nullptr, inv) == WCL_OK && n_inv == 1);
    host::free_bytes = 0;
    HOST_CHECK(name, eo_fields(b, ws, 0.1, 1.0, WCL_F32, true, nullptr, &f2) == WCL_ENOMEM);
    HOST_CHECK(name, site_inverse(b, ws, 0.1, 1.0, nullptr, inv2) == WCL_ENOMEM);
    host::free_bytes = (size_t)1 << 40;
    HOST_CHECK(name, eo_fields(a, ws, 0.1, 1.0, WCL_F32, true, nullptr, &f2) == WCL_OK);
    HOST_CHECK(name, f2.ainv == f.ainv);   // the case in question
    HOST_CHECK(name, n_eo == 2);
    HOST_CHECK(name, site_inverse(a, ws, 0.1, 1.0, nullptr, inv2) == WCL_OK);
    HOST_CHECK(name, inv2[0] == inv[0]);
    HOST_CHECK(name, n_inv == 2);
    wcl_workspace_delete(ws);
    std::printf("ok %s\n", name);
    return 0;
}

int main() { return rebuilt_after_failed_growth(); }
