// Drives the solver's workspaces and the device memory accounting on a
// host-side runtime (hip_host.h); the launches are counted, not run.
#include "hip_host.h"

#include "wcl_api.hip"
#include "wcl_solver.hip"
#include "wcl_stage.cpp"
#include "wcl_server.cpp"

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
    n_eo = n_inv = 0;
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

// The even-odd fields and the site-term inverse of the Jacobi domain solver are
// kept from call to call, but a budget that holds either is enough for both in
// turn, and kept split links do not take the room of another call's fields.
static int kept_fields_give_way() {
    const char* name = "kept-fields-give-way";
    const int64_t V = 8 * 8 * 8 * 8;
    const size_t inverse = clover_bytes(WCL_F64, V) + clover_bytes(WCL_F32, V) + clover_bytes(WCL_F16, V);
    Fixture fx(inverse + 256);
    wcl_lattice* lat = fx.lattice(8);
    void* inv[3];
    EoFields f64, f32;
    for (int k = 0; k < 2; ++k) {
        HOST_CHECK(name, site_inverse(lat, lattice_ws(lat), 0.1, 1.0, nullptr, inv) == WCL_OK);
        Workspace* ws = lattice_ws(lat);
        HOST_CHECK(name, eo_fields(lat, ws, 0.1, 1.0, WCL_F64, false, nullptr, &f64) == WCL_OK);
        HOST_CHECK(name, eo_fields(lat, ws, 0.1, 1.0, WCL_F32, true, nullptr, &f32) == WCL_OK);
        HOST_CHECK(name, host::blocks.count(f64.ainv) && host::blocks.count(f64.clov));   // this call's own stay
    }
    // with room for split links they are made; a later call gets their room
    fx.ctx.budget = inverse + 256 + 2 * gauge_bytes(WCL_F64, V / 2) + 16 * spinor_rhs_bytes(WCL_F64, V);
    EoFields g;
    HOST_CHECK(name, eo_fields(lat, lattice_ws(lat), 0.1, 1.0, WCL_F64, true, nullptr, &g) == WCL_OK && g.links);
    void* v = nullptr;
    const size_t rest = fx.ctx.budget - clover_bytes(WCL_F64, V) - 256;   // all but A^{-1} and C of this call
    Workspace* ws = lattice_ws(lat);
    HOST_CHECK(name, eo_fields(lat, ws, 0.1, 1.0, WCL_F64, false, nullptr, &f64) == WCL_OK);
    HOST_CHECK(name, ws->get("vectors", rest, &v) == WCL_OK);
    HOST_CHECK(name, ws->get("more", 256, &v) == WCL_ENOMEM);
    HOST_CHECK(name, host::blocks.count(f64.ainv) && host::blocks.count(f64.clov));
    wcl_free_workspace(lat);
    HOST_CHECK(name, fx.ctx.in_use == 0);
    std::printf("ok %s\n", name);
    return 0;
}

// A transfer's staging is charged what the transfer needs, also when a larger
// idle block is at hand: another thread's allocation that fits the budget
// beside it is not refused.
static int small_staging_beside_idle_block() {
    const char* name = "small-staging-beside-idle-block";
    const size_t M = (size_t)1 << 20;
    Fixture fx(200 * M);
    void *p = nullptr, *big = nullptr, *other = nullptr;
    HOST_CHECK(name, wcl_stage_alloc(&fx.ctx, &big, 75 * M) == WCL_OK);   // a large upload leaves its block
    wcl_stage_free(&fx.ctx, big, 75 * M, true);
    HOST_CHECK(name, fx.ctx.in_use == 0);
    HOST_CHECK(name, wcl_stage_alloc(&fx.ctx, &p, 2 * M) == WCL_OK);      // a small one
    HOST_CHECK(name, wcl_dev_alloc(&fx.ctx, &other, 190 * M) == WCL_OK);  // meanwhile
    wcl_dev_free(&fx.ctx, other, 190 * M);
    wcl_stage_free(&fx.ctx, p, 2 * M, true);
    HOST_CHECK(name, fx.ctx.in_use == 0 && host::blocks.size() == 1);     // the 75 MiB gave way
    // two sizes in turn: each block serves its own size again
    HOST_CHECK(name, wcl_stage_alloc(&fx.ctx, &big, 75 * M) == WCL_OK);
    wcl_stage_free(&fx.ctx, big, 75 * M, true);
    for (int k = 0; k < 4; ++k) {
        void* q = nullptr;
        const size_t n = k % 2 ? 75 * M : 2 * M;
        HOST_CHECK(name, wcl_stage_alloc(&fx.ctx, &q, n) == WCL_OK && q == (k % 2 ? big : p));
        HOST_CHECK(name, fx.ctx.in_use == n);
        wcl_stage_free(&fx.ctx, q, n, true);
    }
    // never more than two, nor more than 128 MiB
    for (size_t n : {3 * M, 4 * M, 100 * M, 60 * M, 129 * M}) {
        HOST_CHECK(name, wcl_stage_alloc(&fx.ctx, &p, n) == WCL_OK);
        wcl_stage_free(&fx.ctx, p, n, true);
        size_t sum = 0;
        for (auto& kv : host::blocks) sum += kv.second;
        HOST_CHECK(name, host::blocks.size() <= 2 && sum <= 128 * M && fx.ctx.in_use == 0);
    }
    // they give way when idle, and an allocation past the budget is refused
    HOST_CHECK(name, wcl_dev_alloc(&fx.ctx, &other, 200 * M) == WCL_OK && host::blocks.size() == 1);
    HOST_CHECK(name, wcl_stage_alloc(&fx.ctx, &p, M) == WCL_ENOMEM);
    wcl_dev_free(&fx.ctx, other, 200 * M);
    std::printf("ok %s\n", name);
    return 0;
}

// A call that fails hands its staging block back only when nothing queued can
// still use it: the next call may take the block at once, on another stream.
static bool fail_pack = false;
int launch_pack_clover(const Geom&, const double*, void*, void*, void*, hipStream_t) {
    return fail_pack ? WCL_EHIP : WCL_OK;
}
static int failed_call_leaves_no_work() {
    const char* name = "failed-call-leaves-no-work";
    Fixture fx;
    wcl_lattice* lat = fx.lattice(4);
    lat->has_gauge = true;
    void* pinned = nullptr;   // a pinned source is copied asynchronously
    const size_t n = (size_t)lat->V * 72;
    hipHostMalloc(&pinned, n * sizeof(double), 0);
    std::memset(pinned, 0, n * sizeof(double));
    fail_pack = true;
    HOST_CHECK(name, wcl_upload_clover(lat, (const double*)pinned) == WCL_EHIP);
    for (auto& kv : host::queues) HOST_CHECK(name, kv.second.done == kv.second.work.size());
    fail_pack = false;
    HOST_CHECK(name, wcl_upload_clover(lat, (const double*)pinned) == WCL_OK);
    std::printf("ok %s\n", name);
    return 0;
}

// A request that fails is reported only when nothing queued reads its source
// any more: the caller may free it then.
int launch_pack_spinor(const Geom&, int, int, const double*, void*, size_t, hipStream_t) {
    return fail_pack ? WCL_EHIP : WCL_OK;
}
static int failed_request_releases_source() {
    const char* name = "failed-request-releases-source";
    Fixture fx;
    int handle = 0;
    wcl_server srv;
    srv.ctx = &fx.ctx;
    wcl_server::Slot slot;
    slot.st = (hipStream_t)&handle;
    slot.ws = wcl_workspace_new(&fx.ctx);
    Job j;
    j.lat = fx.lattice(4);
    void* pinned = nullptr;
    hipHostMalloc(&pinned, (size_t)j.lat->V * 24 * sizeof(double), 0);
    j.req.eta_host = j.req.phi_host = (double*)pinned;
    slot.jobs.push_back(j);
    fail_pack = true;
    srv.run_job(&slot);
    fail_pack = false;
    HOST_CHECK(name, srv.done.size() == 1 && srv.done.begin()->second.status == WCL_EHIP);
    host::Queue& q = host::queue(slot.st);
    HOST_CHECK(name, !q.work.empty() && q.done == q.work.size());
    wcl_workspace_delete(slot.ws);
    std::printf("ok %s\n", name);
    return 0;
}

int main() {
    return kept_fields_give_way() || failed_request_releases_source() || rebuilt_after_failed_growth() || small_staging_beside_idle_block() || failed_call_leaves_no_work();
}
