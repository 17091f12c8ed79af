// Host-only check of what the library's runtime does when device memory runs short, on the
// scripted device of host_check.cpp with bounded memory (tests/hoststub_memory), built and
// run by tests/test_host_memory.py.
#define main host_check_main
#include "host_check.cpp"
#undef main

namespace {

// Open a trajectory of N^2, take one step, close it: the context keeps its memory.
void serve_one(rd_ctx *ctx, int N, rd_status pump_status = RD_OK) {
    const size_t n = (size_t)N * N;
    rd_problem p = ac(N);
    rd_opts o = opts(1e-3, RD_FP64);
    double *u = (double *)std::calloc(n, sizeof(double));
    rd_traj *t = nullptr;
    CHECK(rd_traj_open(ctx, &p, &o, u, nullptr, &t) == RD_OK);
    uint64_t tk = 0;
    CHECK(rd_traj_submit(t, 0.01, &tk) == RD_OK);
    rd_info info{};
    for (int k = 0; k < 100 && rd_poll(ctx, tk, &info) == RD_E_BUSY; ++k) CHECK(rd_serve_pump(ctx, 0) == pump_status);
    CHECK(rd_poll(ctx, tk, &info) == RD_OK && info.iters == model_iters(0.01, 1e-3));
    CHECK(rd_traj_read(t, u, nullptr) == RD_OK && all_equal(u, n, (double)info.iters));
    CHECK(rd_traj_close(t) == RD_OK);
    std::free(u);
}

// An allocation that failed and was made good, or that the call reported, is not the
// error of a later launch.
void failed_allocations_leave_no_error() {
    rd_ctx *ctx = nullptr;
    CHECK(rd_create(0, &ctx) == RD_OK);
    serve_one(ctx, 128);
    // no room but the kept memory: admission frees it and goes on
    const long before = hipmem::failures();
    hipmem::capacity() = hipmem::used() + 2 * 64 * 64 * sizeof(double);
    serve_one(ctx, 64);
    CHECK(hipmem::failures() > before && hipmem::last_error() == hipSuccess);
    // room for tables only: refused, and the next call is served
    hipmem::capacity() = hipmem::used() + 65536;
    rd_problem p = ac(64), big = ac(256);
    rd_opts o = opts(1e-3, RD_FP64);
    double *u = (double *)std::calloc(256 * 256, sizeof(double));
    rd_info info;
    CHECK(rd_step(ctx, &big, &o, 0.01, u, u, nullptr, &info) == RD_E_NOMEM);
    CHECK(hipmem::last_error() == hipSuccess);
    rd_traj *t = nullptr;
    CHECK(rd_traj_open(ctx, &big, &o, u, nullptr, &t) == RD_E_NOMEM && hipmem::last_error() == hipSuccess);
    // a trajectory that has to wait for another's memory does not disturb it
    hipmem::capacity() = (size_t)1 << 40;
    rd_traj *a = nullptr;
    uint64_t ta = 0, tb = 0;
    CHECK(rd_traj_open(ctx, &p, &o, u, nullptr, &a) == RD_OK && rd_traj_submit(a, 0.01, &ta) == RD_OK);
    CHECK(rd_traj_open(ctx, &big, &o, u, nullptr, &t) == RD_OK);
    CHECK(rd_serve_pump(ctx, 0) == RD_OK);
    CHECK(rd_traj_submit(t, 0.01, &tb) == RD_OK);
    hipmem::capacity() = hipmem::used();
    CHECK(rd_traj_submit(a, 0.01, &ta) == RD_OK);
    for (int k = 0; k < 100 && rd_poll(ctx, ta, &info) == RD_E_BUSY; ++k) CHECK(rd_serve_pump(ctx, 0) == RD_OK);
    CHECK(rd_poll(ctx, ta, &info) == RD_OK && rd_poll(ctx, tb, &info) == RD_E_BUSY);
    hipmem::capacity() = (size_t)1 << 40;
    for (int k = 0; k < 100 && rd_poll(ctx, tb, &info) == RD_E_BUSY; ++k) CHECK(rd_serve_pump(ctx, 0) == RD_OK);
    CHECK(rd_poll(ctx, tb, &info) == RD_OK);
    std::free(u);
    rd_destroy(ctx);
}

// Whatever a context needs memory for, it gets that of its closed trajectories: every call
// on a device that is full but for it succeeds as it does on an empty one.
void kept_memory_serves_every_call() {
    for (int call = 0; call < 8; ++call) {
        rd_ctx *ctx = nullptr;
        CHECK(rd_create(0, &ctx) == RD_OK);
        serve_one(ctx, 256);
        const int N = 128;
        rd_problem p = ac(N);
        rd_opts o = opts(1e-3, call == 4 ? RD_FP32_MIXED : RD_FP64);
        double *u = (double *)std::calloc((size_t)N * N, sizeof(double)), *v = (double *)std::calloc((size_t)N * N, 8);
        const size_t full = hipmem::used();
        hipmem::capacity() = full;
        rd_info info;
        if (call == 0 || call == 4) {
            CHECK(rd_step(ctx, &p, &o, 0.01, u, u, nullptr, &info) == RD_OK);
        } else if (call == 1) {
            rd_adapt a{};
            a.ht0 = 0.02;
            a.eta = 0.5;
            a.n_hi = 12;
            a.n_lo = 4;
            a.ht_min = 1e-9;
            a.max_rejects = 5;
            rd_adapt_info ai;
            CHECK(rd_advance(ctx, &p, &o, &a, 0.0, 0.1, u, nullptr, &ai, nullptr, nullptr, nullptr, 0) == RD_OK);
        } else if (call == 2) {
            CHECK(rd_precond_solve(ctx, &p, 0.01, RD_FP64, u, v, nullptr) == RD_OK);
        } else if (call == 3) {
            double res;
            CHECK(rd_residual(ctx, &p, 0.01, u, v, v, nullptr, &res) == RD_OK);
        } else if (call == 5) {
            serve_one(ctx, N);
        } else if (call == 6) {
            rd_traj *t = nullptr;
            CHECK(rd_traj_open(ctx, &p, &o, u, nullptr, &t) == RD_OK);
        } else {
            // the same shape again: nothing is given back, nothing new is needed
            hipmem::failures() = 0;
            serve_one(ctx, 256);
            CHECK(hipmem::failures() == 0 && hipmem::used() == full);
        }
        CHECK(hipmem::used() <= full && hipmem::last_error() == hipSuccess);
        hipmem::capacity() = (size_t)1 << 40;
        std::free(u);
        std::free(v);
        rd_destroy(ctx);
        CHECK(hipmem::used() == 0);
    }
}

// With a budget, admitted workspaces and kept memory together never exceed it, also while an
// admission allocates: served one after another, trajectories of several shapes need at most
// the budget beside their own states, tables and lists.
void kept_memory_stays_in_the_budget() {
    rd_ctx *ctx = nullptr;
    CHECK(rd_create(0, &ctx) == RD_OK);
    const int sizes[] = {64, 128, 256};
    for (int N : sizes) serve_one(ctx, N);   // tables, lists and streams of every size
    rd_opts o = opts(1e-3, RD_FP64);
    rd_problem big = ac(256);
    const size_t budget = rd_footprint_bytes(&big, &o);
    CHECK(rd_serve_set_budget(ctx, 1) == RD_OK);   // nothing kept
    const size_t base = hipmem::used();
    CHECK(rd_serve_set_budget(ctx, budget) == RD_OK);
    for (int r = 0; r < 12; ++r) {
        const int N = sizes[(r * 2 + r / 3) % 3];
        hipmem::peak() = hipmem::used();
        serve_one(ctx, N);
        CHECK(hipmem::peak() <= base + budget + (size_t)N * N * sizeof(double));
        CHECK(hipmem::used() <= base + budget);
    }
    // some is kept; setting the budget, also to the same or to none, gives it back
    for (size_t b : {budget, (size_t)0}) {
        CHECK(hipmem::used() > base);
        CHECK(rd_serve_set_budget(ctx, b) == RD_OK && hipmem::used() == base);
        serve_one(ctx, 128);
    }
    rd_destroy(ctx);
}

}  // namespace

int main() {
    kept_memory_stays_in_the_budget();
    failed_allocations_leave_no_error();
    kept_memory_serves_every_call();
    CHECK(hipmem::used() == 0);
    if (g_fail) {
        std::fprintf(stderr, "%d checks failed\n", g_fail);
        return 1;
    }
    std::printf("host memory checks passed\n");
    return 0;
}
