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

}  // namespace

int main() {
    failed_allocations_leave_no_error();
    CHECK(hipmem::used() == 0);
    if (g_fail) {
        std::fprintf(stderr, "%d checks failed\n", g_fail);
        return 1;
    }
    std::printf("host memory checks passed\n");
    return 0;
}
