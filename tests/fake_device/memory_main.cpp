// Driver of the CPU tests of the library's memory handling (tests/test_memory_cpu.py): the
// built library on the stand-in runtime of fake_hip.h.  One argument names the check; prints "ok".
#include <cstdio>
#include <cstring>
#include <functional>

#include "fake_hip.h"
#include "lbm3.h"

namespace tcg {
hipError_t pool_malloc(void** p, size_t bytes);
void pool_free(void* p);
void pool_trim();
size_t pool_kept();
}  // namespace tcg

using fake::device;

static int g_bad = 0;
#define CHECK(c)                                                       \
    do {                                                               \
        if (!(c)) {                                                    \
            std::printf("line %d: %s (%s)\n", __LINE__, #c, lbm3_last_error()); \
            ++g_bad;                                                   \
        }                                                              \
    } while (0)

static lbm3_params params(int nx, int ny, int precision = LBM3_FP64)
{
    lbm3_params p{};
    p.nx = nx;
    p.ny = ny;
    for (int k = 0; k < 3; ++k) p.rho0[k] = p.tau[k] = 1.0, p.sigma[k] = 0.01 + 0.001 * k;
    p.precision = precision;
    return p;
}
constexpr size_t MiB = (size_t)1 << 20, GiB = (size_t)1 << 30;

// What the pool keeps: blocks of 1 MiB and more, the smallest that fits and is not more than a
// quarter larger, at most 1/32 of the device in all, the oldest given back first
static void check_pool()
{
    auto get = [](size_t n) {
        void* p = nullptr;
        CHECK(tcg::pool_malloc(&p, n) == hipSuccess && p);
        return p;
    };
    void *a = get(2 * GiB), *b = get(3 * GiB), *c = get(MiB - 1), *d = get(5 * GiB);
    CHECK(device().used == 10 * GiB + MiB - 1);
    tcg::pool_free(c);  // too small to be kept
    CHECK(device().used == 10 * GiB && tcg::pool_kept() == 0);
    tcg::pool_free(b);
    tcg::pool_free(a);
    CHECK(device().used == 10 * GiB && tcg::pool_kept() == 5 * GiB);
    CHECK(get(2 * GiB - GiB / 4) == a);  // 2 GiB is less than a quarter more
    CHECK(get(2 * GiB) != b);            // 3 GiB is not
    CHECK(tcg::pool_kept() == 3 * GiB);
    tcg::pool_free(a);
    // 3 + 2 + 5 GiB pass the 9 GiB of a 288 GiB device: the oldest, b, goes back
    device().freed.clear();
    tcg::pool_free(d);
    CHECK(tcg::pool_kept() == 7 * GiB && device().freed.size() == 1 && device().freed[0] == 3 * GiB);
    // a block beyond the limit by itself is not kept and drives nothing out
    void* e = get(10 * GiB);
    tcg::pool_free(e);
    CHECK(tcg::pool_kept() == 7 * GiB && device().freed.back() == 10 * GiB);
    // a fresh allocation that finds no memory takes all of it back
    device().capacity = device().used + GiB;
    void* f = get(2 * GiB + GiB / 2 + GiB);
    CHECK(tcg::pool_kept() == 0);
    tcg::pool_free(f);
    CHECK(lbm3_release_cached() == LBM3_OK && tcg::pool_kept() == 0);
    tcg::pool_free(nullptr);
    tcg::pool_free((void*)1);  // not the pool's: ignored
}

// A use of the library from creation to destruction; false when a call failed
static bool lattice(int nx, int ny, int prec)
{
    lbm3_params p = params(nx, ny, prec);
    std::vector<double> rho((size_t)3 * nx * ny, 0.3), f((size_t)27 * nx * ny);
    lbm3_t* h = nullptr;
    lbm3_obs o;
    bool ok = lbm3_create(&p, nullptr, &h) == LBM3_OK && lbm3_init_fields(h, rho.data(), nullptr) == LBM3_OK &&
              lbm3_step(h, 5) == LBM3_OK && lbm3_observables(h, &o, rho.data(), f.data()) == LBM3_OK &&
              lbm3_set_tile(h, 64, 2) == LBM3_OK && lbm3_set_steps_per_launch(h, 2) == LBM3_OK &&
              lbm3_observables(h, &o, nullptr, nullptr) == LBM3_OK;
    lbm3_destroy(h);
    return ok;
}
static bool batch(int n, int prec)
{
    std::vector<lbm3_params> p(5, params(n, n + 3, prec));
    std::vector<double> rho((size_t)3 * n * (n + 3), 0.3);
    lbm3_batch_t* b = nullptr;
    lbm3_obs o;
    bool ok = lbm3_batch_create(p.data(), 5, nullptr, &b) == LBM3_OK;
    for (int i = 0; i < 5 && ok; ++i) ok = lbm3_batch_init_fields(b, i, rho.data(), nullptr) == LBM3_OK;
    ok = ok && lbm3_batch_step(b, 23) == LBM3_OK && lbm3_batch_observables(b, 3, &o, rho.data()) == LBM3_OK &&
         lbm3_batch_set_steps_per_launch(b, 2) == LBM3_OK && lbm3_batch_set_tile(b, 0, 64, 4) == LBM3_OK &&
         lbm3_batch_observables(b, 4, &o, rho.data()) == LBM3_OK;
    lbm3_batch_destroy(b);
    return ok;
}
static bool box(int n, int q, int prec)
{
    lbm3_params p = params(n, n, prec);
    std::vector<double> rho((size_t)3 * n * n * n, 0.3), f((size_t)3 * q * n * n * n);
    lbm3d_t* h = nullptr;
    lbm3d_obs o;
    bool ok = lbm3d_create_lattice(&p, n, q, nullptr, &h) == LBM3_OK && lbm3d_init_fields(h, rho.data()) == LBM3_OK &&
              lbm3d_step(h, 3) == LBM3_OK && lbm3d_observables(h, &o, rho.data(), f.data()) == LBM3_OK;
    lbm3d_destroy(h);
    return ok;
}
static bool gradient(int nx, int ny, int steps, int every)
{
    lbm3_params p = params(nx, ny);
    std::vector<double> rho((size_t)3 * nx * ny, 0.3), g((size_t)nx * ny, 0.1);
    double ds[3];
    lbm3_t* h = nullptr;
    bool ok = lbm3_create(&p, nullptr, &h) == LBM3_OK && lbm3_init_fields(h, rho.data(), nullptr) == LBM3_OK &&
              lbm3_adjoint_record(h, steps, every) == LBM3_OK && lbm3_adjoint(h, g.data(), ds, rho.data()) == LBM3_OK;
    lbm3_destroy(h);
    return ok;
}

// Whatever of the device's memory the pool keeps is there for every allocation of the library: a
// use that fits the device without the kept block fits with it, also where only its last
// allocation, or any before, finds no memory.
static void check_retry()
{
    const std::vector<std::function<bool()>> uses = {
        [] { return lattice(61, 47, LBM3_FP64); },  [] { return lattice(800, 700, LBM3_FP32); },
        [] { return batch(37, LBM3_FP32_STORAGE); }, [] { return batch(300, LBM3_FP64); },
        [] { return box(20, 19, LBM3_FP64); },       [] { return box(12, 27, LBM3_FP32_STORAGE); },
        [] { return gradient(40, 30, 12, 4); }};
    for (size_t u = 0; u < uses.size(); ++u) {
        device().capacity = 288 * GiB;
        tcg::pool_trim();
        const size_t before = device().used;
        device().peak = before;
        CHECK(uses[u]());
        tcg::pool_trim();
        const size_t need = device().peak - before;
        for (size_t part = 0; part <= 64; ++part) {
            device().capacity = 288 * GiB;
            void* p = nullptr;
            CHECK(tcg::pool_malloc(&p, GiB) == hipSuccess);
            tcg::pool_free(p);
            CHECK(tcg::pool_kept() == GiB);
            // (the device's total size is what it was: only the free part shrinks)
            const size_t free_b = part == 64 ? 0 : need - 1 - need * part / 64;
            void* ballast = nullptr;
            const size_t rest = device().capacity - device().used - free_b;
            CHECK(hipMalloc(&ballast, rest) == hipSuccess);
            const bool ok = uses[u]();
            if (!ok) std::printf("use %zu with %zu of %zu bytes free and 1 GiB kept\n", u, free_b, need);
            CHECK(ok);
            (void)hipFree(ballast);
            tcg::pool_trim();
            CHECK(device().used == before);
        }
    }
}

// Each runtime call of a reverse sweep failing in turn: an error is returned, no work is left on the
// sweep's streams (its workspace goes to another owner next, and the host arrays of its copies
// end with the call), and no event or memory is lost.
static void check_faults()
{
    const int nx = 24, ny = 20;
    std::vector<double> rho((size_t)3 * nx * ny, 0.3), g((size_t)nx * ny, 0.1);
    double ds[3];
    int failures = 0;
    for (int at = 0;; ++at) {
        lbm3_params p = params(nx, ny);
        lbm3_t* h = nullptr;
        CHECK(lbm3_create(&p, nullptr, &h) == LBM3_OK && lbm3_init_fields(h, rho.data(), nullptr) == LBM3_OK &&
              lbm3_adjoint_record(h, 6, 2) == LBM3_OK);
        CHECK(lbm3_adjoint(h, g.data(), ds, rho.data()) == LBM3_OK);  // the handle's streams are there
        CHECK(lbm3_init_fields(h, rho.data(), nullptr) == LBM3_OK && lbm3_adjoint_record(h, 6, 2) == LBM3_OK);
        const size_t events = device().events.size();
        device().calls = 0;
        device().fail_at = at;
        device().failed = false;
        const int rc = lbm3_adjoint(h, g.data(), ds, rho.data());
        const bool failed = device().failed;
        device().fail_at = -1;
        CHECK((rc != LBM3_OK) == failed);
        for (hipStream_t s : device().streams)
            if (device().pending.count(s)) {
                std::printf("call %d failed: work left on a stream of the sweep\n", at);
                ++g_bad;
            }
        CHECK(device().events.size() == events);
        lbm3_destroy(h);
        tcg::pool_trim();
        CHECK(device().used == 0 && device().events.empty() && device().streams.empty());
        if (!failed) break;
        ++failures;
    }
    CHECK(failures > 20);
}

int main(int argc, char** argv)
{
    const std::string what = argc > 1 ? argv[1] : "";
    if (what == "pool") check_pool();
    else if (what == "retry") check_retry();
    else if (what == "faults") check_faults();
    else ++g_bad;
    std::printf(g_bad ? "FAILED\n" : "ok\n");
    return g_bad != 0;
}
