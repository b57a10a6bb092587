// Driver of the CPU tests of the library's choice of launches (tests/test_memory_cpu.py): the built
// library on the stand-in runtime of fake_hip.h.
//   clear            a shape set and cleared: the launches of a new handle again; prints "ok"
//   box nx ny nz q p the rows of lanes of the tiles that a box of precision p takes
#include <cstdio>
#include <cstdlib>
#include <cstring>

#include "fake_hip.h"
#include "lbm3.h"

using fake::device;

static int g_bad = 0;
#define CHECK(c)                                                                \
    do {                                                                        \
        if (!(c)) {                                                             \
            std::printf("line %d: %s (%s)\n", __LINE__, #c, lbm3_last_error()); \
            ++g_bad;                                                            \
        }                                                                       \
    } while (0)

static lbm3_params params(int nx, int ny, int precision)
{
    lbm3_params p{};
    p.nx = nx;
    p.ny = ny;
    for (int k = 0; k < 3; ++k) p.rho0[k] = p.tau[k] = 1.0, p.sigma[k] = 0.01;
    p.precision = precision;
    return p;
}

// The kernels of the last calls, without the first step's (from the 27 populations)
static std::vector<std::string> kernels(size_t from)
{
    std::vector<std::string> out;
    for (size_t i = from; i < device().launches.size(); ++i) out.push_back(device().launches[i].kernel);
    return out;
}
static bool all_of(const std::vector<std::string>& k, const char* name)
{
    for (const auto& s : k)
        if (s.find(name) == std::string::npos) return false;
    return !k.empty();
}

static void check_clear()
{
    for (int prec : {LBM3_FP64, LBM3_FP32_STORAGE, LBM3_FP32}) {
        const int nx = 97, ny = 64;
        std::vector<double> rho((size_t)3 * nx * ny, 0.3);
        lbm3_params p = params(nx, ny, prec);
        lbm3_t* h = nullptr;
        int t0 = 0, r0 = 0, t1 = 0, r1 = 0;
        CHECK(lbm3_create(&p, nullptr, &h) == LBM3_OK && lbm3_init_fields(h, rho.data(), nullptr) == LBM3_OK &&
              lbm3_step(h, 1) == LBM3_OK && lbm3_get_tile(h, &t0, &r0) == LBM3_OK);
        size_t n = device().launches.size();
        CHECK(lbm3_step(h, 4) == LBM3_OK && all_of(kernels(n), "k_block2"));
        CHECK(lbm3_set_tile(h, 256, 5) == LBM3_OK);
        n = device().launches.size();
        CHECK(lbm3_step(h, 4) == LBM3_OK && all_of(kernels(n), "k_tiles"));
        CHECK(lbm3_set_tile(h, 0, 0) == LBM3_EINVAL);  // as ever
        CHECK(lbm3_clear_tile(h) == LBM3_OK);
        n = device().launches.size();
        CHECK(lbm3_step(h, 4) == LBM3_OK && all_of(kernels(n), "k_block2"));
        CHECK(lbm3_get_tile(h, &t1, &r1) == LBM3_OK && t0 == t1 && r0 == r1);
        lbm3_destroy(h);

        std::vector<lbm3_params> ps(6, p);
        lbm3_batch_t* b = nullptr;
        CHECK(lbm3_batch_create(ps.data(), 6, nullptr, &b) == LBM3_OK);
        for (int i = 0; i < 6; ++i) CHECK(lbm3_batch_init_fields(b, i, rho.data(), nullptr) == LBM3_OK);
        CHECK(lbm3_batch_step(b, 1) == LBM3_OK);
        auto stepped = [&](const char* name) {
            n = device().launches.size();
            CHECK(lbm3_batch_step(b, 4) == LBM3_OK);
            std::vector<std::string> k;
            for (const auto& s : kernels(n))
                if (s.find("k_block") != std::string::npos || s.find("k_tiles") != std::string::npos) k.push_back(s);
            return all_of(k, name);
        };
        CHECK(stepped("k_block"));
        for (int side : {0, nx}) {
            CHECK(lbm3_batch_set_tile(b, side, 64, 8) == LBM3_OK && stepped("k_tiles"));
            CHECK(lbm3_batch_set_tile(b, 0, 0, 0) == LBM3_EINVAL);
            CHECK(lbm3_batch_clear_tile(b) == LBM3_OK && stepped("k_block"));
        }
        lbm3_batch_destroy(b);
    }
    CHECK(lbm3_clear_tile(nullptr) == LBM3_EINVAL && lbm3_batch_clear_tile(nullptr) == LBM3_EINVAL);
}

static void box(char** a)
{
    lbm3_params p = params(std::atoi(a[0]), std::atoi(a[1]), std::atoi(a[4]));
    const int nz = std::atoi(a[2]);
    std::vector<double> rho((size_t)3 * p.nx * p.ny * nz, 0.3);
    lbm3d_t* h = nullptr;
    CHECK(lbm3d_create_lattice(&p, nz, std::atoi(a[3]), nullptr, &h) == LBM3_OK && lbm3d_init_fields(h, rho.data()) == LBM3_OK);
    const size_t n = device().launches.size();
    CHECK(lbm3d_step(h, 2) == LBM3_OK && all_of(kernels(n), "k3_march"));
    std::printf("%u\n", device().launches.back().block / 32);
    lbm3d_destroy(h);
}

int main(int argc, char** argv)
{
    if (argc == 7 && !std::strcmp(argv[1], "box")) {
        box(argv + 2);
    } else {
        if (argc == 2 && !std::strcmp(argv[1], "clear")) check_clear();
        else ++g_bad;
        std::printf(g_bad ? "FAILED\n" : "ok\n");
    }
    return g_bad != 0;
}
