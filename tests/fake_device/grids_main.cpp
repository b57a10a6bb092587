// Driver of the CPU test of the block grids (tests/test_memory_cpu.py): every node of a lattice in
// exactly one block, no block larger than its lanes allow, every workgroup a block of its own.
#include <cstdio>
#include <cstring>

#include "lbm3_internal.h"

using namespace tcg;

static int g_bad = 0;

static void check(const BlockGrid& g, int nx, int ny, int halo, int cus)
{
    const int cmax = g.lanes_x - 2 * halo, rmax = g.lanes_y - 2 * halo;
    std::vector<unsigned char> hit((size_t)nx * ny, 0);
    bool bad = g.count < 1;
    for (int wg = 0; wg < g.count && !bad; ++wg) {
        int x0, y0, cols, rows;
        g.block(wg, x0, y0, cols, rows);
        bad = cols < 1 || cols > cmax || rows < 1 || rows > rmax || x0 < 0 || y0 < 0 || x0 + cols > nx || y0 + rows > ny;
        for (int y = y0; y < y0 + rows && !bad; ++y)
            for (int x = x0; x < x0 + cols; ++x) ++hit[(size_t)y * nx + x];
    }
    for (unsigned char h : hit) bad |= h != 1;
    if (bad) {
        std::printf("%d x %d on %d compute units: %d blocks of %d x %d lanes\n", nx, ny, cus, g.count, g.lanes_x, g.lanes_y);
        ++g_bad;
    }
}

int main()
{
    const int sides[] = {1, 2, 3, 5, 6, 7, 22, 23, 27, 28, 29, 31, 56, 57, 61, 97, 112, 113, 256, 301, 352, 353, 448, 449, 1021, 1311};
    for (int cus : {256, 304, 64, 1, 0})
        for (int nx : sides)
            for (int ny : sides) {
                KParams kp{};
                kp.nx = nx;
                kp.ny = ny;
                const BlockGrid g = block_grid(kp, cus);
                check(g, nx, ny, 2, cus);
                if ((g.lanes_y == kBlockYSmall) != (g.count <= cus) && g.lanes_y == kBlockYSmall) ++g_bad;
                const BlockGrid g2 = block_grid2(kp, cus);
                if (g2.count > cus) ++g_bad;
                if (g2.count > 0) check(g2, nx, ny, 5, cus);
            }
    // the longest sides that blocks take: 7 x 2^18 nodes
    for (int n : {65535, 65534, 32767})
        for (int m : {1, 2, 27, 28}) {
            KParams kp{};
            kp.nx = n;
            kp.ny = m;
            check(block_grid(kp, 256), n, m, 2, 256);
            kp.nx = m;
            kp.ny = n;
            check(block_grid(kp, 256), m, n, 2, 256);
        }
    std::printf(g_bad ? "FAILED\n" : "ok\n");
    return g_bad != 0;
}
