// Host-side tile plans for the fused step (shared by the plain and batched forms).
#include <algorithm>

#include "lbm3_internal.h"

namespace tcg {

void plan_lattice(int inst, int nx, int ny, int threads, int rows, int elem_bytes,
                  std::vector<Tile>& out, int halo)
{
    const int wmax = threads - 2 * halo;
    const int nseg = std::max(1, (ny + std::max(rows, 1) - 1) / std::max(rows, 1));
    // Aligned strips: widths in units of A elements and strips starting at x = halo (mod A), so
    // that lane 0 of every wavefront (column x0 - halo + 64 w) sits on a unit boundary.  Used
    // when nx is a multiple of A and a unit-aligned strip width fits the workgroup.  The
    // single step takes 128-byte units (one cache line).  The two-step pass (halo 6) takes
    // units of four columns (32 bytes in FP64, 16 in FP32), which lets the strips fill the
    // device: at 4096 columns 17 strips of 240-244 columns give 255 workgroups for 256 CUs
    // (one per CU), where line-aligned strips of at most 240 columns need 18 strips and leave
    // 252 (measured: FP64 3.7% faster; FP32 storage 7% and FP32 5% faster than with
    // eight-column units).
    const int A = halo == 6 ? 4 : 128 / elem_bytes;
    const int wA = wmax / A * A;
    const bool aligned = nx % A == 0 && wA >= A && nx > 2 * halo;
    const int nstrips = aligned ? (nx / A + wA / A - 1) / (wA / A) : (nx + wmax - 1) / wmax;
    // strips (x0, cols) and segments (y0, rows)
    std::vector<int> sx0(nstrips), scols(nstrips), sy0(nseg), srows(nseg);
    int x0 = aligned ? halo : 0;
    for (int sx = 0; sx < nstrips; ++sx) {
        scols[sx] = aligned ? ((nx / A) / nstrips + (sx < (nx / A) % nstrips ? 1 : 0)) * A
                            : nx / nstrips + (sx < nx % nstrips ? 1 : 0);
        sx0[sx] = x0;
        x0 += scols[sx];
    }
    int y0 = 0;
    for (int sy = 0; sy < nseg; ++sy) {
        srows[sy] = ny / nseg + (sy < ny % nseg ? 1 : 0);
        sy0[sy] = y0;
        y0 += srows[sy];
    }
    // row of tiles after row of tiles: side-by-side tiles march the same rows at the same
    // time, so the halo columns they share are still in L2 when the second one reads them
    for (int sy = 0; sy < nseg; ++sy)
        for (int sx = 0; sx < nstrips; ++sx)
            if (srows[sy] > 0 && scols[sx] > 0) {
                Tile t{};
                t.inst = inst;
                t.x0 = sx0[sx];
                t.y0 = sy0[sy];
                t.rows = srows[sy];
                t.cols = scols[sx];
                out.push_back(t);
            }
}

void plan_blocks(int inst, int nx, int ny, int cmax, int rmax, std::vector<Tile>& out)
{
    const int nbx = (nx + cmax - 1) / cmax, nby = (ny + rmax - 1) / rmax;
    int y0 = 0;
    for (int by = 0; by < nby; ++by) {
        const int rows = ny / nby + (by < ny % nby ? 1 : 0);
        int x0 = 0;
        for (int bx = 0; bx < nbx; ++bx) {
            const int cols = nx / nbx + (bx < nx % nbx ? 1 : 0);
            Tile t{};
            t.inst = inst;
            t.x0 = x0;
            t.y0 = y0;
            t.rows = rows;
            t.cols = cols;
            out.push_back(t);
            x0 += cols;
        }
        y0 += rows;
    }
}

// Blocks of 8 rows of lanes while they are at most one per compute unit: the step's time is
// then that of one workgroup, whose four waves have a SIMD each (64^2 FP64: 5.0 us a step
// against 6.8 us with 16 rows, 128^2 5.3 against 7.0, FP32 4.4 against 5.3).  Beyond, 16 rows,
// which compute fewer halo nodes (256^2 FP64: 8.0 us against 8.9, 1024^2 FP32 26.7 against 31.5).
static BlockGrid grid_of(const KParams& kp, int lanes_x, int lanes_y, int halo)
{
    const int cmax = lanes_x - 2 * halo, rmax = lanes_y - 2 * halo;
    BlockGrid g{};
    g.kp = kp;
    g.lanes_x = lanes_x;
    g.lanes_y = lanes_y;
    g.nbx = (kp.nx + cmax - 1) / cmax;
    const int nby = (kp.ny + rmax - 1) / rmax;
    g.count = g.nbx * nby;
    g.inv = (uint32_t)((((uint64_t)1 << 32) + g.nbx - 1) / g.nbx);
    g.bw = kp.nx / g.nbx;
    g.rw = kp.nx % g.nbx;
    g.bh = kp.ny / nby;
    g.rh = kp.ny % nby;
    return g;
}

BlockGrid block_grid(const KParams& kp, int cus)
{
    const BlockGrid g = grid_of(kp, kBlockCols + 4, kBlockYSmall, 2);
    return g.count <= cus ? g : grid_of(kp, kBlockCols + 4, kBlockY, 2);
}

// A pass's time is that of one workgroup while there is at most one per compute unit, and grows
// with the workgroup's lanes (us per step, blocks of 16 x 16, 32 x 16, 32 x 24 and 32 x 32 lanes
// and single steps: FP64 96^2 3.8, 4.7, 6.5, 7.7 and 5.0; 160^2 6.5, 5.1, 6.7, 8.2 and 5.3; 256^2
// 13.0, 9.6, 7.1, 8.7 and 7.9; 320^2 18.3, 11.9, 12.3, 9.0 and 10.8; FP32 96^2 3.2, 3.6, 4.3, 5.1
// and 4.6; 256^2 8.2, 5.7, 5.1, 6.1 and 5.9; 320^2 11.1, 7.4, 6.6, 6.2 and 7.4).  More blocks than
// compute units, and single steps, whose blocks hold fewer halo nodes, are faster: 384^2 FP64 12.9
// at best and 11.7.
BlockGrid block_grid2(const KParams& kp, int cus)
{
    const int shapes[4][2] = {{16, 16}, {32, 16}, {32, 24}, {32, 32}};
    for (const auto& s : shapes) {
        const BlockGrid g = grid_of(kp, s[0], s[1], 5);
        if (g.count <= cus) return g;
    }
    return BlockGrid{};
}

std::vector<Tile> xcd_order(const std::vector<Tile>& L, int nxcd)
{
    const int T = (int)L.size();
    std::vector<Tile> out(T);
    std::vector<int> start(nxcd + 1, 0);
    for (int x = 0; x < nxcd; ++x) start[x + 1] = start[x] + (T - x + nxcd - 1) / nxcd;
    for (int b = 0; b < T; ++b) {
        const int x = b % nxcd, k = b / nxcd;
        out[b] = L[start[x] + k];
    }
    return out;
}

// A step reads one state buffer and writes the other at the same offsets at the same time.
// With the two an even number of MiB apart (what two separate allocations of a size that is
// a multiple of 2 MiB give), the FP64 two-step pass ran at 29.0k MLUPS at 4096^2; an odd
// number of MiB apart, at 30.0k, in every run (measured with distances of the buffer size
// plus 0, 64 KiB, 1, 2 and 3 MiB): the concurrent read and write streams then fall on
// different HBM channels.
hipError_t alloc_state_pair(size_t bytes, void* buf[2])
{
    constexpr size_t MiB = (size_t)1 << 20;
    const size_t off = (bytes + 2 * MiB - 1) / (2 * MiB) * (2 * MiB) + MiB;
    buf[0] = buf[1] = nullptr;
    void* base = nullptr;
    hipError_t e = device_malloc(&base, off + bytes);
    if (e != hipSuccess) return e;
    buf[0] = base;
    buf[1] = (char*)base + off;
    return hipSuccess;
}

void free_state_pair(void* buf[2])
{
    if (buf[0]) (void)hipFree(buf[0]);
    buf[0] = buf[1] = nullptr;
}

int auto_rows(int nx, int ny, int threads, int slots, int elem_bytes, int halo)
{
    std::vector<Tile> probe;
    plan_lattice(0, nx, 1, threads, 1, elem_bytes, probe, halo);
    const int nstrips = (int)probe.size();
    if (slots < 1) slots = 1;
    // time ~ rounds * (rows per segment + 2 halo warm-up rows: a step's pipeline is two
    // rows deep and its factored pull starts two source rows further down, six rows in
    // all, twelve for the two-step pass); fewest rounds, then fewest rows
    double best = 1e300;
    int best_rows = std::min(ny, 64);
    for (int nseg = 1; nseg <= ny; ++nseg) {
        const int rows = (ny + nseg - 1) / nseg;
        if (rows < 2 && nseg > 1) break;
        if (rows > 512) continue;
        const long tiles = (long)nstrips * nseg;
        const long rounds = (tiles + slots - 1) / slots;
        const double cost = (double)rounds * (rows + 2 * halo) * (1.0 + 1e-9 * nseg);
        if (cost < best) {
            best = cost;
            best_rows = rows;
        }
    }
    return best_rows;
}

int device_cus()
{
    int dev = 0, cus = 0;
    if (hipGetDevice(&dev) != hipSuccess) return 0;
    if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess) return 0;
    return cus;
}

int device_slots(Prec prec, int threads) { return blocks_per_cu(prec, threads) * device_cus(); }

int device_slots_pair(Prec prec, int threads)
{
    int per_cu = 0;
    if (prec == Prec::F64) per_cu = tiles_f64_pair_occupancy(threads);
    if (prec == Prec::F32) per_cu = tiles_f32_pair_occupancy(threads);
    if (prec == Prec::F32S) per_cu = tiles_f32s_pair_occupancy(threads);
    return per_cu * device_cus();
}

}  // namespace tcg
