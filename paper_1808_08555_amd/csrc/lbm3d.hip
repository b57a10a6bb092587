// The three-dimensional form of the ternary step: the paper's model (Sec. 2) on the standard
// D3Q19 or D3Q27 lattice, the force of Eq. (7) with Guo's term, any segregation law, in
// FP64, FP32, or FP32 storage with FP64 arithmetic (stochastic rounding on store).
//
// State: factored per node, Q + 9 values before streaming: f_dag_i (Q), c_k (3), V_0 and V_1
// (3 each; V_2 = -(V_0 + V_1)), from which Eq. (13) gives every recoloured population,
// f_ddag_{i,k} = c_k f_dag_i + w_i V_k . e_i.  Two buffers (read one, write the other), 28
// values per node for D3Q19 and 36 for D3Q27 in place of the 57 and 81 populations; with FP32
// storage one word more, further bits of the c_k (split_c).  A freshly
// initialised lattice holds its three densities instead (FP64, at the start of the first buffer);
// the first step reads those.
//
// A step is one launch of the fused march (k3_march): workgroups own x-y blocks of a z
// segment and march up z.  What a node's densities need of its neighbours' factored values
// splits by source plane, and so does the divergence of the stress, so that one plane of
// c_k and V_k and one plane of stress in LDS serve the whole step; every sum that spans planes
// is carried in registers from plane to plane.
#include <algorithm>
#include <cmath>
#include <new>
#include <vector>

#include "lbm3_device.h"
#include "lbm3_handle.h"
#include "lbm3_rounding.h"

namespace tcg {
namespace {

// Links: rest, six axis links, twelve edge links (the D3Q19 lattice ends here), eight corner
// links (D3Q27); link i odd and i + 1 are opposite.  c_s^2 = 1/3 on both.  D3Q19 weights 1/3,
// 1/18, 1/36; D3Q27 weights 8/27, 2/27, 1/54, 1/216.  In FP32 the nearest floats sum to
// 1 + 1.5e-8 (D3Q19) and 1 + 7.5e-9 (D3Q27), and every collision would scale the mass by that
// sum (the equilibrium's zeroth moment); the float weights are therefore chosen one ulp off
// where needed so that their sum is exactly 1: D3Q19 one ulp above 1/3 and one ulp below
// 1/18 and 1/36; D3Q27 one ulp below 8/27 and one ulp above 1/54.
constexpr int L3X[27] = {0, 1, -1, 0, 0, 0, 0, 1, -1, 1, -1, 1, -1, 1, -1, 0, 0, 0, 0, 1, -1, 1, -1, 1, -1, -1, 1};
constexpr int L3Y[27] = {0, 0, 0, 1, -1, 0, 0, 1, -1, -1, 1, 0, 0, 0, 0, 1, -1, 1, -1, 1, -1, 1, -1, -1, 1, 1, -1};
constexpr int L3Z[27] = {0, 0, 0, 0, 0, 1, -1, 0, 0, 0, 0, 1, -1, -1, 1, 1, -1, -1, 1, 1, -1, -1, 1, 1, -1, 1, -1};
template <typename C, int Q>
__device__ __forceinline__ C w3(int i)
{
    static_assert(Q == 19 || Q == 27, "D3Q19 or D3Q27");
    if constexpr (Q == 19) {
        if constexpr (sizeof(C) == 8)
            return i == 0 ? 1.0 / 3.0 : (i <= 6 ? 1.0 / 18.0 : 1.0 / 36.0);
        else
            return i == 0 ? 0x1.555558p-2f : (i <= 6 ? 0x1.c71c70p-5f : 0x1.c71c70p-6f);
    } else {
        if constexpr (sizeof(C) == 8)
            return i == 0 ? 8.0 / 27.0 : (i <= 6 ? 2.0 / 27.0 : (i <= 18 ? 1.0 / 54.0 : 1.0 / 216.0));
        else
            return i == 0 ? 0x1.2f684ap-2f : (i <= 6 ? 0x1.2f684cp-4f : (i <= 18 ? 0x1.2f684ep-6f : 0x1.2f684cp-8f));
    }
}
constexpr int PK3[3] = {0, 0, 1}, PL3[3] = {1, 2, 2};

struct Geo3 {
    int nx, ny, nz;
    int64_t N;
    int64_t zbytes;  // bytes of one z plane of a factored state
};

// Layout of a factored state.  The nodes of a z plane, in order y nx + x, form groups of 128
// bytes' worth (16 FP64, 32 FP32); a group holds value after value, one 128-byte line each, and
// groups and planes follow one another.  All values of a node are then at constant
// distances, so a plane's Q loads share one base address in scalar registers and one offset per
// lateral neighbour, with the value in the instruction (separate planes of values cost
// four scalar and one 64-bit vector instruction per access to form the address).
constexpr int kLine = 128;
template <typename S>
constexpr int64_t group3()
{
    return kLine / (int64_t)sizeof(S);
}
// byte offset of node n = y nx + x of a z plane
template <typename S, int NV, typename Off>
__host__ __device__ __forceinline__ Off node_off3(int64_t n)
{
    const int64_t G = group3<S>();
    return (Off)(n / G) * (Off)(NV * kLine) + (Off)(n % G) * (Off)sizeof(S);
}
template <typename S>
int64_t zbytes3(int nx, int ny, int nv)
{
    return ((int64_t)nx * ny + group3<S>() - 1) / group3<S>() * nv * kLine;
}
// values of a node: f_dag_i (Q), c_k (3), V_0 and V_1 (6) and, where stores round, the word of
// the c_k's further bits
template <typename S, typename C, int Q>
constexpr int kVals3 = Q + 9 + (kRounds<S, C> ? 1 : 0);
inline int vals3(Prec prec, int q) { return q + 9 + (prec == Prec::F32S ? 1 : 0); }

// With FP32 storage of FP64 arithmetic a c_k keeps the ten mantissa bits after a float's 23 as
// well, the three of a node in one word (bits 10 k to 10 k + 9).  One c_k multiplies the f_dag_i of
// every link: rounded to a float, its error would pass to a density whole, where those of
// 3 Q populations, rounded one by one, average.  Split in two: the float toward zero, and the
// bits; both of the value rounded stochastically to 33 mantissa bits (as round_stochastic, whose
// notes on zero, Inf and NaN hold; below the smallest normal float the further bits change a
// value by no more than the float's own last place).  RMS error of the densities against FP64,
// 3 Q populations, c_k in floats, and with the bits: random mixture 20^3 after 10 steps D3Q19
// 1.5e-8, 2.5e-8, 1.3e-8, D3Q27 1.7e-8, 2.5e-8, 1.4e-8; two spheres after 100 3.0e-8, 4.2e-8,
// 2.8e-8 and 3.1e-8, 3.5e-8, 2.9e-8.  Us per step at 128^3 without the bits and with them: D3Q19
// 217 and 220, D3Q27 268 and 276.
__device__ __forceinline__ float split_c(double v, uint32_t bits, int k, uint32_t& word)
{
    const uint64_t s = (uint64_t)__double_as_longlong(v) + (uint64_t)(bits >> 13);
    word |= ((uint32_t)(s >> 19) & 0x3ffu) << (10 * k);
    return (float)__longlong_as_double((long long)(s & ~((1ull << 29) - 1ull)));
}
__device__ __forceinline__ double join_c(float hi, uint32_t word, int k)
{
    const uint64_t u = (uint64_t)__double_as_longlong((double)hi);
    return __longlong_as_double((long long)(u | (uint64_t)((word >> (10 * k)) & 0x3ffu) << 19));
}

// A 32-bit lane offset is made new to the optimiser at each use (lbm3_device.h); a 64-bit one is
// used as it is.
__device__ __forceinline__ void refresh(uint64_t&) {}
// Has x computed here: a sum that only the next iteration reads would be moved to the end of
// this one, with everything that it is made of kept in registers till then.
template <typename C>
__device__ __forceinline__ void settle(C& x) { asm volatile("" : "+v"(x)); }

// Value `v` (a constant) at byte offset `off` of the plane at the uniform address `base`.  The
// instruction's offset is 13 bits with sign: the base is taken 16 values up.
template <typename S, typename Off>
__device__ __forceinline__ S ld_value(uint64_t base, Off off, int v)
{
    typedef const __attribute__((address_space(1))) char gchar;
    typedef const __attribute__((address_space(1))) S gS;
    return *(gS*)((gchar*)(base + 16 * kLine) + off + (v - 16) * kLine);
}
template <typename S, typename Off>
__device__ __forceinline__ void st_value(uint64_t base, Off off, int v, S x)
{
    typedef __attribute__((address_space(1))) char gchar;
    typedef __attribute__((address_space(1))) S gS;
    *(gS*)((gchar*)(base + 16 * kLine) + off + (v - 16) * kLine) = x;
}

// The node indices of (x, y, z) and its neighbours: the wrapped coordinates at offsets -1,
// 0, +1 per axis, formed once per node (no division per neighbour).
struct Nb3 {
    int64_t zo[3], yo[3];
    int xo[3];
    __device__ __forceinline__ Nb3(const Geo3& g, int x, int y, int z)
    {
        xo[0] = x == 0 ? g.nx - 1 : x - 1, xo[1] = x, xo[2] = x == g.nx - 1 ? 0 : x + 1;
        const int y0 = y == 0 ? g.ny - 1 : y - 1, y2 = y == g.ny - 1 ? 0 : y + 1;
        const int z0 = z == 0 ? g.nz - 1 : z - 1, z2 = z == g.nz - 1 ? 0 : z + 1;
        yo[0] = (int64_t)y0 * g.nx, yo[1] = (int64_t)y * g.nx, yo[2] = (int64_t)y2 * g.nx;
        const int64_t pl = (int64_t)g.nx * g.ny;
        zo[0] = z0 * pl, zo[1] = z * pl, zo[2] = z2 * pl;
    }
    // the node at offset (dx, dy, dz), each in -1..1
    __device__ __forceinline__ int64_t at(int dx, int dy, int dz) const { return zo[dz + 1] + yo[dy + 1] + xo[dx + 1]; }
};

// e_i . (a0, a1, a2) over the nonzero components of link i (each +-1), added in x, y, z
// order.  A zero component would only add an exact zero, so this is the value of the full
// sum (up to the sign of a zero result) without the products by zero, which floating point
// cannot drop by itself.
template <typename C>
__device__ __forceinline__ C edot(int i, C a0, C a1, C a2)
{
    const int e[3] = {L3X[i], L3Y[i], L3Z[i]};
    const C a[3] = {a0, a1, a2};
    C r = C(0);
    bool any = false;
#pragma unroll
    for (int c = 0; c < 3; ++c)
        if (e[c] != 0) {
            const C v = e[c] > 0 ? a[c] : -a[c];
            r = any ? r + v : v;
            any = true;
        }
    return r;
}

// Eq. (12) over the (Q - 1)/2 pairs of opposite links: 3 sum_i w_i e_i [phi(x + e_i) -
// phi(x - e_i)], phi(dx, dy, dz) the field at offset (dx, dy, dz) from the node (zero
// components of e_i skipped, as in edot); the differences of a weight class are added before
// they are weighted
template <typename C, int Q, typename Get>
__device__ __forceinline__ void grad3(Get phi, C (&d)[3])
{
    C a[3], e[3] = {C(0), C(0), C(0)}, c[3] = {C(0), C(0), C(0)};
#pragma unroll
    for (int i = 1; i < Q; i += 2) {
        const C df = phi(L3X[i], L3Y[i], L3Z[i]) - phi(-L3X[i], -L3Y[i], -L3Z[i]);
        const int v[3] = {L3X[i], L3Y[i], L3Z[i]};
#pragma unroll
        for (int q = 0; q < 3; ++q) {
            if (v[q] == 0) continue;
            if (i < 7) a[q] = df;  // the links +x, +y, +z
            else if (i < 19) e[q] += v[q] > 0 ? df : -df;
            else c[q] += v[q] > 0 ? df : -df;
        }
    }
    const C wa = C(3) * w3<C, Q>(1), we = C(3) * w3<C, Q>(7);
#pragma unroll
    for (int q = 0; q < 3; ++q) {
        d[q] = fma(wa, a[q], we * e[q]);
        if constexpr (Q == 27) d[q] = fma(C(3) * w3<C, Q>(19), c[q], d[q]);
    }
}

// Eq. (12)'s weighted differences of a vector field v over one plane of nodes, split by the
// plane they serve: sum_i w_i e_i . v(x + e_i) at a node of the plane itself takes M from it, at
// the node below (the plane is its e_z = +1 neighbour) P + Z, at the node above P - Z.
// v(a, ox, oy): component a at lateral offset (ox, oy).  Opposite neighbours are subtracted
// first, so data symmetric about the node give exact zeros.
template <typename C, int Q, typename Get>
__device__ __forceinline__ void plane_div(Get v, C& M, C& P, C& Z)
{
    const C wa = w3<C, Q>(1), we = w3<C, Q>(7);
    const C axis = (v(0, 1, 0) - v(0, -1, 0)) + (v(1, 0, 1) - v(1, 0, -1));
    const C diag = ((v(0, 1, 1) - v(0, -1, -1)) + (v(0, 1, -1) - v(0, -1, 1))) +
                   ((v(1, 1, 1) - v(1, -1, -1)) + (v(1, -1, 1) - v(1, 1, -1)));
    M = wa * axis + we * diag;
    P = we * axis;
    Z = wa * v(2, 0, 0) + we * ((v(2, 1, 0) + v(2, -1, 0)) + (v(2, 0, 1) + v(2, 0, -1)));
    if constexpr (Q == 27) {
        const C wc = w3<C, Q>(19);
        P += wc * diag;
        Z += wc * ((v(2, 1, 1) + v(2, -1, -1)) + (v(2, 1, -1) + v(2, -1, 1)));
    }
}

// Stress T = sum_pairs sigma C (|G|^2 I - G G^T)/|G| (xx, xy, xz, yy, yz, zz; Eq. 7 with C_kl
// of Eq. 6) and the recolouring vectors V_0, V_1 (V[3k + a]; Eq. 13 with the segregation law,
// V_k = sum_{l != k} beta_kl (rho_k rho_l / rho) n_kl) of a node from its concentrations cc,
// their gradients gc and its densities rk.
template <typename C>
__device__ __forceinline__ void stress3(const C (&gc)[3][3], const C (&cc)[3], const C (&rk)[3], const KParams& kp,
                                        C (&t)[6], C (&V)[6])
{
    C ct = C(kp.ct_coef) * (cc[0] * cc[1] * cc[2]);
    ct = ct < C(1) ? ct : C(1);
    C an[3][3];  // a_p n_p with a_p = beta_p rho_k rho_l / rho
#pragma unroll
    for (int q = 0; q < 6; ++q) t[q] = C(0);
#pragma unroll
    for (int p = 0; p < 3; ++p) {
        const int k = PK3[p], l = PL3[p];
        C G[3], xx, yy, zz;
        {
            // the products of G nearly cancel where a fluid is present only as a trace; their
            // rounding is left as the plain evaluation's
#pragma clang fp contract(off)
#pragma unroll
            for (int a = 0; a < 3; ++a) G[a] = cc[l] * gc[k][a] - cc[k] * gc[l][a];
            xx = G[0] * G[0];
            yy = G[1] * G[1];
            zz = G[2] * G[2];
        }
        const C g2 = (xx + yy) + zz;
        // zero at or below the guard (selected, not branched over: the three pairs' chains of
        // dependent operations then run beside one another)
        const C inv = g2 > C(kp.guard * kp.guard) ? rsqrt_nr(g2) : C(0);
        const C a_p = fma(ct, C(kp.beta0 * kp.g[p]), C(kp.beta0)) * (rk[k] * cc[l]) * inv;
#pragma unroll
        for (int a = 0; a < 3; ++a) an[p][a] = a_p * G[a];
        C cf = C(kp.cfac[p]) * (rk[k] * rk[l]);
        cf = cf < C(1) ? cf : C(1);
        const C s = C(kp.sigma[p]) * cf * inv;
        t[0] += s * (yy + zz);
        t[1] -= s * (G[0] * G[1]);
        t[2] -= s * (G[0] * G[2]);
        t[3] += s * (xx + zz);
        t[4] -= s * (G[1] * G[2]);
        t[5] += s * (xx + yy);
    }
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        V[a] = an[0][a] + an[1][a];
        V[3 + a] = an[2][a] - an[0][a];
    }
}

// Collision with Guo's term (Eqs. 1-3, 8-11) of one node from its density rho, 1/tau, totals
// ft, force F and half-force velocity u: f_dag_i = (1 - 1/tau) f_i + (1/tau) f_eq_i + Phi_i, each
// handed to put(i, value).  With A = (1/tau) w rho and B = w (1 - 1/(2 tau)) of a weight class,
//   (1/tau) f_eq_i + Phi_i = [A (1 - 1.5 u.u) - 3 B u.F] + e.u e.(4.5 A u + 9 B F) + e.(3 A u + 3 B F):
// the first two terms are the same for a link and its opposite, the last changes sign, so
// each pair of links forms them once (half the operations of forming them per link).
template <typename C, int Q, typename Put>
__device__ __forceinline__ void collide3(C rho, C itau, const C (&ft)[Q], const C (&F)[3], const C (&u)[3], Put put)
{
    const C uu = u[0] * u[0] + u[1] * u[1] + u[2] * u[2];
    const C uF = u[0] * F[0] + u[1] * F[1] + u[2] * F[2];
    const C omi = C(1) - itau, c0 = C(1) - C(1.5) * uu, tr = itau * rho, pref = C(1) - C(0.5) * itau;
    const C s0 = tr * c0 - C(3) * pref * uF;  // the symmetric part without the weight and e
    C X[3], Y[3];  // 4.5 A u + 9 B F and 3 A u + 3 B F without the weight
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        const C tu = tr * u[a], pF = pref * F[a];
        X[a] = C(4.5) * tu + C(9) * pF;
        Y[a] = C(3) * tu + C(3) * pF;
    }
    put(0, fma(ft[0], omi, w3<C, Q>(0) * s0));
#pragma unroll
    for (int i = 1; i < Q; i += 2) {
        const C w = w3<C, Q>(i);
        const C E = w * fma(edot<C>(i, u[0], u[1], u[2]), edot<C>(i, X[0], X[1], X[2]), s0);
        const C O = w * edot<C>(i, Y[0], Y[1], Y[2]);
        put(i, fma(ft[i], omi, E + O));
        put(i + 1, fma(ft[i + 1], omi, E - O));
    }
}

// ---- the fused step: one kernel per step, marching along z
// A workgroup of TX x TY lanes (lane t at tile column t % TX, tile row t / TX; each wave is
// two whole tile rows) owns the output nodes [x0, x0 + cols) x [y0, y0 + rows) x
// [z0, z0 + depth), cols <= TX - 4 and rows <= TY - 4.  Lane (tx, ty) sits on node column
// (x0 - sx + tx, y0 - 2 + ty) (wrapped), sx = 2 or 3.  Iteration j takes source plane s = z0 - 3 + j, two
// barriers:
//   stage 1 (lanes within two columns and rows of the owned ones): the densities that plane s streams to planes
//            s + 1, s and s - 1, from the lane's f_dag_i(x - e_i) of plane s and the c_k, V_k of
//            plane s in LDS (one ring of nodes beyond the lanes').  sum_i w_i e_i . V_k(x - e_i)
//            is plane_div of V_k.  Plane s - 1 is then complete; its c_k go into a
//            three-plane LDS ring.
//   stage 2, plane s - 2 (lanes within one): grad c_k (Eq. 12) from the ring,
//            stress into LDS, V_k; the owned nodes store c_k, V_0, V_1.  The next plane's c_k,
//            V_k go into LDS.
//   stage 3, plane s - 3 (the owned nodes' lanes): the stress of plane s - 2 completes
//            F = div T; collision, f_dag_i stored.
// The totals f_i = f_dag_i(x - e_i) (the c_k sum to 1 and the V_k to 0) are used in stage 3,
// three iterations later.  Each owning lane keeps in LDS those of as many links as fit
// (Hold3: 9 of 19 in FP64, 16 with FP32 storage, 14 in FP32) and loads the others again: all
// would take 4 Q values per node (three planes waiting and one arriving), more than registers
// and LDS have.  Loading all again cost, D3Q19 128^3: FP64 344 us a step against 325, FP32 storage
// 242 against 226, FP32 199 against 180.
// Global loads are issued up to an iteration before their use, into the registers that their
// previous values have just left (D3Q27 in FP64 issues its f_dag_i after stage 2, so that
// they are not in registers beside stage 2's: no spills, 735 -> 462 us at 128^3).
// What bounds it: memory, bytes and path.  A D3Q19 FP64 step at 128^3 moves 1.41 GB, 1.50 times what
// it needs, at 4.6 TB/s, 74% of a large copy's rate.  It takes 142 us without its loads and
// stores; the stores alone add 109 us, the loads' path through L1 most of the rest (about 15
// cycles per wave instruction, whatever its width).  Measured against the march over 3 Q stored
// populations that it replaced, us per step at 128^3 (FP64 / FP32 storage / FP32): D3Q19 723 /
// 413 / 338 -> 310 / 222 / 193, D3Q27 1159 / 667 / 460 -> 430 / 277 / 250; 48^3 D3Q19 FP64 63 -> 37 (34 with the
// small tiles).
// Non-temporal stores made it 1-15% slower, non-temporal loads 10-20%.
// The arithmetic of every node has a fixed order, so the result does not depend on the tile
// shape.  RMS error of the densities against that of the march over 3 Q populations, mean ratio
// over 48 drawn boxes after 20, 100 and 300 steps: FP32 D3Q19 0.29, 0.89 and 0.97, D3Q27 0.17, 0.56
// and 0.79; FP64 (random mixture and spheres, against 80 bits) 0.5 to 1.04 up to 100 steps.
// With FP64 arithmetic two waves per SIMD fit in registers (512 lanes of 256), with
// FP32 three (768 lanes): 336 owned columns of 512 lanes, 560 of 768.
// Small boxes take tiles of 8 rows of lanes (see plan3).
template <int ROWS>
struct Tile3Shape {
    static constexpr int TX = 32, TY = ROWS, T = TX * TY;
    static constexpr int CX = TX + 2, CY = TY + 2;  // nodes whose c_k, V_k the lanes need
    static constexpr int SX = TX - 2, SY = TY - 2;  // lanes that form the stress
};

constexpr int kSmallRows3 = 8;
template <typename C>
constexpr int kRows3 = sizeof(C) == 4 ? 24 : 16;

// sx: columns from the tile's first lane to its first owned node, 2 or 3 (see plan3)
struct Tile3 {
    int32_t x0, y0, z0, cols, rows, depth, sx;
};

// Links whose totals are kept in LDS from stage 1 to stage 3 (the others are loaded again): a
// value of a link with e_z = -1 waits 2 iterations, with e_z = 0 three, with e_z = +1 four, so the
// links are taken in that order while their slots (one storage-type value per owning lane
// each) fit in what the 160 KB of LDS have left.
template <typename S, typename C, int Q, int ROWS>
struct Hold3 {
    using Sh = Tile3Shape<ROWS>;
    static constexpr int lanes = (Sh::TX - 4) * (Sh::TY - 4);
    static constexpr int base = (9 * Sh::CX * Sh::CY + 9 * Sh::T + 6 * Sh::SX * Sh::SY) * (int)sizeof(C);
    static constexpr int slots = (160 * 1024 - 64 - base) / (lanes * (int)sizeof(S));
    static constexpr int wait(int i) { return L3Z[i] + 3; }  // iterations
    // first slot of link i, or -1
    static constexpr int first(int i)
    {
        int n = 0;
        for (int ez = -1; ez <= 1; ++ez)
            for (int k = 0; k < Q; ++k) {
                if (L3Z[k] != ez) continue;
                const bool fits = n + ez + 3 <= slots;
                if (k == i) return fits ? n : -1;
                if (fits) n += ez + 3;
            }
        return -1;
    }
    static constexpr int used()
    {
        int n = 0;
        for (int i = 0; i < Q; ++i) n += first(i) >= 0 ? wait(i) : 0;
        return n;
    }
};

// What a state holds: the three initial densities (FP64) or the factored values.
enum class In3 : int { Rho = 0, Fac = 1 };

template <typename S, typename C, int Q, int ROWS>
struct alignas(16) March3Lds {
    using Sh = Tile3Shape<ROWS>;
    using Hold = Hold3<S, C, Q, ROWS>;
    C c[3][3][Sh::T];          // c_k of the new densities, by plane mod 3
    C cv[9][Sh::CX * Sh::CY];  // c_k, V_0, V_1 of the source plane (lanes beyond the halo may read
                               // one element before it)
    C T[6][Sh::SX * Sh::SY];   // stress of one plane
    S held[Hold::used()][Hold::lanes];  // totals of the owned nodes
};

// The population of link i of a fluid at rest with density r, as a state in S holds it.
template <typename S, typename C, int Q>
__device__ __forceinline__ C rest_pop(int i, double r)
{
    return C(S(w3<C, Q>(i) * C(r)));
}

template <typename S, typename C, bool OBS, int Q, In3 IN, typename Off, int ROWS>
__device__ __forceinline__ void march3(const void* __restrict__ in, const Geo3& g, const KParams& kp, const Tile3& tl,
                                       S* __restrict__ out, March3Lds<S, C, Q, ROWS>& L, double (&acc)[8],
                                       double* __restrict__ rho_out, uint32_t salt)
{
    using Sh = Tile3Shape<ROWS>;
    using Hold = Hold3<S, C, Q, ROWS>;
    constexpr int TX = Sh::TX, T3 = Sh::T, NV = kVals3<S, C, Q>;
    const int t = threadIdx.x, tx = t % TX, ty = t / TX;
    const int sx = tl.sx;  // lane tx sits on column x0 - sx + tx
    const bool in2 = tx >= sx - 1 && tx <= tl.cols + sx && ty >= 1 && ty <= tl.rows + 2;
    const bool in3 = tx >= sx && tx < tl.cols + sx && ty >= 2 && ty <= tl.rows + 1;
    const int x = wrapi(tl.x0 - sx + tx, g.nx), y = wrapi(tl.y0 - 2 + ty, g.ny);
    // byte offsets within a plane of the nine lateral neighbours, by 3 (e_y + 1) + e_x + 1
    Off lo[9];
    {
        const int xs[3] = {x == 0 ? g.nx - 1 : x - 1, x, x == g.nx - 1 ? 0 : x + 1};
        const int64_t ys[3] = {(int64_t)(y == 0 ? g.ny - 1 : y - 1) * g.nx, (int64_t)y * g.nx,
                               (int64_t)(y == g.ny - 1 ? 0 : y + 1) * g.nx};
#pragma unroll
        for (int a = 0; a < 9; ++a) lo[a] = node_off3<S, NV, Off>(ys[a / 3] + xs[a % 3]);
    }
    const int64_t pl = (int64_t)g.nx * g.ny, np = (int64_t)y * g.nx + x;  // nodes of a plane; the lane's
    const uint64_t fin = (uint64_t)in, fout = (uint64_t)out;
    const double* rin = (const double*)in;
    // the lane's node in cv, c and T.  Each is one LDS address, kept opaque: an access reaches 64
    // KiB past its address register, and the optimiser would otherwise take all three from
    // the start of LDS and hold the sums that do not fit in registers.
    typedef __attribute__((address_space(3))) C lds_t;
    lds_t* cv = (lds_t*)&L.cv[0][0] + ((ty + 1) * Sh::CX + tx + 3 - sx);
    lds_t* cl = (lds_t*)&L.c[0][0][0] + t;
    lds_t* Tl = (lds_t*)&L.T[0][0] + ((ty - 1) * Sh::SX + (tx - 1));
    typedef __attribute__((address_space(3))) S held_t;
    held_t* hl = (held_t*)&L.held[0][0] + ((ty - 2) * (Sh::TX - 4) + (tx - 2));
    constexpr int NC = Sh::CX * Sh::CY, NT = Sh::SX * Sh::SY;
    settle(cv);
    settle(cl);
    settle(Tl);
    settle(hl);
    // The ring of nodes around the lanes': one more c_k, V_k for lanes of the first and, where it
    // has sides, of the last wave, which own no node (their tile rows are the halo's) and so
    // load no totals.
    const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
    const bool edge = wave == 0 || wave == T3 / 64 - 1;
    const bool edge_cv = wave == 0 || (edge && sx == 2);
    const int e = wave == 0 ? t : t - (T3 - 128);  // 0 .. 127
    const int cw = sx == 2 ? Sh::CX : TX;          // nodes of the ring's rows
    int ru, rw;
    if (e < cw) ru = e, rw = 0;
    else if (e < 2 * cw) ru = e - cw, rw = Sh::CY - 1;
    else if (e < 2 * cw + Sh::TY) ru = 0, rw = e - 2 * cw + 1;
    else ru = Sh::CX - 1, rw = e - 2 * cw - Sh::TY + 1;
    const bool ring = edge_cv && e < 2 * cw + (sx == 2 ? 2 * Sh::TY : 0) && ru <= tl.cols + 5 && rw <= tl.rows + 5;
    Off ro = node_off3<S, NV, Off>((int64_t)wrapi(tl.y0 - 3 + rw, g.ny) * g.nx + wrapi(tl.x0 - 3 + ru, g.nx));
    lds_t* cr = (lds_t*)&L.cv[0][0] + rw * Sh::CX + ru;
    settle(cr);

    // f_dag_i(x - e_i) of source plane s for every link; the c_k, V_k of source plane s; the
    // f_dag_i(x - e_i) that meet at plane p
    auto at = [](int i) { return 3 * (1 - L3Y[i]) + 1 - L3X[i]; };
    auto load_f = [&](int s, S (&v)[Q]) {
        const uint64_t base = fin + s * g.zbytes;
#pragma unroll
        for (int a = 0; a < 9; ++a) refresh(lo[a]);
#pragma unroll
        for (int i = 0; i < Q; ++i) v[i] = ld_value<S>(base, lo[at(i)], i);
    };
    auto load_cv = [&](int s, Off& o, auto& v) {
        const uint64_t base = fin + s * g.zbytes;
        refresh(o);
#pragma unroll
        for (int i = 0; i < NV - Q; ++i) v[i] = ld_value<S>(base, o, Q + i);
    };
    auto load_t = [&](int p, S (&v)[Q]) {
        const uint64_t base[3] = {fin + (p == 0 ? g.nz - 1 : p - 1) * g.zbytes, fin + p * g.zbytes,
                                  fin + (p == g.nz - 1 ? 0 : p + 1) * g.zbytes};
#pragma unroll
        for (int a = 0; a < 9; ++a) refresh(lo[a]);
#pragma unroll
        for (int i = 0; i < Q; ++i)
            if (Hold::first(i) < 0) v[i] = ld_value<S>(base[1 - L3Z[i]], lo[at(i)], i);
    };

    C D0[3], D1[3], rA[3], rB[3], Fa[3], Fb[3], rhoA = C(1), itauA = C(1);
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        D0[k] = D1[k] = Fa[k] = Fb[k] = C(0);
        rA[k] = rB[k] = C(1);
    }
    // vf: f_dag_i; vc: c_k, V_k of the lane's node; vx: totals, or in the two edge waves the c_k,
    // V_k of the ring
    S vf[Q], vx[Q], vc[NV - Q];
#pragma unroll
    for (int i = 0; i < Q; ++i) vf[i] = vx[i] = S(0);

    constexpr bool kLate = Q == 27 && sizeof(S) == 8;
    const int J = tl.depth + 6;
    RowCursor sf(tl.z0 - 3, g.nz), sc(tl.z0 - 3, g.nz);  // the next plane of load_f and of load_cv
    RowCursor dst(tl.z0 - 4, g.nz), tot(tl.z0, g.nz);    // plane s - 1; the next plane of load_t
    auto expand = [&](lds_t* p, const S* v) {
#pragma unroll
        for (int i = 0; i < 9; ++i) {
            if constexpr (kRounds<S, C>)
                p[i * NC] = i < 3 ? join_c(v[i], __float_as_uint(v[9]), i) : C(v[i]);
            else
                p[i * NC] = v[i];
        }
    };
    auto publish = [&]() {
        expand(cv, vc);
        if (ring) expand(cr, vx);
    };
    auto load_next_cv = [&]() {
        const int s = sc.next();
        load_cv(s, lo[4], vc);
        if (edge_cv) load_cv(s, ro, vx);
    };
    if constexpr (IN == In3::Fac) {
        load_next_cv();
        load_f(sf.next(), vf);
        publish();
        load_next_cv();
    }
    __syncthreads();
    int slot = 0;        // ring slot of plane s - 1
    int h2 = 0, h3 = 0, h4 = 0;  // j mod 2, 3, 4
#pragma unroll 1
    for (int j = 0; j < J; ++j) {
        // the ring's planes s - 1, s - 2, s - 3
        lds_t* const c0 = cl + slot * (3 * T3);
        lds_t* const c1 = cl + (slot == 0 ? 2 : slot - 1) * (3 * T3);
        slot = slot == 2 ? 0 : slot + 1;
        lds_t* const c2 = cl + slot * (3 * T3);
        const int zd = dst.next();
        // ---- stage 1 (every lane: those past the tile's halo sum what is never read)
        __builtin_amdgcn_sched_barrier(0);
        C rk[3];
        if constexpr (IN == In3::Fac) {
            // What the plane gives to planes s + 1 (P0), s (Z0) and s - 1 (rk) is summed by itself and
            // then added, the source columns from the corners to the centre, so that in each sum
            // the small weights come first: 19 or 27 additions to one sum let the density of an FP32
            // fluid at rest drift by 10 and 24 units of 2^-24 (RMS over densities from 0.8 to 1.2, 60
            // steps), these by 0.5 and 1.1.
            C P0[3] = {C(0), C(0), C(0)}, Z0[3] = {C(0), C(0), C(0)};
            constexpr int OX[9] = {-1, 1, -1, 1, 0, -1, 1, 0, 0}, OY[9] = {-1, -1, 1, 1, -1, 0, 0, 1, 0};
            rk[0] = rk[1] = rk[2] = C(0);
#pragma unroll
            for (int a = 0; a < 9; ++a) {
                const int n = OY[a] * Sh::CX + OX[a];
                const C c0 = cv[n], c1 = cv[NC + n], c2 = cv[2 * NC + n];
#pragma unroll
                for (int i = 0; i < Q; ++i)
                    if (L3X[i] == -OX[a] && L3Y[i] == -OY[a]) {
                        const C f = C(vf[i]);
                        C(&d)[3] = L3Z[i] < 0 ? rk : (L3Z[i] == 0 ? Z0 : P0);
                        d[0] = fma(c0, f, d[0]);
                        d[1] = fma(c1, f, d[1]);
                        d[2] = fma(c2, f, d[2]);
                    }
            }
#pragma unroll
            for (int k = 0; k < 3; ++k) {
                settle(rk[k]);
                settle(P0[k]);
                settle(Z0[k]);
            }
            if (in3) {
                // the totals that waited come out, those of this plane go in
                held_t* const h[3] = {hl + h2 * Hold::lanes, hl + h3 * Hold::lanes, hl + h4 * Hold::lanes};
#pragma unroll
                for (int i = 0; i < Q; ++i)
                    if (Hold::first(i) >= 0) {
                        held_t* const a = h[L3Z[i] + 1] + Hold::first(i) * Hold::lanes;
                        vx[i] = *a;
                        *a = vf[i];
                    }
            }
            h2 ^= 1;
            h3 = h3 == 2 ? 0 : h3 + 1;
            h4 = (h4 + 1) & 3;
            if constexpr (!kLate) load_f(sf.next(), vf);
            __builtin_amdgcn_sched_barrier(0);
            C m[2], p[2], z[2];
#pragma unroll
            for (int k = 0; k < 2; ++k) {
                plane_div<C, Q>([&](int a, int ox, int oy) { return cv[(3 + 3 * k + a) * NC + oy * Sh::CX + ox]; }, m[k],
                                p[k], z[k]);
                __builtin_amdgcn_sched_barrier(0);
            }
            const C dn[2] = {p[0] + z[0], p[1] + z[1]}, up[2] = {p[0] - z[0], p[1] - z[1]};
#pragma unroll
            for (int k = 0; k < 2; ++k) {
                rk[k] -= dn[k];
                Z0[k] -= m[k];
                P0[k] -= up[k];
            }
            rk[2] += dn[0] + dn[1];
            Z0[2] += m[0] + m[1];
            P0[2] += up[0] + up[1];
#pragma unroll
            for (int k = 0; k < 3; ++k) {
                rk[k] += D1[k];
                D1[k] = D0[k] + Z0[k];
                D0[k] = P0[k];
                settle(rk[k]);
                settle(D0[k]);
                settle(D1[k]);
            }
        } else {
            double r[3];
#pragma unroll
            for (int k = 0; k < 3; ++k) r[k] = rin[k * g.N + (int64_t)zd * pl + np];
#pragma unroll
            for (int k = 0; k < 3; ++k) {
                rk[k] = C(0);
#pragma unroll
                for (int i = Q - 1; i >= 0; --i) rk[k] += rest_pop<S, C, Q>(i, r[k]);
            }
        }
        // c_k = rho_k / rho with the remainder's correction: exactly 1 in a pure fluid, where a
        // quotient one ulp off would change the density by as much in every step
        const C rho = (rk[0] + rk[1]) + rk[2], irho = recip(rho);
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            const C c = rk[k] * irho;
            c0[k * T3] = fma(fma(-c, rho, rk[k]), irho, c);
        }
        __syncthreads();
        // ---- stage 2
        const C rho3 = rhoA, itau3 = itauA;  // of plane s - 3
        if (j >= 4 && in2) {
            lds_t* const cz[3] = {c2, c1, c0};  // by dz + 1
            C gc[3][3], cc[3], tt[6], V[6];
#pragma unroll
            for (int k = 0; k < 3; ++k) {
                grad3<C, Q>([&](int dx, int dy, int dz) { return cz[dz + 1][k * T3 + dy * TX + dx]; }, gc[k]);
                cc[k] = c1[k * T3];
            }
            stress3<C>(gc, cc, rA, kp, tt, V);
#pragma unroll
            for (int q = 0; q < 6; ++q) Tl[q * NT] = tt[q];
            // tau = 3 nu + 1/2 with rho / nu = sum_k rho_k / nu_k (Eqs. 10-11)
            rhoA = (rA[0] + rA[1]) + rA[2];
            const C rn = rA[0] * C(kp.inv_nu[0]) + rA[1] * C(kp.inv_nu[1]) + rA[2] * C(kp.inv_nu[2]);
            itauA = rn * recip(C(3) * rhoA + C(0.5) * rn);
            if constexpr (!OBS) {
                const int z2 = tl.z0 - 5 + j;  // plane s - 2
                if (in3 && z2 >= tl.z0 && z2 < tl.z0 + tl.depth) {
                    NodeBits bits((uint32_t)(z2 * pl + np) * (3u * Q) ^ salt);
                    bits.skip(Q);
                    const uint64_t base = fout + z2 * g.zbytes;
                    refresh(lo[4]);
                    if constexpr (kRounds<S, C>) {
                        uint32_t word = 0;
#pragma unroll
                        for (int k = 0; k < 3; ++k) st_value<S>(base, lo[4], Q + k, split_c(cc[k], bits.next(), k, word));
                        st_value<S>(base, lo[4], Q + 9, __uint_as_float(word));
                    } else {
#pragma unroll
                        for (int k = 0; k < 3; ++k) st_value<S>(base, lo[4], Q + k, S(cc[k]));
                    }
#pragma unroll
                    for (int a = 0; a < 6; ++a) st_value<S>(base, lo[4], Q + 3 + a, to_storage<S, C>(V[a], bits));
                }
            }
        }
        if constexpr (IN == In3::Fac) {
            publish();
            if constexpr (kLate) load_f(sf.next(), vf);
            load_next_cv();
        }
        __syncthreads();
        // ---- stage 3
        if (j >= 4 && in3) {
            C F[3];
            constexpr int QI[3][3] = {{0, 1, 2}, {1, 3, 4}, {2, 4, 5}};
#pragma unroll
            for (int b = 0; b < 3; ++b) {
                C m, p, z;
                plane_div<C, Q>([&](int a, int ox, int oy) { return Tl[QI[a][b] * NT + oy * Sh::SX + ox]; }, m, p, z);
                F[b] = C(3) * (Fb[b] + (p + z));
                Fb[b] = Fa[b] + m;
                Fa[b] = p - z;
            }
            const int z3 = tl.z0 - 6 + j;  // plane s - 3
            if (j >= 6) {
                C ft[Q];
                if constexpr (IN == In3::Fac) {
#pragma unroll
                    for (int i = 0; i < Q; ++i) ft[i] = C(vx[i]);
                } else {
                    double r[3];
#pragma unroll
                    for (int k = 0; k < 3; ++k) r[k] = rin[k * g.N + (int64_t)z3 * pl + np];
#pragma unroll
                    for (int i = 0; i < Q; ++i)
                        ft[i] = (rest_pop<S, C, Q>(i, r[0]) + rest_pop<S, C, Q>(i, r[1])) + rest_pop<S, C, Q>(i, r[2]);
                }
                C u[3] = {C(0), C(0), C(0)};
                const C ir = recip(rho3);
#pragma unroll
                for (int i = 0; i < Q; ++i) {
                    if (L3X[i] != 0) u[0] += L3X[i] > 0 ? ft[i] : -ft[i];
                    if (L3Y[i] != 0) u[1] += L3Y[i] > 0 ? ft[i] : -ft[i];
                    if (L3Z[i] != 0) u[2] += L3Z[i] > 0 ? ft[i] : -ft[i];
                }
#pragma unroll
                for (int a = 0; a < 3; ++a) u[a] = (u[a] + C(0.5) * F[a]) * ir;
                if constexpr (OBS) {
#pragma unroll
                    for (int k = 0; k < 3; ++k) acc[k] += double(rB[k]);
#pragma unroll
                    for (int a = 0; a < 3; ++a) acc[3 + a] += double(rho3 * u[a]);
                    const double uu = double(u[0] * u[0] + u[1] * u[1] + u[2] * u[2]);
                    acc[6] += 0.5 * double(rho3) * uu;
                    const double um = sqrt(uu);
                    acc[7] = (um > acc[7] || um != um) ? um : acc[7];
                    if (rho_out) {
#pragma unroll
                        for (int k = 0; k < 3; ++k) rho_out[k * g.N + (int64_t)z3 * pl + np] = double(rB[k]);
                    }
                } else {
                    NodeBits bits((uint32_t)(z3 * pl + np) * (3u * Q) ^ salt);
                    const uint64_t base = fout + z3 * g.zbytes;
                    refresh(lo[4]);
                    collide3<C, Q>(rho3, itau3, ft, F, u,
                                   [&](int i, C v) { st_value<S>(base, lo[4], i, to_storage<S, C>(v, bits)); });
                }
            }
        }
        // the totals of the next iteration's plane
        if constexpr (IN == In3::Fac) {
            if (j >= 5 && !edge) load_t(tot.next(), vx);
        }
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            if constexpr (OBS) rB[k] = rA[k];
            rA[k] = rk[k];
        }
    }
}

// S: storage type, C: compute type.  With FP32 storage of FP64 arithmetic each stored value
// is rounded stochastically with the random bits of its node (key: node index and the step's
// salt; f_dag_i first, then c_k, V_0, V_1).  OBS: the observables of the state instead of its
// next step, and with rho_out the densities.
template <typename S, typename C, bool OBS, int Q, In3 IN, typename Off, int ROWS>
__global__ __launch_bounds__(Tile3Shape<ROWS>::T) __attribute__((amdgpu_waves_per_eu(Tile3Shape<ROWS>::T / 256))) void k3_march(
    const void* __restrict__ in, Geo3 g, KParams kp, const Tile3* __restrict__ tiles, S* __restrict__ out,
    double* __restrict__ partials, double* __restrict__ rho_out, uint32_t salt)
{
    using Sh = Tile3Shape<ROWS>;
    constexpr int T3 = Sh::T;
    static_assert(T3 % 64 == 0 && (2 * Sh::TX) % 64 == 0, "each wave is whole tile rows");
    static_assert(2 * Sh::CX + 2 * Sh::TY <= 128, "one lane of two waves per node of the outer ring");
    static_assert(sizeof(double) * 8 * (T3 / 64) <= sizeof(C) * 3 * 3 * T3, "c ring too small for the reduction");
    __shared__ March3Lds<S, C, Q, ROWS> L;
    const Tile3 tl = tiles[blockIdx.x];
    const int t = threadIdx.x;
    double acc[8] = {0, 0, 0, 0, 0, 0, 0, 0};
    march3<S, C, OBS, Q, IN, Off, ROWS>(in, g, kp, tl, out, L, acc, rho_out, salt);
    if constexpr (OBS) {
        // wavefront reductions, then the waves' results in order (the c ring is free once
        // every lane has passed the last barrier of the march)
        __syncthreads();
        for (int q = 0; q < 7; ++q) acc[q] = wave_sum(acc[q]);
        acc[7] = wave_max(acc[7]);
        double* red = reinterpret_cast<double*>(&L.c[0][0][0]);
        constexpr int W = T3 / 64;
        if ((t & 63) == 0)
            for (int q = 0; q < 8; ++q) red[q * W + (t >> 6)] = acc[q];
        __syncthreads();
        if (t < 8) {
            double v = red[t * W];
            for (int w = 1; w < W; ++w) {
                const double o = red[t * W + w];
                v = t < 7 ? v + o : ((o > v || o != o) ? o : v);
            }
            partials[(int64_t)blockIdx.x * 8 + t] = v;
        }
    }
}

// Node-parallel kernels (initialisation, export): blocks of 256 consecutive nodes (x
// fastest, then y, then z) on a one-dimensional grid.  Workgroups go to the eight XCDs in
// turn; block b takes the node range of logical block xcd_block(b), so that each XCD works
// through one contiguous run of blocks.  The map is a bijection of [0, T) for any T.
__device__ __forceinline__ int64_t xcd_block(int64_t b, int64_t T)
{
    const int64_t x = b & 7, k = b >> 3, q = T >> 3, r = T & 7;
    return x * q + (x < r ? x : r) + k;
}

// (x, y, z) of this thread's node; false past the last node
__device__ __forceinline__ bool node3(const Geo3& g, int& x, int& y, int& z)
{
    const int64_t n = xcd_block(blockIdx.x, gridDim.x) * 256 + threadIdx.x;
    if (n >= g.N) return false;
    // N <= 2^29 (checked at creation): 32-bit division suffices
    const uint32_t n32 = (uint32_t)n, nx = (uint32_t)g.nx, ny = (uint32_t)g.ny;
    const uint32_t p = n32 / nx, zz = p / ny;
    x = (int)(n32 - p * nx), y = (int)(p - zz * ny), z = (int)zz;
    return true;
}

// the post-streaming populations f[3][Q][N] of the state, f_{i,k} = c_k f_dag_i + w_i V_k . e_i
// at x - e_i (or those of the fluid at rest)
template <typename S, typename C, int Q>
__global__ __launch_bounds__(256) void k3_export(const void* __restrict__ in, In3 fmt, Geo3 g, double* __restrict__ f)
{
    int x, y, z;
    if (!node3(g, x, y, z)) return;
    const Nb3 nb(g, x, y, z);
    const int64_t j = nb.at(0, 0, 0);
    if (fmt == In3::Rho) {
        const double* rho = (const double*)in;
#pragma unroll
        for (int i = 0; i < Q; ++i)
#pragma unroll
            for (int k = 0; k < 3; ++k)
                f[(int64_t)(k * Q + i) * g.N + j] = double(rest_pop<S, C, Q>(i, rho[k * g.N + j]));
        return;
    }
    const int64_t pl = (int64_t)g.nx * g.ny;
#pragma unroll
    for (int i = 0; i < Q; ++i) {
        const int64_t zs = nb.zo[1 - L3Z[i]];
        const int64_t o = node_off3<S, kVals3<S, C, Q>, int64_t>(nb.at(-L3X[i], -L3Y[i], -L3Z[i]) - zs);
        const char* b = (const char*)in + zs / pl * g.zbytes + o;
        auto value = [&](int v) { return C(*(const S*)(b + v * kLine)); };
        auto conc = [&](int k) {
            if constexpr (kRounds<S, C>)
                return join_c(*(const S*)(b + (Q + k) * kLine), *(const uint32_t*)(b + (Q + 9) * kLine), k);
            else
                return value(Q + k);
        };
        const C fd = value(i);
        C V[3][3];
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            V[0][a] = value(Q + 3 + a);
            V[1][a] = value(Q + 6 + a);
            V[2][a] = -(V[0][a] + V[1][a]);
        }
#pragma unroll
        for (int k = 0; k < 3; ++k)
            f[(int64_t)(k * Q + i) * g.N + j] =
                double(fma(conc(k), fd, w3<C, Q>(i) * edot<C>(i, V[k][0], V[k][1], V[k][2])));
    }
}


}  // namespace
}  // namespace tcg

using namespace tcg;

struct lbm3d {
    lbm3_params p{};
    KParams kp{};
    Geo3 g{};
    hipStream_t stream = nullptr;
    Prec prec = Prec::F64;
    int q = 19;                         // links: 19 or 27
    void* buf[2] = {nullptr, nullptr};  // the state, in the storage type of prec
    In3 fmt = In3::Rho;                 // what buf[cur] holds
    Tile3* dtiles = nullptr;     // the march's tile list
    int ntiles = 0;
    double* partials = nullptr;  // [ntiles][8]
    double* staging = nullptr;   // [3q][N] for exports
    double* rho = nullptr;       // [3][N] densities for exports
    int rows = 0;  // rows of lanes of its tiles
    int cur = 0;
    int64_t step = 0;
    bool ready = false;
};

static dim3 grid3(const Geo3& g) { return dim3((unsigned)((g.N + 255) / 256)); }

static void release3(lbm3d* h)
{
    if (h->stream) (void)hipStreamSynchronize(h->stream);
    free_state_pair(h->buf);
    for (void* q : {(void*)h->partials, (void*)h->staging, (void*)h->rho})
        if (q) (void)hipFree(q);
    if (h->dtiles) (void)hipFree(h->dtiles);
}

// n split into `parts` parts as equal as possible: part q is [start, start + len)
static void split_even(int n, int parts, int q, int& start, int& len)
{
    const int base = n / parts, extra = n % parts;
    start = q * base + (q < extra ? q : extra);
    len = base + (q < extra ? 1 : 0);
}

// The march's tiles: the x-y plane cut into at most (TX - 4) x (TY - 4) node blocks (the
// tile shape of the compute type), the z axis into `nseg` segments chosen so that rounds of
// resident workgroups x (segment depth + 6 warm-up planes) is least, down to one plane a segment
// (48^3 D3Q19 FP64: 12 segments of 4 planes 56 us, 24 of 2 planes 48 us).  Workgroups go to the
// XCDs in turn, so the list is permuted for each XCD to take a contiguous run of it
// (neighbouring blocks, whose halos it then finds in its own L2).
//
// Tiles of 8 rows of lanes (28 x 4 nodes) take less time per plane, their four waves having a
// SIMD each, but own a third of the nodes: a plane's time is 0.72 of the large tile's with FP64
// arithmetic, 0.9 in FP32, where three of the small ones share a compute unit, and the plan with
// the least of rounds x planes x that time is taken (us per step, large and small tiles: D3Q19
// FP64 32^3 31.8 and 26.6, 48^3 36.8 and 34.7, 64^3 56.0 and 60.8, 96^3 134 and 187; FP32 32^3 24.4
// and 19.9, 64^3 40.9 and 37.4, 80^3 53.1 and 68.3; D3Q27 FP64 32^3 39.4 and 32.9, 48^3 50.7 and
// 46.7, FP32 64^3 49.9 and 45.0).
static std::vector<Tile3> plan3(const Geo3& g, const int (&slots)[2], Prec prec, int& rows)
{
    constexpr int TX = Tile3Shape<kSmallRows3>::TX;
    const int shapes[2] = {prec == Prec::F32 ? kRows3<float> : kRows3<double>, kSmallRows3};
    const double plane[2] = {1.0, prec == Prec::F32 ? 0.9 : 0.72};
    int ntx = 1, nty = 1, nseg = 1;
    double best = 1e300;
    for (int k = 0; k < 2; ++k) {
        const int TY = shapes[k], nx = (g.nx + TX - 5) / (TX - 4), ny = (g.ny + TY - 5) / (TY - 4);
        const int64_t per_seg = (int64_t)nx * ny, n = std::max(slots[k], 1);
        if (k == 1 && g.zbytes >= ((int64_t)1 << 32)) break;
        for (int s = 1; s <= g.nz; ++s) {
            const int depth = (g.nz + s - 1) / s;
            const int64_t rounds = (per_seg * s + n - 1) / n;
            const double cost = (double)rounds * (depth + 6) * plane[k] * (1.0 + 1e-9 * s);
            if (cost < best) {
                best = cost;
                nseg = s;
                ntx = nx;
                nty = ny;
                rows = TY;
            }
        }
    }
    // Where no tile has more than TX - 6 columns the lanes start one column earlier: they then
    // cover every column whose c_k, V_k stage 1 reads, and the ring of nodes around the lanes'
    // has no sides, whose nodes lie in a cache line each (D3Q19 FP64 128^3 325 -> 304 us, FP32
    // storage 226 -> 214, 127^3 231 -> 216; FP32 D3Q19 52^3 44 -> 35, 96^3 78 -> 74, 127^3 187 -> 175,
    // 144^3 259 -> 241, D3Q27 127^3 239 -> 230, slower among 13 sides from 40 to 160 only at 128^3:
    // 180 -> 193, D3Q27 238 -> 249).  Tiles of both kinds side by side were slower (160^3, 27 and 26
    // columns: 384 -> 400).
    const int sx = (g.nx + ntx - 1) / ntx <= TX - 6 ? 3 : 2;
    std::vector<Tile3> L;
    L.reserve((size_t)ntx * nty * nseg);
    for (int zs = 0; zs < nseg; ++zs)
        for (int ty = 0; ty < nty; ++ty)
            for (int tx = 0; tx < ntx; ++tx) {
                Tile3 t{};
                split_even(g.nx, ntx, tx, t.x0, t.cols);
                split_even(g.ny, nty, ty, t.y0, t.rows);
                split_even(g.nz, nseg, zs, t.z0, t.depth);
                t.sx = sx;
                L.push_back(t);
            }
    const int T = (int)L.size(), nxcd = 8;
    std::vector<Tile3> out(T);
    std::vector<int> start(nxcd + 1, 0);
    for (int x = 0; x < nxcd; ++x) start[x + 1] = start[x] + (T - x + nxcd - 1) / nxcd;
    for (int b = 0; b < T; ++b) out[b] = L[start[b % nxcd] + b / nxcd];
    return out;
}

template <typename S, typename C, int Q, In3 IN, typename Off, int ROWS>
static hipError_t launch_march_r(lbm3d* h, bool obs, double* rho_out)
{
    const void* in = h->buf[h->cur];
    const dim3 grid(h->ntiles), block(Tile3Shape<ROWS>::T);
    if (obs)
        hipLaunchKernelGGL((k3_march<S, C, true, Q, IN, Off, ROWS>), grid, block, 0, h->stream, in, h->g, h->kp,
                           (const Tile3*)h->dtiles, (S*)nullptr, h->partials, rho_out, 0u);
    else
        hipLaunchKernelGGL((k3_march<S, C, false, Q, IN, Off, ROWS>), grid, block, 0, h->stream, in, h->g, h->kp,
                           (const Tile3*)h->dtiles, (S*)h->buf[h->cur ^ 1], (double*)nullptr, (double*)nullptr,
                           step_salt(h->step));
    return hipGetLastError();
}

template <typename S, typename C, int Q, In3 IN, typename Off>
static hipError_t launch_march_f(lbm3d* h, bool obs, double* rho_out)
{
    return h->rows == kSmallRows3 ? launch_march_r<S, C, Q, IN, Off, kSmallRows3>(h, obs, rho_out)
                                  : launch_march_r<S, C, Q, IN, Off, kRows3<C>>(h, obs, rho_out);
}

// Offsets within a z plane fit 32 bits below 4 GiB a plane (15 to 38 million nodes); larger
// planes (never with small tiles), and every first step, take the 64-bit instantiation.
template <typename S, typename C, int Q>
static hipError_t launch_march_q(lbm3d* h, bool obs, double* rho_out)
{
    if (h->fmt == In3::Rho) return launch_march_f<S, C, Q, In3::Rho, uint64_t>(h, obs, rho_out);
    if (h->g.zbytes >= ((int64_t)1 << 32)) return launch_march_r<S, C, Q, In3::Fac, uint64_t, kRows3<C>>(h, obs, rho_out);
    return launch_march_f<S, C, Q, In3::Fac, uint32_t>(h, obs, rho_out);
}

template <typename S, typename C>
static hipError_t launch_march_t(lbm3d* h, bool obs, double* rho_out)
{
    return h->q == 27 ? launch_march_q<S, C, 27>(h, obs, rho_out) : launch_march_q<S, C, 19>(h, obs, rho_out);
}

// One step into the other buffer, or (obs) the observables' partial sums and, with rho_out,
// the densities [3][N].
static hipError_t launch_march(lbm3d* h, bool obs, double* rho_out = nullptr)
{
    switch (h->prec) {
        case Prec::F64: return launch_march_t<double, double>(h, obs, rho_out);
        case Prec::F32S: return launch_march_t<float, double>(h, obs, rho_out);
        case Prec::F32: return launch_march_t<float, float>(h, obs, rho_out);
    }
    return hipErrorInvalidValue;
}

template <typename S, typename C, int ROWS>
static hipError_t march_occupancy_t(int q, int* per_cu)
{
    constexpr int T = Tile3Shape<ROWS>::T;
    return q == 27 ? hipOccupancyMaxActiveBlocksPerMultiprocessor(
                         per_cu, k3_march<S, C, false, 27, In3::Fac, uint32_t, ROWS>, T, 0)
                   : hipOccupancyMaxActiveBlocksPerMultiprocessor(
                         per_cu, k3_march<S, C, false, 19, In3::Fac, uint32_t, ROWS>, T, 0);
}

// workgroups per compute unit, of either tile
static hipError_t march_occupancy(Prec prec, int q, bool small, int* per_cu)
{
    switch (prec) {
        case Prec::F64:
            return small ? march_occupancy_t<double, double, kSmallRows3>(q, per_cu)
                         : march_occupancy_t<double, double, kRows3<double>>(q, per_cu);
        case Prec::F32S:
            return small ? march_occupancy_t<float, double, kSmallRows3>(q, per_cu)
                         : march_occupancy_t<float, double, kRows3<double>>(q, per_cu);
        case Prec::F32:
            return small ? march_occupancy_t<float, float, kSmallRows3>(q, per_cu)
                         : march_occupancy_t<float, float, kRows3<float>>(q, per_cu);
    }
    return hipErrorInvalidValue;
}

template <int Q>
static hipError_t launch_export3_q(lbm3d* h, double* fout)
{
    const dim3 gr = grid3(h->g), bl(256);
    const void* in = h->buf[h->cur];
    switch (h->prec) {
        case Prec::F64: hipLaunchKernelGGL((k3_export<double, double, Q>), gr, bl, 0, h->stream, in, h->fmt, h->g, fout); break;
        case Prec::F32S: hipLaunchKernelGGL((k3_export<float, double, Q>), gr, bl, 0, h->stream, in, h->fmt, h->g, fout); break;
        case Prec::F32: hipLaunchKernelGGL((k3_export<float, float, Q>), gr, bl, 0, h->stream, in, h->fmt, h->g, fout); break;
    }
    return hipGetLastError();
}

static hipError_t launch_export3(lbm3d* h, double* fout)
{
    return h->q == 27 ? launch_export3_q<27>(h, fout) : launch_export3_q<19>(h, fout);
}

extern "C" {

int lbm3d_create_lattice(const lbm3_params* p, int32_t nz, int32_t q, void* hip_stream, lbm3d_t** out)
{
    if (out) *out = nullptr;
    if (!out) {
        set_error("out is NULL");
        return LBM3_EINVAL;
    }
    int rc = validate_params(p);
    if (rc) return rc;
    if (q != 19 && q != 27) {
        set_error("the three-dimensional form takes the D3Q19 or the D3Q27 lattice (q = 19 or 27, got %d)", (int)q);
        return LBM3_EINVAL;
    }
    if (nz < 1 || nz > 65535) {
        set_error("nz must be in 1..65535 (got %d)", nz);
        return LBM3_EINVAL;
    }
    if ((int64_t)p->nx * p->ny * nz > ((int64_t)1 << 29)) {
        set_error("the three-dimensional form takes at most 2^29 nodes (got %d x %d x %d)", (int)p->nx, (int)p->ny,
                  nz);
        return LBM3_EINVAL;
    }
    if (p->forcing != LBM3_FORCING_GUO) {
        set_error("the three-dimensional form runs the force of Eq. (7) with Guo's term only");
        return LBM3_EUNSUPPORTED;
    }
    lbm3d* h = new (std::nothrow) lbm3d();
    if (!h) {
        set_error("host allocation failed");
        return LBM3_ENOMEM;
    }
    h->p = *p;
    h->prec = prec_of(p->precision);
    h->q = q;
    derive(p, &h->kp, nullptr, nullptr, nullptr);
    h->g = Geo3{p->nx, p->ny, nz, (int64_t)p->nx * p->ny * nz,
                h->prec == Prec::F64 ? zbytes3<double>(p->nx, p->ny, vals3(h->prec, q))
                                     : zbytes3<float>(p->nx, p->ny, vals3(h->prec, q))};
    h->stream = (hipStream_t)hip_stream;
    const int64_t N = h->g.N;
    hipError_t e = hipSuccess;
    int dev = 0, cus = 0, slots[2] = {0, 0};
    e = hipGetDevice(&dev);
    if (e == hipSuccess) e = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
    for (int k = 0; k < 2 && e == hipSuccess; ++k) {
        e = march_occupancy(h->prec, q, k == 1, &slots[k]);
        slots[k] *= cus;
    }
    std::vector<Tile3> tiles;
    if (e == hipSuccess) {
        tiles = plan3(h->g, slots, h->prec, h->rows);
        h->ntiles = (int)tiles.size();
    }
    if (e == hipSuccess) e = alloc_state_pair((size_t)h->g.zbytes * nz, h->buf);
    if (e == hipSuccess) e = device_malloc((void**)&h->dtiles, tiles.size() * sizeof(Tile3));
    if (e == hipSuccess)
        e = hipMemcpy(h->dtiles, tiles.data(), tiles.size() * sizeof(Tile3), hipMemcpyHostToDevice);
    if (e == hipSuccess) e = device_malloc((void**)&h->partials, tiles.size() * 8 * sizeof(double));
    if (e == hipSuccess) e = device_malloc((void**)&h->staging, (size_t)3 * q * N * sizeof(double));
    if (e == hipSuccess) e = device_malloc((void**)&h->rho, (size_t)3 * N * sizeof(double));
    if (e != hipSuccess) {
        rc = hip_fail(e, "hipMalloc (three-dimensional lattice)");
        release3(h);
        delete h;
        return rc;
    }
    *out = h;
    return LBM3_OK;
}

int lbm3d_create(const lbm3_params* p, int32_t nz, void* hip_stream, lbm3d_t** out)
{
    return lbm3d_create_lattice(p, nz, 19, hip_stream, out);
}

int lbm3d_init_fields(lbm3d_t* h, const double* rho)
{
    if (!h) {
        set_error("handle is NULL");
        return LBM3_EINVAL;
    }
    const int64_t N = h->g.N;
    int rc = check_rho_fields(rho, nullptr, N);
    if (rc) return rc;
    // the densities are the state until the first step (Q + 9 values of at least 4 bytes hold
    // three of 8)
    hipError_t e = hipMemcpyAsync(h->buf[0], rho, (size_t)3 * N * sizeof(double), hipMemcpyHostToDevice, h->stream);
    if (e == hipSuccess) e = hipStreamSynchronize(h->stream);
    if (e != hipSuccess) return hip_fail(e, "three-dimensional init");
    h->cur = 0;
    h->fmt = In3::Rho;
    h->step = 0;
    h->ready = true;
    return LBM3_OK;
}

int lbm3d_step(lbm3d_t* h, int64_t n)
{
    if (!h || n < 0) {
        set_error(!h ? "handle is NULL" : "n must be >= 0");
        return LBM3_EINVAL;
    }
    if (!h->ready) {
        set_error("lbm3d_step before lbm3d_init_fields");
        return LBM3_ESTATE;
    }
    for (int64_t s = 0; s < n; ++s) {
        hipError_t e = launch_march(h, false);
        if (e != hipSuccess) return hip_fail(e, "three-dimensional step launch");
        h->cur ^= 1;
        h->fmt = In3::Fac;
        h->step += 1;
    }
    return LBM3_OK;
}

int lbm3d_observables(lbm3d_t* h, lbm3d_obs* out, double* rho_out, double* f_out)
{
    if (!h) {
        set_error("handle is NULL");
        return LBM3_EINVAL;
    }
    if (!h->ready) {
        set_error("lbm3d_observables before lbm3d_init_fields");
        return LBM3_ESTATE;
    }
    const size_t nblocks = (size_t)h->ntiles;
    const int64_t N = h->g.N;
    hipError_t e = launch_march(h, true, rho_out ? h->rho : nullptr);
    std::vector<double> part(nblocks * 8);
    if (e == hipSuccess)
        e = hipMemcpyAsync(part.data(), h->partials, part.size() * sizeof(double), hipMemcpyDeviceToHost, h->stream);
    if (e == hipSuccess && rho_out)
        e = hipMemcpyAsync(rho_out, h->rho, (size_t)3 * N * sizeof(double), hipMemcpyDeviceToHost, h->stream);
    if (e == hipSuccess && f_out) {
        e = launch_export3(h, h->staging);
        if (e == hipSuccess)
            e = hipMemcpyAsync(f_out, h->staging, (size_t)3 * h->q * N * sizeof(double), hipMemcpyDeviceToHost,
                               h->stream);
    }
    if (e == hipSuccess) e = hipStreamSynchronize(h->stream);
    if (e != hipSuccess) return hip_fail(e, "three-dimensional observables");
    lbm3d_obs o{};
    o.step = h->step;
    bool finite = true;
    for (size_t b = 0; b < nblocks; ++b) {
        for (int q = 0; q < 7; ++q) {
            const double v = part[b * 8 + q];
            if (!std::isfinite(v)) finite = false;
            if (q < 3) o.mass[q] += v;
            else if (q < 6) o.momentum[q - 3] += v;
            else o.kinetic_energy += v;
        }
        const double um = part[b * 8 + 7];
        if (!std::isfinite(um)) finite = false;
        o.u_max = std::max(o.u_max, um);
    }
    o.nonfinite = finite ? 0 : 1;
    if (out) *out = o;
    if (!finite) {
        set_error("the three-dimensional state is not finite at step %lld", (long long)h->step);
        return LBM3_ENONFINITE;
    }
    return LBM3_OK;
}

int lbm3d_destroy(lbm3d_t* h)
{
    if (!h) return LBM3_OK;
    release3(h);
    delete h;
    return LBM3_OK;
}

}  // extern "C"
