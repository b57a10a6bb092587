"""The three-dimensional form through the C ABI (lbm3d_*), on the D3Q19 and the D3Q27
lattice, against the three-dimensional oracle, which is pinned to the two-dimensional oracle
(tests/test_oracle_d3.py)."""
import numpy as np
import pytest

import oracle
from oracle import d3
from paper_1808_08555_amd import inputs, lbm3

pytestmark = pytest.mark.gpu

SIG, TAU = (0.011, 0.013, 0.017), (0.7, 1.0, 1.3)
QS = [19, 27]


def _gpu(rho, steps, sigma=SIG, tau=TAU, law="paper", precision="fp64", q=19):
    nz, ny, nx = rho.shape[1:]
    L = lbm3.Lattice3D(nx, ny, nz, sigma, tau, beta_law=law, precision=precision, q=q).init(rho)
    try:
        return L.step(steps).state()
    finally:
        L.close()


def _oracle(rho, steps, sigma=SIG, tau=TAU, law="paper", q=19):
    nz, ny, nx = rho.shape[1:]
    p = oracle.Params(nx, ny, sigma, tau, beta_law=law)
    return d3.run(p, nz, d3.init(p, nz, rho, q), steps)


@pytest.mark.parametrize("q", QS)
@pytest.mark.parametrize("law", ["paper", "leclaire"])
def test_parity_random_mixture(law, q):
    """13 x 11 x 9 random mixtures (three fluids at most nodes), 10 steps, to 1e-11."""
    rho = inputs.random_mixture_3d(13, 11, 9, 4, tiny_fraction=0.05)
    err = np.abs(_gpu(rho, 10, law=law, q=q) - _oracle(rho, 10, law=law, q=q)).max()
    print(q, law, err)
    assert err <= 1e-11


@pytest.mark.parametrize("q", QS)
def test_parity_two_spheres_along_the_trajectory(q):
    """Tangent spheres of fluids 0 and 1 (R = 6) in fluid 2 on 30 x 26 x 22.  After 50 steps
    the GPU state equals the oracle's to 1e-11.  Further on, round-off differences of the
    colour traces grow about 1.1-1.2x per step (measured: 2e-13 at step 50, 4e-9 at 150,
    6e-5 at 200 for the coloured populations), as in two dimensions, so the longer run is
    checked one step at a time: from the GPU's own state at steps 150-152, one GPU step
    equals one oracle step to 1e-15."""
    rho = inputs.spheres(30, 26, 22, [(0, 9.0, 13.0, 11.0, 6.0), (1, 21.0, 13.0, 11.0, 6.0)])
    p = oracle.Params(30, 26, SIG, TAU)
    L = lbm3.Lattice3D(30, 26, 22, SIG, TAU, q=q).init(rho)
    try:
        g = L.step(50).state()
        o = d3.run(p, 22, d3.init(p, 22, rho, q), 50)
        assert np.abs(g - o).max() <= 1e-11
        L.step(100)
        worst = 0.0
        for _ in range(3):
            prev = L.state()
            worst = max(worst, float(np.abs(L.step(1).state() - d3.step(p, 22, prev)).max()))
        print("one step from the GPU state:", worst)
        assert worst <= 1e-15
    finally:
        L.close()


@pytest.mark.parametrize("q", QS)
@pytest.mark.parametrize("shape", [(1, 2, 3), (2, 1, 1), (3, 4, 1), (257, 3, 2), (61, 23, 7)])
def test_parity_degenerate_and_ragged(shape, q):
    """Lattices narrower than the stencil in some direction, and ragged ones of several tiles
    in x and y (tiles own 28 x 12 columns for D3Q19 and 28 x 10 for D3Q27 in FP64 arithmetic,
    28 x 20 in FP32)."""
    nx, ny, nz = shape
    rho = inputs.random_mixture_3d(nx, ny, nz, 21, tiny_fraction=0.0)
    assert np.abs(_gpu(rho, 5, q=q) - _oracle(rho, 5, q=q)).max() <= 1e-11


@pytest.mark.parametrize("q3", QS)
def test_uniform_along_z_equals_the_2d_step(q3):
    """A lattice uniform along z evolves as the two-dimensional lattice (populations summed
    over the links' z component): GPU against GPU, 300 steps."""
    w = inputs.double_droplet(48, 9.0, 1.0, 1.3, seed=2, steps=0)
    rho3 = np.repeat(w.rho[:, None], 4, axis=1)
    f3 = _gpu(rho3, 300, w.sigma, w.tau, q=q3)
    L = lbm3.Lattice(48, 48, w.sigma, w.tau).init(w.rho)
    f2 = L.step(300).state()
    L.close()
    e, _ = d3.lattice(q3)
    EX2, EY2 = [0, 1, 0, -1, 0, 1, -1, -1, 1], [0, 0, 1, 0, -1, 1, 1, -1, -1]
    proj = np.zeros_like(f2)
    for q in range(9):
        for i in range(q3):
            if e[i, 0] == EX2[q] and e[i, 1] == EY2[q]:
                proj[:, q] += f3[:, i, 0]
    assert np.abs(proj - f2).max() <= 1e-12


@pytest.mark.parametrize("q", QS)
def test_observables_match_the_oracle(q):
    rho = inputs.spheres(20, 18, 16, [(0, 7.0, 9.0, 8.0, 4.0), (1, 13.0, 9.0, 8.0, 4.0)])
    L = lbm3.Lattice3D(20, 18, 16, SIG, TAU, q=q).init(rho).step(50)
    obs, r, f = L.observables(want_rho=True, want_f=True)
    L.close()
    p = oracle.Params(20, 18, SIG, TAU)
    o = d3.observables(p, 16, f)
    print(obs, o)
    assert obs["step"] == 50 and obs["nonfinite"] == 0
    assert np.abs(obs["mass"] / o["mass"] - 1).max() < 1e-13
    assert np.abs(obs["momentum"] - o["momentum"]).max() < 1e-12
    assert abs(obs["kinetic_energy"] / o["kinetic_energy"] - 1) < 1e-9
    assert abs(obs["u_max"] / o["u_max"] - 1) < 1e-9
    assert np.abs(r - f.sum(axis=1)).max() < 1e-14


def test_error_paths():
    with pytest.raises(lbm3.Lbm3Error) as e:
        lbm3.Lattice3D(8, 8, 0)
    assert e.value.code == lbm3.LBM3_EINVAL
    import ctypes
    h = ctypes.c_void_p()
    p = lbm3.make_params(8, 8, forcing="perturbation")
    assert lbm3.lib().lbm3d_create(ctypes.byref(p), 8, None, ctypes.byref(h)) == lbm3.LBM3_EUNSUPPORTED
    L = lbm3.Lattice3D(8, 8, 8)
    try:
        with pytest.raises(lbm3.Lbm3Error) as e:
            L.step(1)
        assert e.value.code == lbm3.LBM3_ESTATE
        bad = np.ones((3, 8, 8, 8))
        bad[1, 2, 3, 4] = -1.0
        with pytest.raises(lbm3.Lbm3Error) as e:
            L.init(bad)
        assert e.value.code == lbm3.LBM3_EINVAL
    finally:
        L.close()


@pytest.mark.parametrize("q", QS)
def test_sphere_young_laplace(q):
    """A sphere of fluid 0 in fluid 2 (48^3, sigma = 0.01, tau = 1, 4000 steps): the pressure
    jump p_in - p_out (p = rho/3, inside r < R/2, outside r > R + 6) against the
    three-dimensional Young-Laplace law 2 sigma / R, with R from the sphere's volume:
    within 4% at R = 12 (measured 2.9%), and closer than at R = 8 (measured 6.2%), as the
    discretization error falls with the radius."""
    import math
    n, ratio = 48, {}
    for R in (8.0, 12.0):
        c = (n - 1) / 2
        L = lbm3.Lattice3D(n, n, n, (0.01, 0.01, 0.01), (1.0, 1.0, 1.0), q=q).init(
            inputs.spheres(n, n, n, [(0, c, c, c, R)]))
        obs, r, _ = L.step(4000).observables(want_rho=True)
        L.close()
        z, y, x = np.mgrid[0:n, 0:n, 0:n].astype(float)
        rr = np.sqrt((x - c) ** 2 + (y - c) ** 2 + (z - c) ** 2)
        tot = r.sum(0)
        Reff = (3 * (r[0] / tot).sum() / (4 * math.pi)) ** (1 / 3)
        dp = tot[rr < Reff / 2].mean() / 3 - tot[rr > Reff + 6].mean() / 3
        ratio[R] = dp / (2 * 0.01 / Reff)
        print(f"D3Q{q} R={R}: R_eff={Reff:.3f} dp={dp:.4e} ratio={ratio[R]:.4f} u_max={obs['u_max']:.2e}")
    assert abs(ratio[12.0] - 1) < 0.04
    assert abs(ratio[12.0] - 1) < abs(ratio[8.0] - 1)


@pytest.mark.parametrize("q", QS)
@pytest.mark.parametrize("precision,rtol", [("fp32_storage", 2e-6), ("fp32", 2e-5)])
def test_reduced_precision_parity(precision, rtol, q):
    """FP32 storage (FP64 arithmetic, each stored population rounded stochastically) and FP32
    arithmetic against the FP64 oracle after 10 steps, relative to the largest population:
    a random mixture with interfaces everywhere and two tangent spheres."""
    cases = [inputs.random_mixture_3d(13, 11, 9, 4, tiny_fraction=0.0),
             inputs.spheres(30, 26, 22, [(0, 9.0, 13.0, 11.0, 6.0), (1, 21.0, 13.0, 11.0, 6.0)])]
    for rho in cases:
        g, o = _gpu(rho, 10, precision=precision, q=q), _oracle(rho, 10, q=q)
        err = np.abs(g - o).max() / np.abs(o).max()
        print(q, precision, rho.shape, "max rel |df|:", err)
        assert err <= rtol


@pytest.mark.parametrize("q", QS)
@pytest.mark.parametrize("precision,bar", [("fp32_storage", 1e-6), ("fp32", 1.2e-4)])
def test_reduced_precision_mass_drift(precision, bar, q):
    """Per-fluid mass over 2000 steps of two tangent spheres (R = 8, 40 x 32 x 32): FP32
    storage keeps the drift below 1e-6 (unbiased stochastic rounding), FP32 arithmetic below
    the 2D bar of one ulp (6e-8) per step (1.2e-4).  Stochastic rounding is deterministic:
    a second run gives the same bits."""
    rho = inputs.spheres(40, 32, 32, [(0, 12.0, 16.0, 16.0, 8.0), (1, 28.0, 16.0, 16.0, 8.0)])
    runs = []
    for _ in range(2 if precision == "fp32_storage" else 1):
        L = lbm3.Lattice3D(40, 32, 32, SIG, TAU, precision=precision, q=q).init(rho)
        try:
            m0 = L.observables()[0]["mass"]
            obs, r, _ = L.step(2000).observables(want_rho=True)
        finally:
            L.close()
        drift = np.abs(obs["mass"] / m0 - 1).max()
        print(q, precision, "mass drift over 2000 steps:", drift)
        assert obs["nonfinite"] == 0 and drift < bar
        runs.append(r)
    if len(runs) == 2:
        assert np.array_equal(runs[0], runs[1])


@pytest.mark.parametrize("precision,rtol", [("fp64", 1e-11), ("fp32", 2e-5)])
@pytest.mark.parametrize("q", QS)
@pytest.mark.parametrize("shape", [(28, 12, 2), (29, 13, 5), (56, 25, 1), (17, 31, 12), (33, 47, 3), (1, 40, 9), (130, 1, 4)])
def test_factored_march_at_the_edges_of_its_tiles(shape, q, precision, rtol):
    """Lattices whose sides are a tile's 28 x 12 (FP32: 28 x 20) columns, one more, ragged
    parts of them and a single node, with one to many planes per segment; the factored state
    after 1 step (read from the initial densities) and 4 (read from itself)."""
    nx, ny, nz = shape
    rho = inputs.random_mixture_3d(nx, ny, nz, 21, tiny_fraction=0.0)
    for steps in (1, 4):
        o = _oracle(rho, steps, q=q)
        err = np.abs(_gpu(rho, steps, q=q, precision=precision) - o).max() / np.abs(o).max()
        print(shape, q, precision, steps, err)
        assert err <= rtol


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("q", QS)
@pytest.mark.parametrize("cell,times", [((45, 19, 8), (5, 5, 1)), ((28, 24, 9), (8, 4, 1)), ((31, 5, 60), (3, 7, 3))])
def test_large_and_small_tiles_agree_bitwise(cell, times, q, precision):
    """A box small enough for tiles of 28 x 4 nodes, and the periodic repetition of it that takes
    the large tiles: node by node the same populations, bit for bit."""
    nx, ny, nz = cell
    rho = inputs.random_mixture_3d(nx, ny, nz, 22, tiny_fraction=0.0)
    reps = times[::-1]
    A = lbm3.Lattice3D(nx, ny, nz, SIG, TAU, q=q, precision=precision).init(rho)
    B = lbm3.Lattice3D(nx * times[0], ny * times[1], nz * times[2], SIG, TAU, q=q, precision=precision)
    B.init(np.ascontiguousarray(np.tile(rho, (1,) + reps)))
    fa, fb = A.step(3).state(), B.step(3).state()
    A.close()
    B.close()
    assert np.isfinite(fa).all()
    assert np.array_equal(np.tile(fa, (1,) * (fa.ndim - 3) + reps), fb)


def test_plane_beyond_32_bit_offsets_equals_the_2d_step():
    """A plane of 4.1 GiB (5000 x 3840 nodes, D3Q19, FP64) takes the march with 64-bit offsets;
    one plane deep, the lattice is uniform along z and its densities follow the two-dimensional
    step (1e-12, as in the uniform-lattice test)."""
    nx, ny = 5000, 3840
    w = inputs.droplet_tiling(nx if nx == ny else 256, cell=128, R=24.0)
    rho = np.ascontiguousarray(np.tile(w.rho, (1, -(-ny // 256), -(-nx // 256)))[:, :ny, :nx])
    L3 = lbm3.Lattice3D(nx, ny, 1, SIG, TAU).init(rho[:, None])
    r3 = L3.step(3).densities()[:, 0]
    L3.close()
    L2 = lbm3.Lattice(nx, ny, SIG, TAU).init(rho)
    r2 = L2.step(3).densities()
    L2.close()
    assert np.abs(r3 - r2).max() <= 1e-12


def _rounded_stochastically(v, rng):
    """Each value of v rounded to one of its two neighbouring floats, up with the probability
    that makes the expected value v."""
    a = v.astype(np.float32)
    up = np.nextafter(a, np.where(v > a, np.float32(np.inf), np.float32(-np.inf)), dtype=np.float32)
    gap = up.astype(float) - a
    return np.where(rng.random(v.shape) * np.abs(gap) < np.abs(v - a), up, a).astype(float)


@pytest.mark.parametrize("q", QS)
def test_fp32_storage_is_as_exact_as_populations_rounded_one_by_one(q):
    """A random mixture of three fluids on 20^3, 10 steps, FP32 storage: the densities' RMS error
    against the FP64 oracle is no larger than with all 3 Q populations held in FP32, each rounded
    stochastically (the oracle's step with that rounding, on the CPU).  The model's
    seeds lie within 3% of their mean; 5% allows for the GPU's own draw beside them."""
    rho = inputs.random_mixture_3d(20, 20, 20, 4, tiny_fraction=0.0)
    p = oracle.Params(20, 20, SIG, TAU)
    exact = d3.run(p, 20, d3.init(p, 20, rho, q), 10).sum(axis=1)
    rms = lambda r: float(np.sqrt(((r - exact) ** 2).mean()))  # noqa: E731
    model = []
    for seed in range(3):
        rng = np.random.default_rng(seed)
        f = d3.init(p, 20, rho, q).astype(np.float32).astype(float)
        for _ in range(10):
            f = _rounded_stochastically(d3.step(p, 20, f), rng)
        model.append(rms(f.sum(axis=1)))
    L = lbm3.Lattice3D(20, 20, 20, SIG, TAU, precision="fp32_storage", q=q).init(rho).step(10)
    err = rms(L.densities())
    L.close()
    print(q, "rms error", err, "3 Q populations", model)
    assert err <= 1.05 * np.mean(model)


@pytest.mark.parametrize("q", QS)
@pytest.mark.parametrize("r", [1.0, 0.9993, 0.87])
def test_fp32_fluid_at_rest_keeps_its_density(r, q):
    """A uniform fluid at rest, FP32, 60 steps: its density stays within 4 units of 2^-24.  A step's
    roundings (of the Q products w_i rho, and of their sum, small ones first) come to less than
    that, and the drift ends at a density that they leave as it is; summed link by link it went on
    to 8 units and more."""
    rho = np.zeros((3, 5, 13, 33))
    rho[2] = np.float32(r)
    L = lbm3.Lattice3D(33, 13, 5, (0.01,) * 3, precision="fp32", q=q).init(rho).step(60)
    d = (L.densities() - rho) * 2.0 ** 24
    L.close()
    print(q, r, d.min(), d.max())
    assert np.abs(d).max() <= 4


@pytest.mark.parametrize("q", QS)
def test_fp32_is_as_exact_as_populations_summed_in_fp32(q):
    """A random mixture of three fluids on 20^3, one step, FP32: the densities' RMS error against
    the FP64 oracle is no larger than that of the exact populations, each rounded to FP32, added
    one after another in FP32."""
    rho = inputs.random_mixture_3d(20, 20, 20, 4, tiny_fraction=0.0)
    p = oracle.Params(20, 20, SIG, TAU)
    f = d3.step(p, 20, d3.init(p, 20, rho, q))
    exact = f.sum(axis=1)
    model = np.zeros(exact.shape, np.float32)
    for i in range(q):
        model += f[:, i].astype(np.float32)
    rms = lambda r: float(np.sqrt(((r - exact) ** 2).mean()))  # noqa: E731
    L = lbm3.Lattice3D(20, 20, 20, SIG, TAU, precision="fp32", q=q).init(rho).step(1)
    err = rms(L.densities())
    L.close()
    print(q, "rms error", err, "populations", rms(model))
    assert err <= rms(model)
