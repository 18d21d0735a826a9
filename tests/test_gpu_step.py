"""Parity of the HIP FP32 step with the FP64 oracle, element by element, on
seeded inputs; sampled parity at full workload sizes; physics properties of
the GPU results.  Tolerance: max |Delta rho| / rho_l <= 1e-5 (and the same
bound on every population)."""
import numpy as np
import pytest
import torch

import paper_1809_02390_amd as pkg
import workloads as wl
from oracle import lbm, measure
from tests._gpu_helpers import (crop_periodic, device_samples, fp32_state_of, lattice, oracle_init, params_pair,
                                sampled_oracle, sampled_oracle_moments)

pytestmark = pytest.mark.gpu
TOL = 1e-5


def droplet_case(nx, ny, tr=0.8, seed=0, du=0.02):
    _, co = params_pair(nx, ny, tr=tr)
    rho = wl.droplets(nx, ny, co.rho_g, co.rho_l, co.width, [(nx * 0.45, ny * 0.55)], [min(nx, ny) * 0.3])
    rng = np.random.default_rng(seed)
    ux, uy = (wl._f32(rng.uniform(-du, du, (ny, nx))) for _ in range(2))
    return co, rho, ux, uy


def compare(lat, f_ref, co, tol=TOL):
    f = lat.state().double().cpu().numpy()
    err_f = np.abs(f - f_ref).max() / co.rho_l
    err_r = np.abs(f.sum(0) - f_ref.sum(0)).max() / co.rho_l
    assert err_r <= tol and err_f <= tol, (err_r, err_f)
    return err_r


def test_init_is_equilibrium():
    co, rho, ux, uy = droplet_case(70, 37)
    lat = lattice(70, 37, rho, ux, uy, tr=0.8)
    assert lat.time == 0
    f = lat.state().double().cpu().numpy()
    assert np.abs(f - oracle_init(co, rho, ux, uy)).max() < 2e-7


def test_set_get_state_roundtrip_is_exact():
    co, rho, ux, uy = droplet_case(33, 21)
    f0 = torch.tensor(oracle_init(co, rho, ux, uy), dtype=torch.float32, device="cuda")
    lat = pkg.Lattice(33, 21, tr=0.8).set_state(f0)
    assert torch.equal(lat.state(), f0)


@pytest.mark.parametrize("nx,ny,steps", [(70, 37, 40), (64, 16, 25), (129, 17, 10), (5, 200, 20), (772, 37, 40),
                                         (1300, 410, 10), (1024, 256, 10), (1024, 512, 6)])
def test_step_parity_ragged(nx, ny, steps):
    """Several tiles and a ragged tail in both directions; 772 x 37 also has
    interior tiles (the fast addressing path) next to edge tiles.  The first
    chunk of one step runs the one-step kernel, on 64 x 4 tiles (all these
    lattices fit the caches; test_gpu_large_tiles.py has the 256 x 8 tiles).
    The rest runs several steps per launch: 4 x 4 tiles on the smallest, 8 x 8
    on 772 x 37, 16 x 16 on 1300 x 410, 64 x 16 on 1024 x 256 and 1024 x
    512."""
    co, rho, ux, uy = droplet_case(nx, ny, seed=nx)
    lat = lattice(nx, ny, rho, ux, uy, tr=0.8)
    f = oracle_init(co, rho, ux, uy)
    for chunk in (1, steps - 1):
        lat.step(chunk)
        f = lbm.run(f, co, chunk)
        compare(lat, f, co)
    assert lat.time == steps


def test_step_parity_sheared_droplet():
    """Moving interface with |u| up to 0.1: a 60 x 50 droplet at T_r = 0.6,
    W = 6 in a periodic velocity field.  A sign error in any single R, T or
    X entry (supplement Eqs. 34, 37, 40) moves the oracle's state after 10
    steps by >= 5e-5 rho_l (tests/test_oracle_step.py::
    test_sheared_droplet_sees_every_correction_entry), so this gate sees
    every entry of the cubic-velocity corrections of the kernel."""
    _, co = params_pair(60, 50, tr=0.6, width=6.0)
    rho, ux, uy = wl.sheared_droplet(co)
    lat = lattice(60, 50, rho, ux, uy, tr=0.6, width=6.0)
    f = oracle_init(co, rho, ux, uy)
    for chunk in (1, 4, 5):
        lat.step(chunk)
        f = lbm.run(f, co, chunk)
        compare(lat, f, co)
    assert lat.time == 10


@pytest.mark.parametrize("nx,ny", [(1, 1), (1, 64), (3, 2), (2, 5), (64, 1)])
def test_step_parity_degenerate(nx, ny):
    """Lattices narrower than the stencil: periodic images of a node are its
    own neighbours.  One step (the one-step kernel), then 19 (up to four
    steps per launch on 4 x 4 tiles)."""
    _, co = params_pair(nx, ny, tr=0.7)
    rng = np.random.default_rng(nx * 100 + ny)
    if nx == 1 and ny == 64:
        rho = wl.flat_slab(1, 64, co.rho_g, co.rho_l, 3.0)
    else:
        rho = wl._f32(rng.uniform(0.15, 0.21, (ny, nx)))
    lat = lattice(nx, ny, rho, tr=0.7)
    f = oracle_init(co, rho)
    for chunk in (1, 19):
        lat.step(chunk)
        f = lbm.run(f, co, chunk)
        compare(lat, f, co)


def test_uniform_state_is_fixed_point():
    rho = np.full((16, 64), 0.2, np.float32)
    lat = lattice(64, 16, rho, tr=0.7)
    f0 = lat.state().clone()
    lat.step(10)
    assert torch.allclose(lat.state(), f0, rtol=0, atol=2e-8)


def test_flat_slab_5000_steps():
    """64x64 slab (tanh length W, noise 1e-4, seed 1), T_r = 0.8, W = 10:
    density parity every 1000 steps up to 5000, and conservation."""
    _, co = params_pair(64, 64, tr=0.8, width=10.0)
    rho = wl.slab_64(co)
    lat = lattice(64, 64, rho, tr=0.8, width=10.0)
    m0 = lat.moments(fields=False)
    f = oracle_init(co, rho)
    worst = 0.0
    for _ in range(5):
        lat.step(1000)
        f = lbm.run(f, co, 1000, lbm.collide_sequence)
        r_gpu = lat.moments()[0].double().cpu().numpy()
        worst = max(worst, np.abs(r_gpu - f.sum(0)).max() / co.rho_l)
    assert worst <= TOL, worst
    m1 = lat.moments(fields=False)
    assert abs(m1[0] - m0[0]) / m0[0] < 1e-6
    assert abs(m1[1]) < 1e-6 * m0[0] and abs(m1[2]) < 1e-6 * m0[0]


def test_moments_fields_and_totals():
    co, rho, ux, uy = droplet_case(70, 37, seed=9)
    lat = lattice(70, 37, rho, ux, uy, tr=0.8)
    lat.step(30)
    f = lbm.run(oracle_init(co, rho, ux, uy), co, 30)
    r_ref, ux_ref, uy_ref = lbm.macroscopic(f, co)
    r, u, v, tot = lat.moments()
    assert np.abs(r.double().cpu().numpy() - r_ref).max() / co.rho_l < TOL
    assert np.abs(u.double().cpu().numpy() - ux_ref).max() < 1e-5
    assert np.abs(v.double().cpu().numpy() - uy_ref).max() < 1e-5
    mass, jx, jy = measure.totals(f)
    assert tot[0] == pytest.approx(mass, rel=1e-6)
    assert abs(tot[1] - jx) < 1e-6 * mass and abs(tot[2] - jy) < 1e-6 * mass


@pytest.mark.parametrize("nx,ny,n", [(4096, 1024, 6), (1000, 700, 5), (2048 + 37, 1024 + 11, 7),
                                     (16384, 8192, 2), (16384, 1, 3), (20000, 9, 4), (7, 60000, 4),
                                     (70, 9000, 3), (512, 512, 5), (600, 583, 4), (256, 256, 7),
                                     (300, 200, 6), (37, 29, 5), (5, 200, 3), (64, 1, 4), (3, 2, 5),
                                     (1, 1, 4)])
def test_two_step_launches_match_single_steps(nx, ny, n):
    """lbm_step(n) on FP32 lattices runs two steps per launch in marching
    strips (16384 x 8192), on 64 x 24 tiles (4096 x 1024 and others), 64 x 16
    (512^2) or 16 x 16 (20000 x 9), and up to four on smaller ones (32 x 8 on
    256^2, 4 x 4 on 37 x 29): interior tiles with 32-bit offsets, edge tiles
    with wrapped 64-bit addresses, ragged tiles, an odd remainder as one
    single step, a state above 4 GiB, and lattices thinner than the loaded
    region, down to one node, where it wraps more than once: bitwise the
    result of n calls of lbm_step(1)."""
    _, co = params_pair(nx, ny, tr=0.7, width=10.0)
    rng = np.random.default_rng(nx + ny)
    rho = wl._f32(0.5 * (co.rho_g + co.rho_l) + rng.uniform(-0.01, 0.01, (ny, nx)))
    a = lattice(nx, ny, rho, tr=0.7, width=10.0)
    for _ in range(n):
        a.step(1)
    fa = a.state()
    a.close()
    b = lattice(nx, ny, rho, tr=0.7, width=10.0).step(n)
    assert b.time == n and torch.equal(b.state(), fa)


@pytest.mark.parametrize("nx,ny", [(1000, 700), (512, 512), (300, 200)])
def test_two_step_chain_matches_single_steps(nx, ny):
    """lbm_step_saved_chain over distinct buffers (several steps per launch,
    the states between them written too; 64 x 24, 64 x 16 and 32 x 8 tiles)
    and over alternating buffers (one step per launch): bitwise
    lbm_step_saved, step by step."""
    n = 5
    _, co = params_pair(nx, ny, tr=0.7, width=10.0)
    rho = wl.droplets(nx, ny, co.rho_g, co.rho_l, co.width, [(0.4 * nx, 0.43 * ny), (0.65 * nx, 0.6 * ny)],
                      [0.17 * min(nx, ny), 0.13 * min(nx, ny)])
    lat = lattice(nx, ny, rho, tr=0.7, width=10.0)
    single = [lat.save_state()] + [lat.checkpoint_buffer() for _ in range(n)]
    for j in range(n):
        lat.step_saved(single[j], single[j + 1])
    distinct = [single[0]] + [lat.checkpoint_buffer() for _ in range(n)]
    lat.step_saved_chain(distinct)
    alternating = [single[0], lat.checkpoint_buffer(), lat.checkpoint_buffer()]
    alternating = [alternating[0]] + [alternating[1 + j % 2] for j in range(n)]
    lat.step_saved_chain(alternating)
    state = lambda b: fp32_state_of(b, nx, ny)
    assert all(torch.equal(state(x), state(y)) for x, y in zip(single, distinct))
    assert torch.equal(state(alternating[-1]), state(single[-1]))


# Every problem parameter away from its default: s_p and varpi (with s_q,
# s_e and the model coefficients they set, main Eqs. 7 and 16), s_eps given
# instead of s_e, b and T_r of the Carnahan-Starling EOS, sigma given
# instead of the sound-speed rule, and W.  In the oracle, putting any one of
# s_p, s_eps, varpi, b, T_r, sigma or W of this set back to its default
# moves some population of the 200 x 70 droplet after 6 steps by
# >= 1.6e-3 rho_l, 160 times the bound.  a and R change nothing at a given
# sigma (K_EOS absorbs them: the oracle's states agree bitwise).
NONDEFAULT = dict(s_p=0.8, s_eps=1.4, varpi=0.12, a=0.5, b=2.5, r_gas=1.5, tr=0.85, sigma=0.0021, width=12.0)


@pytest.mark.parametrize("nx,ny", [(200, 70), (1024, 384)])
def test_step_parity_nondefault_parameters(nx, ny):
    """Parity at NONDEFAULT after one step (the one-step kernel) and after
    five more: 200 x 70 (up to four steps per launch, 8 x 8 tiles) and 1024
    x 384 (two, 64 x 24 tiles, one per CU)."""
    _, co = params_pair(nx, ny, **NONDEFAULT)
    rho = wl.droplets(nx, ny, co.rho_g, co.rho_l, co.width, [(nx * 0.45, ny * 0.55)], [min(nx, ny) * 0.3])
    rng = np.random.default_rng(nx)
    ux, uy = (wl._f32(rng.uniform(-0.02, 0.02, (ny, nx))) for _ in range(2))
    lat = lattice(nx, ny, rho, ux, uy, **NONDEFAULT)
    f = oracle_init(co, rho, ux, uy)
    for chunk in (1, 5):
        lat.step(chunk)
        f = lbm.run(f, co, chunk)
        compare(lat, f, co)


def test_deterministic():
    co, rho, ux, uy = droplet_case(96, 80, seed=4)
    a = lattice(96, 80, rho, ux, uy, tr=0.8)
    b = lattice(96, 80, rho, ux, uy, tr=0.8)
    a.step(50)
    b.step(50)
    assert torch.equal(a.state(), b.state())
    assert a.moments(fields=False) == b.moments(fields=False)


def test_errors_from_device_calls():
    with pytest.raises(pkg.LbmError):
        pkg.Lattice(8, 8, tr=0.8).step(1)  # not initialised
    lat = pkg.Lattice(8, 8, tr=0.8)
    with pytest.raises(pkg.LbmError) as e:
        lat.init(np.full((8, 8), 2.0, np.float32))  # beyond the packing limit 4/b = 1
    assert e.value.status == pkg.lbm.LBM_EINVAL
    with pytest.raises(pkg.LbmError):
        lat.init(np.full((8, 8), -0.1, np.float32))
    lat.init(np.full((8, 8), 0.2, np.float32))
    with pytest.raises(pkg.LbmError):
        lat.step(-1)


def test_sampled_parity_spinodal_4096():
    """Full 4096^2 spinodal workload (T_r = 0.7, mean of the coexistence
    densities +- 0.01, seed 3): sampled nodes after 20 steps against oracle
    light-cone crops, including nodes on the periodic boundary."""
    n, steps = 4096, 20
    _, co = params_pair(n, n, tr=0.7, width=10.0)
    rho = wl.spinodal(co, n=n)
    lat = lattice(n, n, rho, tr=0.7, width=10.0)
    lat.step(steps)
    pts = [(0, 0), (n - 1, n - 1), (0, n - 1), (n - 1, 7), (63, 15), (64, 16), (2047, 2048), (1234, 3071),
           (4000, 100), (17, 4095)]
    ref = sampled_oracle(co, rho, pts, steps)
    got = device_samples(lat.state(), pts)
    assert np.abs(got - ref).max() / co.rho_l <= TOL
    tot = lat.moments(fields=False)
    assert tot[0] == pytest.approx(float(rho.sum()), rel=1e-6)


def test_window_parity_spinodal_4096_late_times():
    """The same workload over its 2000 steps, in 100-step windows starting at
    t0 = 0, 500, 1000, 1500 and 1900: oracle runs on light-cone crops of the GPU state
    at t0 (half-width 2 x 100 + 3: one step moves information two nodes,
    streaming plus stencil) and is compared on the 5 x 5 nodes around each
    crop's centre at t0 + 100.  Late windows see developed interfaces, with
    velocities and gradients far from the initial noise."""
    n, window = 4096, 100
    _, co = params_pair(n, n, tr=0.7, width=10.0)
    rho = wl.spinodal(co, n=n)
    lat = lattice(n, n, rho, tr=0.7, width=10.0)
    half = 2 * window + 3
    centres = {0: [(2047, 2048)], 500: [(1500, 2600), (4095, 0)], 1000: [(3000, 700)], 1500: [(9, 2222)],
               1900: [(300, 3333)]}
    for t0 in sorted(centres):
        lat.step(t0 - lat.time)
        st = lat.state()
        crops = [crop_periodic(st, cx, cy, half).double().cpu().numpy() for cx, cy in centres[t0]]
        del st
        lat.step(window)
        st = lat.state()
        for (cx, cy), crop in zip(centres[t0], crops):
            # the crop's own periodic seam is not the lattice's: it may blow
            # up, but it lies 201 nodes from the compared ones, outside the
            # 200-node reach of 100 steps
            with np.errstate(over="ignore", invalid="ignore", divide="ignore"):
                ref = lbm.run(crop, co, window, lbm.collide_sequence)[:, half - 2:half + 3, half - 2:half + 3]
            assert np.all(np.isfinite(ref))
            got = crop_periodic(st, cx, cy, 2).double().cpu().numpy()
            err = np.abs(got - ref).max() / co.rho_l
            assert err <= TOL, (t0, cx, cy, err)
        del st


def test_window_parity_droplet_256():
    """The 256^2 Laplace droplet (R = 40, T_r = 0.8, W = 10) over 20000
    steps: from the GPU state at t0 = 2000, 10000 and 19900, 100 oracle
    steps on the whole periodic lattice against the GPU's next 100 steps."""
    n = 256
    _, co = params_pair(n, n, tr=0.8, width=10.0)
    lat = lattice(n, n, wl.static_droplet(co, n, 40.0), tr=0.8, width=10.0)
    for t0 in (2000, 10000, 19900):
        lat.step(t0 - lat.time)
        f0 = lat.state().double().cpu().numpy()
        lat.step(100)
        compare(lat, lbm.run(f0, co, 100, lbm.collide_sequence), co)


def test_window_parity_coalescence_16384x8192():
    """Largest workload, 100-step window from t0 = 1000 on a light-cone crop
    through the gap between the droplets."""
    nx, ny, t0, window = 16384, 8192, 1000, 100
    _, co = params_pair(nx, ny, tr=0.6, width=10.0)
    lat = lattice(nx, ny, wl.coalescence(co, nx, ny), tr=0.6, width=10.0)
    lat.step(t0)
    half, c = 2 * window + 3, (nx // 2 - 7, ny // 2 + 30)  # in the gap, in the left droplet's interface
    st = lat.state()
    crop = crop_periodic(st, *c, half).double().cpu().numpy()
    del st
    lat.step(window)
    st = lat.state()
    got = crop_periodic(st, *c, 2).double().cpu().numpy()
    del st
    with np.errstate(over="ignore", invalid="ignore", divide="ignore"):  # crop seam, outside the light cone
        ref = lbm.run(crop, co, window, lbm.collide_sequence)[:, half - 2:half + 3, half - 2:half + 3]
    assert np.all(np.isfinite(ref))
    assert np.abs(got - ref).max() / co.rho_l <= TOL


def test_sampled_parity_coalescence_16384x8192():
    """Largest workload: two R = 400 droplets 20 nodes apart, T_r = 0.6."""
    nx, ny, steps = 16384, 8192, 5
    _, co = params_pair(nx, ny, tr=0.6, width=10.0)
    rho = wl.coalescence(co, nx, ny)
    lat = lattice(nx, ny, rho, tr=0.6, width=10.0)
    lat.step(steps)
    cx = nx // 2
    pts = [(cx, ny // 2), (cx - 10, ny // 2), (cx - 410 - 400, ny // 2), (cx + 410, ny // 2 + 400), (0, 0),
           (nx - 1, ny - 1)]
    ref = sampled_oracle(co, rho, pts, steps)
    st = lat.state()
    got = device_samples(st, pts)
    del st
    assert np.abs(got - ref).max() / co.rho_l <= TOL


def test_sampled_parity_largest_lattice():
    """The largest lattice the library accepts, 16384 x 14563 (9 nx ny just
    below 2^31; its FP32 state, 8.6 GB, is read relative to each tile's row
    band and, in the tile rows that wrap, with 64-bit addresses): the spinodal
    field (T_r = 0.7, mean of the coexistence densities +- 0.01, seed 3),
    5 steps, sampled nodes against oracle light-cone crops, including the
    last row and column; rho and u from lbm_moments at the same nodes and
    the FP64 total mass."""
    nx, ny, steps = 16384, 14563, 5
    _, co = params_pair(nx, ny, tr=0.7, width=10.0)
    rho = wl.uniform_noise(nx, ny, 0.5 * (co.rho_g + co.rho_l), 0.01, seed=3)
    lat = lattice(nx, ny, rho, tr=0.7, width=10.0)
    lat.step(steps)
    pts = [(nx // 2, ny // 2), (0, 0), (nx - 1, ny - 1), (0, ny - 1), (nx - 1, 0), (12345, ny - 2), (nx - 3, 9999)]
    ref = sampled_oracle(co, rho, pts, steps)
    st = lat.state()
    got = device_samples(st, pts)
    del st
    assert np.abs(got - ref).max() / co.rho_l <= TOL
    # moments of the same state (64-bit addresses for this size)
    ref_m = sampled_oracle_moments(co, rho, pts, steps)
    r, u, v, tot = lat.moments()
    got_m = np.array([[float(a[y, x]) for a in (r, u, v)] for (x, y) in pts])
    del r, u, v
    lat.close()
    assert np.abs(got_m[:, 0] - ref_m[:, 0]).max() / co.rho_l <= TOL
    assert np.abs(got_m[:, 1:] - ref_m[:, 1:]).max() < 1e-5
    assert tot[0] == pytest.approx(float(np.asarray(rho, np.float32).astype(np.float64).sum()), rel=1e-6)


@pytest.mark.parametrize("nx,ny", [(16384, 7281), (16384, 7282), (16400, 8003)])
def test_sampled_parity_at_the_row_layout_limit(nx, ny):
    """FP32 states are read through 32-bit offsets from uniform bases while
    36 nx ny < 2^32: 16384 x 7281 is the tallest such lattice of that width
    (largest offset 4 294 508 540 bytes); 16384 x 7282 is the first read
    relative to each tile's row band, with 64-bit addresses for the tile
    rows that wrap; 16400 x 8003 does the same with a partial last tile
    column and a partial last tile row.  Spinodal field (T_r = 0.7), 5
    steps, sampled nodes against oracle crops, including the last row and
    column and nodes next to tile edges."""
    steps = 5
    assert (36 * nx * ny < 2 ** 32) == (ny == 7281)
    _, co = params_pair(nx, ny, tr=0.7, width=10.0)
    rho = wl.uniform_noise(nx, ny, 0.5 * (co.rho_g + co.rho_l), 0.01, seed=ny)
    lat = lattice(nx, ny, rho, tr=0.7, width=10.0)
    lat.step(steps)
    pts = [(nx - 1, ny - 1), (0, ny - 1), (nx // 2, ny - 2), (0, 0), (nx - 1, 0), (777, ny // 2),
           (nx - 17, ny - 3), (16383 % nx, 8), (255, 7), (256, ny - 9)]
    ref = sampled_oracle(co, rho, pts, steps)
    st = lat.state()
    got = device_samples(st, pts)
    del st
    lat.close()
    assert np.abs(got - ref).max() / co.rho_l <= TOL


@pytest.mark.parametrize("nx,ny", [(4_000_000, 59), (11_000_000, 21)])
def test_sampled_parity_widest_lattices(nx, ny):
    """Lattices near the node limit (9 nx ny < 2^31) in extreme aspect: at
    4M nodes wide the two-step kernel's 32-bit band offsets would not fit
    (single steps; the one-step kernel's band rows do), at 11M wide neither
    does and every tile row takes 64-bit addresses.  Spinodal field, 5
    steps, sampled nodes against oracle crops."""
    steps = 5
    assert 9 * nx * ny < 2 ** 31 and 36 * nx * ny >= 2 ** 32
    _, co = params_pair(nx, ny, tr=0.7, width=10.0)
    rho = wl.uniform_noise(nx, ny, 0.5 * (co.rho_g + co.rho_l), 0.01, seed=ny)
    lat = lattice(nx, ny, rho, tr=0.7, width=10.0)
    lat.step(steps)
    pts = [(nx - 1, ny - 1), (0, ny - 1), (nx // 2, ny - 2), (0, 0), (nx - 1, 0), (777, ny // 2),
           (nx - 17, ny - 3), (3_999_999 % nx, 8), (255, 7), (nx - 300, 12)]
    ref = sampled_oracle(co, rho, pts, steps)
    del rho
    st = lat.state()
    got = device_samples(st, pts)
    del st
    lat.close()
    assert np.abs(got - ref).max() / co.rho_l <= TOL


def test_two_lattices_on_two_streams_match_single_runs():
    """Every launch goes to its context's stream and contexts share no device
    state: two lattices (FP32 and FP16) stepped in turn on two streams end
    with the bits of the same runs made alone on the default stream."""
    nx, ny, chunks = 300, 200, 10
    _, co = params_pair(nx, ny, tr=0.7, width=10.0)
    rho_a = wl.droplets(nx, ny, co.rho_g, co.rho_l, co.width, [(100, 90)], [30.0])
    rho_b = wl.droplets(nx, ny, co.rho_g, co.rho_l, co.width, [(200, 120), (60, 50)], [25.0, 20.0])
    sa, sb = torch.cuda.Stream(), torch.cuda.Stream()
    la = pkg.Lattice(nx, ny, stream=sa, tr=0.7, width=10.0).init(rho_a)
    lb = pkg.Lattice(nx, ny, stream=sb, tr=0.7, width=10.0, storage="fp16").init(rho_b)
    for _ in range(chunks):
        la.step(20)
        lb.step(20)
    torch.cuda.synchronize()
    got = (la.state(), lb.state())
    torch.cuda.synchronize()
    ref_a = pkg.Lattice(nx, ny, tr=0.7, width=10.0).init(rho_a).step(20 * chunks).state()
    ref_b = pkg.Lattice(nx, ny, tr=0.7, width=10.0, storage="fp16").init(rho_b).step(20 * chunks).state()
    torch.cuda.synchronize()
    assert torch.equal(got[0], ref_a) and torch.equal(got[1], ref_b)


def test_side_stream_results_follow_torch_stream_order():
    """A lattice on a side stream, used from torch's current stream with no
    explicit synchronisation: every call orders its stream after the
    current one and the current one after it, so results read on the
    current stream are complete, and tensors freed on it are not reused
    while the library still reads them."""
    nx, ny = 600, 400
    _, co = params_pair(nx, ny, tr=0.7, width=10.0)
    rho = wl.droplets(nx, ny, co.rho_g, co.rho_l, co.width, [(300, 200)], [60.0])
    ref = lattice(nx, ny, rho, tr=0.7, width=10.0).step(300)
    ref_f, ref_rho = ref.state(), ref.moments()[0]
    side = torch.cuda.Stream()
    lat = pkg.Lattice(nx, ny, stream=side, tr=0.7, width=10.0)
    rho_dev = torch.tensor(rho, dtype=torch.float32, device="cuda")  # written on the current stream
    lat.init(rho_dev)
    del rho_dev
    lat.step(300)  # queued on the side stream
    f = lat.state()  # read back on the current stream without synchronising
    assert torch.equal(f, ref_f)
    r, _, _, _ = lat.moments()
    assert torch.equal(r, ref_rho)


@pytest.mark.parametrize("storage", ["fp32", "fp16", "bf16"])
def test_laplace_law_256(storage):
    """Static droplets R = 20..60 on 256^2 (T_r = 0.8, W = 10, sigma_paper),
    relaxed for 80000 steps (the breathing mode has decayed by 60000).  The
    slope of Delta p against 1/R fitted over R in {20..60} is reported; the
    R = 20 droplet (W/R = 0.5) is mostly interface and its pressure jump
    falls 8 % short of sigma/R in FP32 too, a finite-thickness effect of the
    model (at W = 5 the same droplet is within 3 %:
    test_laplace_small_droplet_thin_interface), so the gated fit is over
    R >= 30: within 3 % of sigma, each R >= 40 within 3 %, R = 20 within 10 %.
    Spurious currents (no bound in the paper) must stay below 1e-3 in
    lattice units.  FP16 storage keeps every bound.  BF16 storage (8-bit
    significand) keeps them for R >= 30; its R = 20 droplet ends between
    radius 13 and 15.7 (FP32: 15.4) depending only on how its rounding falls
    (three equally valid reference fits, same significand), so there it must
    only survive, with its ratio reported."""
    n = 256
    _, co = params_pair(n, n, tr=0.8, width=10.0)
    inv_r, dps, report = [], [], []
    for R in (20, 30, 40, 50, 60):
        lat = lattice(n, n, wl.static_droplet(co, n, R), tr=0.8, width=10.0, storage=storage)
        lat.step(80000)
        r, ux, uy, _ = lat.moments()
        r = r.double().cpu().numpy()
        sigma, radius, dp = measure.laplace_sigma(r, (n // 2, n // 2), co)
        umax = float(torch.hypot(ux, uy).max())
        inv_r.append(1.0 / radius)
        dps.append(dp)
        report.append((R, round(radius, 3), round(sigma / co.sigma, 4), umax))
    slope_all = np.polyfit(inv_r, dps, 1)[0]
    slope = np.polyfit(inv_r[1:], dps[1:], 1)[0]
    print(storage, "R, measured R, sigma/sigma_prescribed, max|u|:", report,
          f"slope / sigma: R 20..60 {slope_all / co.sigma:.4f}, R 30..60 {slope / co.sigma:.4f}")
    assert slope == pytest.approx(co.sigma, rel=0.03), (slope / co.sigma, report)
    for R, radius, ratio, umax in report:
        assert umax < 1e-3, report
        if storage == "bf16" and R == 20:
            assert radius > 10.0, report
            continue
        assert ratio == pytest.approx(1.0, abs=0.03 if R >= 40 else 0.10), report


def test_laplace_small_droplet_thin_interface():
    """The R = 20 droplet with a thinner interface, W = 5 (W/R = 0.25, the
    ratio of the R = 40, W = 10 droplet): its pressure jump is within 3 % of
    sigma/R, so the 8 % shortfall at W = 10 comes from W/R = 0.5, not from
    the droplet's size on the lattice."""
    n = 256
    _, co = params_pair(n, n, tr=0.8, width=5.0)
    lat = lattice(n, n, wl.static_droplet(co, n, 20.0), tr=0.8, width=5.0)
    lat.step(80000)
    r = lat.moments()[0].double().cpu().numpy()
    sigma, radius, _ = measure.laplace_sigma(r, (n // 2, n // 2), co)
    print(f"R = 20, W = 5: radius {radius:.3f}, sigma / sigma_prescribed {sigma / co.sigma:.4f}")
    assert sigma / co.sigma == pytest.approx(1.0, abs=0.03)


def test_coexistence_and_width_gpu():
    """64x64 slab relaxed for 20000 steps: Maxwell densities and W."""
    _, co = params_pair(64, 64, tr=0.8, width=10.0)
    lat = lattice(64, 64, wl.flat_slab(64, 64, co.rho_g, co.rho_l, co.width / wl.TANH_WIDTH_FACTOR),
                  tr=0.8, width=10.0)
    lat.step(20000)
    prof = lat.moments()[0].double().cpu().numpy()[:, 5]
    g, l = measure.bulk_densities(prof)
    assert abs(l - co.rho_l) / co.rho_l < 1e-3
    assert abs(g - co.rho_g) / co.rho_g < 3e-3
    assert measure.interface_width(prof, g, l) == pytest.approx(co.width, rel=0.02)
