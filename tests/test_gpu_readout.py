"""Read-outs and initial states: totals with and without the fields, sums over
more workgroups than one round of the final reduction, the cleared parameter
accumulator, refused initial densities, and more contexts than the pinned
result page holds."""
import numpy as np
import pytest
import torch

import paper_1809_02390_amd as pkg
import workloads as wl
from tests._gpu_helpers import oracle_init, params_pair

pytestmark = pytest.mark.gpu


def _lat(nx, ny, storage="fp32", vel=False, tr=0.7):
    _, co = params_pair(nx, ny, tr=tr)
    rho = wl.uniform_noise(nx, ny, 0.5 * (co.rho_g + co.rho_l), 0.01, seed=nx)
    u = wl._f32(np.random.default_rng(ny).uniform(-0.02, 0.02, (2, ny, nx))) if vel else (None, None)
    return co, rho, u, pkg.Lattice(nx, ny, tr=tr, storage=storage).init(rho, *u)


# 2085 x 1035: 2145 workgroups of 64 x 16 (the final sum keeps eight loads of
# 256 partials in flight: one round and a remainder); 64 x 16: one; 300 x 200
# and 65 x 33: partial tiles.
@pytest.mark.parametrize("nx,ny", [(2085, 1035), (64, 16), (300, 200), (65, 33), (1, 1)])
@pytest.mark.parametrize("storage", ["fp32", "fp16"])
def test_totals(nx, ny, storage):
    """Totals alone equal the totals beside the fields bit for bit; the mass
    is the FP64 sum of the density field to 1e-12 (sums of at most some
    thousand terms in a row, 2^-53 each); the momenta those of the exported populations, whose FP32 node
    sums may round differently: 8 x 2^-24 of the sum of |f|."""
    _, _, _, lat = _lat(nx, ny, storage, vel=True)
    lat.step(2)
    rho, ux, uy, tot = lat.moments()
    assert lat.moments(fields=False) == tot
    mass = rho.double().sum().item()
    assert abs(tot[0] - mass) <= 1e-12 * mass
    f = lat.state().double()
    jx = (f[1] - f[3] + f[5] - f[6] - f[7] + f[8]).sum().item()
    jy = (f[2] - f[4] + f[5] + f[6] - f[7] - f[8]).sum().item()
    bound = 8 * 2.0 ** -24 * f.abs().sum().item()
    assert abs(tot[1] - jx) <= bound and abs(tot[2] - jy) <= bound
    lat.close()


@pytest.mark.parametrize("vel", [False, True])
def test_initial_state_matches_oracle(vel):
    """300 x 201: the initial populations at rest and with velocities, to
    1e-6 of rho_l (a dozen FP32 roundings of terms up to rho_l)."""
    nx, ny = 300, 201
    co, rho, u, lat = _lat(nx, ny, vel=vel)
    ref = oracle_init(co, rho, *u)
    assert np.abs(lat.state().double().cpu().numpy() - ref).max() <= 1e-6 * co.rho_l
    lat.close()


@pytest.mark.parametrize("nx,ny,storage", [(2560, 1603, "fp32"), (4096, 2117, "fp16"), (4096, 2117, "bf16")])
def test_initial_state_by_tiles(nx, ny, storage):
    """Large lattices, partial last tile rows: the state at rest is that of
    zero velocities, stored node by node, bit for bit; and a bad density is
    seen.  2-byte states of this size are stored by tiles (whole rows on 64
    bytes, above 144 MiB); FP32 ones in test_gpu_large_tiles.py."""
    _, rho, _, lat = _lat(nx, ny, storage)
    rho = torch.as_tensor(rho, dtype=torch.float32, device="cuda")
    zero = torch.zeros((ny, nx), device="cuda")
    rest = lat.init(rho).save_state()
    moving = lat.init(rho, zero, zero).save_state()
    used = 9 * nx * ny * (4 if storage == "fp32" else 2)
    assert torch.equal(rest[:used], moving[:used])
    if storage != "fp32":
        assert torch.equal(rest[-2 * nx * ny:], moving[-2 * nx * ny:])
    for at in ((0, 0), (ny - 1, nx - 1)):
        bad = rho.clone()
        bad[at] = float("nan")
        with pytest.raises(pkg.LbmError):
            lat.init(bad)
    lat.close()


@pytest.mark.parametrize("nx,ny", [(1, 1), (3, 2), (70, 37), (512, 512), (2085, 1035), (2560, 1603)])
def test_loaded_state_is_exported_unchanged(nx, ny):
    """lbm_set_state and lbm_get_state of FP32 states: a permutation and its
    inverse, bit for bit."""
    f = torch.randn((9, ny, nx), generator=torch.Generator(device="cuda").manual_seed(nx), device="cuda")
    lat = pkg.Lattice(nx, ny, tr=0.7).set_state(f)
    assert torch.equal(lat.state(), f)
    lat.close()


def test_refused_densities_leave_no_state():
    """A density outside (0, 4/b) or not finite is refused, and a later good
    field is accepted."""
    nx, ny = 70, 37
    _, rho, _, lat = _lat(nx, ny)
    for bad in (0.0, -0.1, 1.0, float("nan"), float("inf")):
        field = torch.as_tensor(rho, dtype=torch.float32, device="cuda").clone()
        field[ny - 1, nx - 1] = bad
        with pytest.raises(pkg.LbmError):
            lat.init(field)
        with pytest.raises(pkg.LbmError):
            lat.step(1)
    u = torch.zeros((ny, nx), device="cuda")
    u[0, 0] = float("inf")
    with pytest.raises(pkg.LbmError):
        lat.init(rho, u, None)
    assert lat.init(rho).step(1).time == 1
    lat.close()


def test_parameter_sums_cleared_once_read():
    """The accumulator read with reset: the same value without and with it,
    then zero (520 x 1040: 1170 workgroups of 64 x 8)."""
    nx, ny = 520, 1040
    _, _, _, lat = _lat(nx, ny)
    lam = torch.randn((9, ny, nx), generator=torch.Generator(device="cuda").manual_seed(1), device="cuda")
    a, b = lat.adjoint_seed(lam), lat.adjoint_buffer()
    lat.adjoint_step(lat.save_state(), a, b)
    first, second, third = lat.adjoint_theta(reset=False), lat.adjoint_theta(), lat.adjoint_theta()
    assert first == second and third == (0.0, 0.0, 0.0) and any(first)
    lat.close()


def test_many_contexts_return_their_own_results():
    """70 contexts at a time, twice: each returns its own mass."""
    for _ in range(2):
        lats = [pkg.Lattice(16, 8, tr=0.7).init(torch.full((8, 16), 0.1 + 0.001 * k)) for k in range(70)]
        for k, lat in enumerate(lats):
            assert lat.moments(fields=False)[0] == pytest.approx(128 * np.float32(0.1 + 0.001 * k), rel=1e-6)
        for lat in lats:
            lat.close()
