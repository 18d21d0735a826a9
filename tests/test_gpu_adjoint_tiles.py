"""The two tiles of the adjoint step (32 x 8 with one node per thread on small
lattices, 64 x 8 with two above): a periodic state repeated over a larger
lattice gives the repeated adjoint and parameter sums in proportion, whichever
tile sweeps it."""
import numpy as np
import pytest
import torch

import paper_1809_02390_amd as pkg
import workloads as wl
from tests._gpu_helpers import params_pair

pytestmark = pytest.mark.gpu

NX, NY = 64, 48


def _sweep(nx, ny, f, lam):
    """Two adjoint steps through the same forward state."""
    lat = pkg.Lattice(nx, ny, tr=0.7).set_state(f)
    src = lat.save_state()
    a, b = lat.adjoint_seed(lam), lat.adjoint_buffer()
    out = lat.adjoint_run([src, src], a, b)
    got = lat.adjoint_get(out), np.array(lat.adjoint_theta())
    lat.close()
    return got


# 8 x 8 copies: 512 x 384, 768 tiles of 32 x 8 (the last size of the small
# tile on 256 CUs); 9 x 9: 576 x 432, 64 x 8 tiles; 1 x 13: one tile column.
@pytest.mark.parametrize("cx,cy", [(8, 8), (9, 9), (1, 13), (13, 1)])
def test_repeated_state_gives_repeated_adjoint(cx, cy):
    """Adjoints bitwise (each node's arithmetic does not depend on its tile);
    the parameter sums, FP64 sums of the same FP32 terms in another order, to
    1e-9 (2^-53 times some thousand additions and a cancellation up to 1e4)."""
    _, co = params_pair(NX, NY, tr=0.7)
    rho = wl.droplets(NX, NY, co.rho_g, co.rho_l, co.width, [(30, 22)], [14.0])
    u = wl._f32(np.random.default_rng(3).uniform(-0.02, 0.02, (2, NY, NX)))
    lat = pkg.Lattice(NX, NY, tr=0.7).init(rho, *u)
    f = lat.step(5).state()
    lat.close()
    lam = torch.randn((9, NY, NX), generator=torch.Generator(device="cuda").manual_seed(2), device="cuda")
    one, theta = _sweep(NX, NY, f, lam)
    rep = lambda t: t.repeat(1, cy, cx)
    many, theta_many = _sweep(NX * cx, NY * cy, rep(f), rep(lam))
    assert torch.equal(many, rep(one))
    assert np.abs(theta_many / (cx * cy) - theta).max() <= 1e-9 * np.abs(theta).max()


@pytest.mark.parametrize("nx,ny", [(33, 9), (97, 40), (36, 100), (129, 17), (1, 1), (3, 2)])
def test_ragged_small_tiles_match_repeated(nx, ny):
    """Remainder columns and rows of the small tile: a ragged lattice against
    its 2 x 2 repetition, whose tiles fall elsewhere; the parameter sums pair
    other rows there: to 1e-6 (FP32 sums of two terms)."""
    gen = torch.Generator(device="cuda").manual_seed(nx)
    _, co = params_pair(nx, ny, tr=0.7)
    rho = 0.5 * (co.rho_g + co.rho_l) + 0.02 * (torch.rand((ny, nx), generator=gen, device="cuda") - 0.5)
    lat = pkg.Lattice(nx, ny, tr=0.7).init(rho)
    f = lat.step(3).state()
    lat.close()
    lam = torch.randn((9, ny, nx), generator=gen, device="cuda")
    one, theta = _sweep(nx, ny, f, lam)
    rep = lambda t: t.repeat(1, 2, 2)
    many, theta_many = _sweep(2 * nx, 2 * ny, rep(f), rep(lam))
    assert torch.equal(many, rep(one))
    assert np.abs(theta_many / 4 - theta).max() <= 1e-6 * np.abs(theta).max()
