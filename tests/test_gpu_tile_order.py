"""Tile order and store policy of the step and adjoint kernels: on lattices
whose state is left in the caches, consecutive launches visit the tiles in
opposite directions.  Every direction gives the same bits, and the states
match the oracle."""
import numpy as np
import pytest
import torch

import paper_1809_02390_amd as pkg
import workloads as wl
from tests._gpu_helpers import device_samples, params_pair, sampled_oracle

pytestmark = pytest.mark.gpu


def _field(nx, ny, seed):
    _, co = params_pair(nx, ny, tr=0.7)
    return co, wl.uniform_noise(nx, ny, 0.5 * (co.rho_g + co.rho_l), 0.01, seed=seed)


# 800 x 801: rows on 64 bytes; 2600 x 257: strips of tiles with a narrower
# last one; 769 x 903: rows off 64 bytes; 900 x 905: two steps on 64 x 16
# tiles, the others on 64 x 24.  One-step states of 20 MiB and more.
@pytest.mark.parametrize("nx,ny", [(800, 801), (2600, 257), (769, 903), (900, 905)])
def test_launch_directions_agree_fp32(nx, ny):
    """Two launches in a row from the same buffers run in opposite
    directions: one-step kernel, adjoint kernel and its parameter sums
    bitwise equal; five steps (two launches of two steps, one of one)
    against the oracle at corner, edge and interior nodes, within the FP32
    gate of 1e-5 of rho_l."""
    co, rho = _field(nx, ny, 5)
    lat = pkg.Lattice(nx, ny, tr=0.7).init(rho)
    src, a, b = lat.save_state(), lat.checkpoint_buffer().zero_(), lat.checkpoint_buffer().zero_()
    lat.step_saved(src, a)
    lat.step_saved(src, b)
    assert torch.equal(a, b)
    lam = torch.randn((9, ny, nx), generator=torch.Generator(device="cuda").manual_seed(7), device="cuda")
    adj = lat.adjoint_seed(lam)
    got = []
    for _ in range(2):
        out = lat.adjoint_buffer().zero_()
        lat.adjoint_step(src, adj, out)
        got.append((lat.adjoint_get(out), lat.adjoint_theta()))
    assert torch.equal(got[0][0], got[1][0]) and got[0][1] == got[1][1]
    lat.step(5)
    pts = [(0, 0), (nx - 1, ny - 1), (nx - 1, 3), (nx // 2, ny // 2), (63, 24)]
    ref = sampled_oracle(co, rho, pts, 5)
    assert np.abs(device_samples(lat.state(), pts) - ref).max() <= 1e-5 * co.rho_l
    lat.close()


@pytest.mark.parametrize("storage", ["fp16", "bf16"])
def test_launch_directions_agree_2_byte(storage):
    """1061 x 1103 (states of 23 MB): a step repeated from the same
    checkpoint runs in the other direction and gives the same bits."""
    nx, ny = 1061, 1103
    _, rho = _field(nx, ny, 6)
    lat = pkg.Lattice(nx, ny, tr=0.7, storage=storage).init(rho)
    src = lat.save_state()
    first = lat.step(1).state()
    second = lat.load_state(src).step(1).state()
    assert torch.equal(first, second)
    lat.close()
