"""Two FP32 steps per launch on lattices large enough for workgroups that walk
down strips of 960 columns: bitwise the single steps, and within the FP32 gate
of the oracle across strips, segments and the wrap."""
import numpy as np
import pytest
import torch

import paper_1809_02390_amd as pkg
import workloads as wl
from tests._gpu_helpers import device_samples, params_pair, sampled_oracle

pytestmark = pytest.mark.gpu


# 960 x 10000: one full strip and no other; 1859 x 6007: a last strip of 899
# columns, one segment per workgroup; 2300 x 5003: of 380, two segments;
# 1000 x 14000: of 40, eight; 3841 x 4099: of one column, sixteen, and an odd
# number of rows whose last segment is short.
@pytest.mark.parametrize("nx,ny", [(960, 10000), (1859, 6007), (2300, 5003), (1000, 14000), (3841, 4099)])
def test_marching_matches_single_steps(nx, ny):
    """Five steps (two launches of two, one of one) bitwise five calls of one
    step; corner, edge and strip-boundary nodes against the oracle, within
    1e-5 of rho_l."""
    _, co = params_pair(nx, ny, tr=0.7)
    rho = wl.uniform_noise(nx, ny, 0.5 * (co.rho_g + co.rho_l), 0.01, seed=nx)
    lat = pkg.Lattice(nx, ny, tr=0.7).init(rho)
    for _ in range(5):
        lat.step(1)
    single = lat.state()
    lat.init(rho).step(5)
    got = lat.state()
    assert torch.equal(got, single)
    pts = [(0, 0), (nx - 1, ny - 1), (959, ny // 2), (960 % nx, ny // 3), (nx // 2, 1)]
    assert np.abs(device_samples(got, pts) - sampled_oracle(co, rho, pts, 5)).max() <= 1e-5 * co.rho_l
    lat.close()
