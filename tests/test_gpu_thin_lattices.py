"""Several steps per launch on lattices thinner than the tile that runs them,
where a tile wraps around the lattice more than once."""
import pytest
import torch

import paper_1809_02390_amd as pkg
import workloads as wl
from tests._gpu_helpers import params_pair

pytestmark = pytest.mark.gpu


def _tiles(nx, ny, tx, ty):
    return -(-nx // tx) * -(-ny // ty)


# 5 x 1000, 1000 x 5: 500 tiles of 4 x 4, 125 of 8 x 8; 20 x 3000 and the
# others: 750 to 1500 tiles of 8 x 8, at most 512 of 32 x 8.
@pytest.mark.parametrize("storage", ["fp32", "fp16", "bf16"])
@pytest.mark.parametrize("nx,ny,tile", [(5, 1000, (8, 8)), (1000, 5, (8, 8)), (20, 3000, (32, 8)), (9, 4090, (32, 8)),
                                        (12000, 5, (32, 8)), (6000, 7, (32, 8))])
def test_thin_lattices_match_single_steps(nx, ny, tile, storage):
    """8 x 8 tiles (up to four steps) and 32 x 8 tiles (three) on lattices
    thinner than they are: 2, 3, 4 and 7 steps in a call bitwise as many
    calls of one step, the reference densities included."""
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    chosen = (4, 4) if _tiles(nx, ny, 4, 4) <= cus else (8, 8) if _tiles(nx, ny, 8, 8) <= 2 * cus else (32, 8)
    if chosen != tile or _tiles(nx, ny, *tile) > 2 * cus:
        pytest.skip(f"{cus} compute units choose another tile")
    _, co = params_pair(nx, ny, tr=0.7)
    rho = wl.uniform_noise(nx, ny, 0.5 * (co.rho_g + co.rho_l), 0.01, seed=nx + ny)
    lat, ref = (pkg.Lattice(nx, ny, tr=0.7, storage=storage).init(rho) for _ in range(2))
    for n in (2, 3, 4, 7):
        lat.step(n)
        for _ in range(n):
            ref.step(1)
        assert torch.equal(lat.state(), ref.state()), n
        if storage != "fp32":
            assert torch.equal(lat.save_state()[-2 * nx * ny:], ref.save_state()[-2 * nx * ny:]), n
    lat.close()
    ref.close()
