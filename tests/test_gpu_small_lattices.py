"""Several time steps per launch on small lattices: bitwise the same steps
taken one call at a time (the one-step kernel), for every tile, storage and
number of steps of a launch, on lattices at the edges of the tiles and down
to one node; the chain of stored states; buffers that alternate."""
import pytest
import torch

import paper_1809_02390_amd as pkg
import workloads as wl
from paper_1809_02390_amd import lbm as L
from tests._gpu_helpers import params_pair

pytestmark = pytest.mark.gpu

# 4 x 4 tiles (up to four steps per launch; also 5 x 500), 8 x 8 (four; also
# 7 x 3000), 32 x 8 (three), 16 x 16 (two; 559 x 583 in FP32: 64 x 24): whole
# tiles, remainders, lattices thinner than the rings
TINY = [(64, 64), (1, 1), (3, 2), (64, 1), (5, 200), (37, 29)]
SMALL = [(128, 128), (131, 77), (5, 500), (250, 65)]
WIDE = [(256, 256), (301, 203), (16384, 1), (7, 3000)]
LAST = [(432, 416), (559, 583), (3, 20000)]


def _init(nx, ny, storage):
    _, co = params_pair(nx, ny, tr=0.7)
    rho = wl.uniform_noise(nx, ny, 0.5 * (co.rho_g + co.rho_l), 0.01, seed=nx + ny)
    return pkg.Lattice(nx, ny, tr=0.7, storage=storage).init(rho)


@pytest.mark.parametrize("storage", ["fp32", "fp16", "bf16"])
@pytest.mark.parametrize("nx,ny", TINY + SMALL + WIDE + LAST)
def test_fused_steps_match_single_steps(nx, ny, storage):
    lat, ref = _init(nx, ny, storage), _init(nx, ny, storage)
    for n in (2, 3, 4, 5, 7):
        lat.step(n)
        for _ in range(n):
            ref.step(1)
        assert torch.equal(lat.state(), ref.state()), n
        if storage != "fp32":  # the reference densities the next step decodes with
            assert torch.equal(lat.save_state()[-2 * nx * ny:], ref.save_state()[-2 * nx * ny:]), n
    lat.close()
    ref.close()


@pytest.mark.parametrize("nx,ny", [(64, 64), (131, 77), (301, 203), (432, 416)])
@pytest.mark.parametrize("cycle", [2, 3, 9])
def test_chain_matches_single_steps(nx, ny, cycle):
    """step_saved_chain over 8 steps with `cycle` buffers in turn (9: all
    distinct): the buffers hold the last states written to them."""
    lat, ref = _init(nx, ny, "fp32"), _init(nx, ny, "fp32")
    n = 8
    bufs = [lat.checkpoint_buffer().zero_() for _ in range(cycle)]
    lat.save_state(bufs[0])
    lat.step_saved_chain([bufs[j % cycle] for j in range(n + 1)])
    used = 9 * nx * ny * 4
    for j in range(n + 1):
        if j > n - cycle:
            assert torch.equal(bufs[j % cycle][:used], ref.save_state()[:used]), j
        ref.step(1)
    lat.close()
    ref.close()


@pytest.mark.parametrize("nx,ny,storage", [(60, 50, "fp32"), (120, 130, "bf16"), (300, 200, "fp32"), (430, 410, "fp16")])
@pytest.mark.parametrize("n", [4, 8, 12])
def test_captured_multiples_of_four(nx, ny, storage, n):
    """A captured lbm_step(n) with n a multiple of 4 ends on the buffer it
    started from for every number of steps per launch: three replays, with
    eager work between them, each bitwise n more eager steps."""
    s = torch.cuda.Stream()
    _, co = params_pair(nx, ny, tr=0.7)
    rho = wl.uniform_noise(nx, ny, 0.5 * (co.rho_g + co.rho_l), 0.01, seed=n)
    lat = pkg.Lattice(nx, ny, stream=s, tr=0.7, storage=storage).init(rho)
    ref = pkg.Lattice(nx, ny, tr=0.7, storage=storage).init(rho)
    g = torch.cuda.CUDAGraph()
    torch.cuda.synchronize()
    with torch.cuda.graph(g, stream=s):
        L.lbm_step(lat.ctx, n)
    torch.cuda.synchronize()
    for k in range(3):
        g.replay()
        ref.step(n)
        torch.cuda.synchronize()
        assert torch.equal(lat.state(), ref.state()), k
    del g
    lat.close()
    ref.close()
