"""lbm_step and lbm_moments_noalloc captured in a HIP graph (torch's
CUDAGraph on the context's stream) and replayed: every replay bitwise equal
to the same calls made eagerly, with eager work of the program and
synchronisations between replays.  A graph records the state buffers of the
captured launches, so the captured lbm_step(n) takes a multiple of 4 steps:
it then ends on the buffer it started from, whatever number of steps the
lattice takes per launch."""
import numpy as np
import pytest
import torch

import paper_1809_02390_amd as pkg
import workloads as wl
from paper_1809_02390_amd import lbm as L
from tests._gpu_helpers import params_pair

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nx,ny,storage,n", [(1024, 384, "fp32", 4), (256, 256, "fp32", 8), (400, 200, "fp16", 4),
                                             (1000, 700, "fp32", 12)])
def test_graph_replays_match_eager_calls(nx, ny, storage, n):
    """1024 x 384 and 1000 x 700 run two steps per launch (two and six
    launches per replay), 256 x 256 and the FP16 lattice up to three.
    Three replays, each checked against an eager lattice advanced by the
    same n steps: the state and the moments (fields and FP64 totals)."""
    _, co = params_pair(nx, ny, tr=0.7)
    rho0 = wl.droplets(nx, ny, co.rho_g, co.rho_l, co.width, [(nx * 0.4, ny * 0.5)], [min(nx, ny) * 0.3])
    rng = np.random.default_rng(nx + n)
    ux0, uy0 = (wl._f32(rng.uniform(-0.02, 0.02, (ny, nx))) for _ in range(2))
    s = torch.cuda.Stream()
    lat = pkg.Lattice(nx, ny, stream=s, tr=0.7, storage=storage).init(rho0, ux0, uy0)
    ref = pkg.Lattice(nx, ny, tr=0.7, storage=storage).init(rho0, ux0, uy0)
    rho, ux, uy = (torch.empty((ny, nx), dtype=torch.float32, device="cuda") for _ in range(3))
    tot = torch.empty(3, dtype=torch.float64, device="cuda")
    g = torch.cuda.CUDAGraph()
    torch.cuda.synchronize()
    with torch.cuda.graph(g, stream=s):
        L.lbm_step(lat.ctx, n)
        L.lbm_moments_noalloc(lat.ctx, rho, ux, uy, tot, n=lat.n)
    torch.cuda.synchronize()
    for k in range(3):
        g.replay()
        ref.step(n)  # eager work between the replays
        r_ref, u_ref, v_ref, tot_ref = ref.moments()
        torch.cuda.synchronize()
        assert torch.equal(lat.state(), ref.state()), k
        assert torch.equal(rho, r_ref) and torch.equal(ux, u_ref) and torch.equal(uy, v_ref), k
        assert tuple(tot.cpu().tolist()) == tuple(tot_ref), k
    del g
    lat.close()
    ref.close()
