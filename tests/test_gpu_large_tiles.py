"""The kernels that only lattices past the caches run, on such lattices with
partial last tile columns and rows, compared node by node: the two-node tiles
of the one-step kernel (FP32 256 x 8, 2-byte 128 x 8) and the states stored
and loaded by streamed whole rows."""
import numpy as np
import pytest
import torch

import paper_1809_02390_amd as pkg
import workloads as wl
from oracle import lbm
from tests._gpu_helpers import oracle_init, params_pair

pytestmark = pytest.mark.gpu

NODE_BYTES = {"fp32": 36, "fp16": 20, "bf16": 20}  # of a state, with its reference density
# the gates of the step tests, of rho_l, for up to 100 steps
GATE = {"fp32": 1e-5, "fp16": 1e-4, "bf16": 1e-3}


# One-step kernel, source and destination above 256 MiB: 2763 = 10 tiles of 256
# and 203, or 21 of 128 and 75; 2510 = 313 rows of 8 and 6; rows off 64 bytes.
@pytest.mark.parametrize("storage", ["fp32", "fp16", "bf16"])
def test_two_node_tiles_match_repeated_lattice(storage):
    """307 x 251 repeated 9 x 10 times, one step at a time: after one and
    three steps every population (2-byte storages: and reference density)
    bitwise that of the small lattice, whose tiles hold one node per thread,
    and within the storage's gate of the oracle on every node."""
    nx, ny, cx, cy = 307, 251, 9, 10
    assert 2 * NODE_BYTES[storage] * nx * cx * ny * cy > 256 << 20
    _, co = params_pair(nx, ny, tr=0.7)
    rho = wl.droplets(nx, ny, co.rho_g, co.rho_l, co.width, [(120, 130)], [60.0])
    u = wl._f32(np.random.default_rng(5).uniform(-0.02, 0.02, (2, ny, nx)))
    rep = lambda a: torch.as_tensor(np.asarray(a), dtype=torch.float32, device="cuda").repeat(cy, cx)
    small = pkg.Lattice(nx, ny, tr=0.7, storage=storage).init(rho, *u)
    large = pkg.Lattice(cx * nx, cy * ny, tr=0.7, storage=storage).init(rep(rho), *map(rep, u))
    f = oracle_init(co, rho, *u)
    for steps in (1, 2):
        for _ in range(steps):
            small.step(1)
            large.step(1)
        f = lbm.run(f, co, steps)
        one = small.state()
        assert torch.equal(large.state(), one.repeat(1, cy, cx))
        if storage != "fp32":
            plane = lambda lat, w, h: lat.save_state()[-2 * w * h:].view(torch.int16).view(h, w)
            assert torch.equal(plane(large, cx * nx, cy * ny), plane(small, nx, ny).repeat(cy, cx))
        assert np.abs(one.double().cpu().numpy() - f).max() <= GATE[storage] * co.rho_l
    small.close()
    large.close()


# Streamed by whole rows: rows on 64 bytes and a state above 144 MiB.  2576 =
# 10 tiles of 256 and 16, 1701 = 212 rows of 8 and 5; 4128 = 64 tiles of 64
# and 32, 2117 = 132 rows of 16 and 5.
@pytest.mark.parametrize("nx,ny,storage", [(2576, 1701, "fp32"), (4128, 2117, "fp16"), (4128, 2117, "bf16")])
def test_streamed_initial_state(nx, ny, storage):
    """The state at rest, stored by tiles, is that of zero velocities, stored
    node by node, bit for bit, and within 1e-6 of rho_l (FP32: a dozen
    roundings of terms up to rho_l) or the storage's gate of the oracle on
    every node; a bad density is seen at the first and the last node."""
    es = 4 if storage == "fp32" else 2
    assert es * nx % 64 == 0 and 2 * 9 * es * nx * ny > 288 << 20
    _, co = params_pair(nx, ny, tr=0.7)
    host = wl.uniform_noise(nx, ny, 0.5 * (co.rho_g + co.rho_l), 0.01, seed=nx)
    rho = torch.as_tensor(host, dtype=torch.float32, device="cuda")
    zero = torch.zeros_like(rho)
    lat = pkg.Lattice(nx, ny, tr=0.7, storage=storage)
    used = 9 * es * nx * ny
    rest = lat.init(rho).save_state()
    err = np.abs(lat.state().double().cpu().numpy() - oracle_init(co, host)).max()
    assert err <= (1e-6 if storage == "fp32" else GATE[storage]) * co.rho_l
    moving = lat.init(rho, zero, zero).save_state()
    assert torch.equal(rest[:used], moving[:used])
    if storage != "fp32":
        assert torch.equal(rest[-2 * nx * ny:], moving[-2 * nx * ny:])
    for at in ((0, 0), (ny - 1, nx - 1)):
        bad = rho.clone()
        bad[at] = float("nan")
        with pytest.raises(pkg.LbmError):
            lat.init(bad)
    lat.close()


def test_streamed_load_is_exported_unchanged():
    """FP32 2576 x 1701: a loaded state comes back bit for bit."""
    f = torch.randn((9, 1701, 2576), generator=torch.Generator(device="cuda").manual_seed(3), device="cuda")
    lat = pkg.Lattice(2576, 1701, tr=0.7).set_state(f)
    assert torch.equal(lat.state(), f)
    lat.close()
