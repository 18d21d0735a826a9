"""Calls that choose between kernels or store policies, timed against another
call of the same lattice that bounds their cost: a choice that loses to the
simpler one shows as a ratio.  Each limit lies between the ratio of the better
choice and that of the worse one (both given with the case); a ratio has to
exceed it in three measurements to fail."""
import numpy as np
import pytest
import torch

import paper_1809_02390_amd as pkg
import workloads as wl
from paper_1809_02390_amd import lbm as L
from tests._gpu_helpers import params_pair

pytestmark = pytest.mark.gpu


def _lat(nx, ny, storage="fp32"):
    _, co = params_pair(nx, ny, tr=0.7)
    rho = torch.as_tensor(wl.uniform_noise(nx, ny, 0.5 * (co.rho_g + co.rho_l), 0.01, seed=nx), dtype=torch.float32,
                          device="cuda")
    return rho, pkg.Lattice(nx, ny, tr=0.7, storage=storage).init(rho)


def _cost(call, repeat):
    """Device time of one of `repeat` calls in a row (ms)."""
    a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    a.record()
    for _ in range(repeat):
        call()
    b.record()
    b.synchronize()
    return a.elapsed_time(b) / repeat


def _ratio(call, bound, repeat):
    """Median cost of call over that of bound, nine measurements in turn."""
    call(), bound()
    t = np.array([[_cost(call, repeat), _cost(bound, repeat)] for _ in range(9)])
    return float(np.median(t[:, 0]) / np.median(t[:, 1]))


def _assert_ratio(call, bound, limit, repeat=20):
    got = [_ratio(call, bound, repeat)]
    while got[-1] > limit and len(got) < 3:
        got.append(_ratio(call, bound, repeat))
    assert got[-1] <= limit, got


def test_short_rows_are_not_stored_in_parts():
    """3 x 100000 (rows of 12 bytes): loading a state and seeding an adjoint
    against exporting a state, which moves the same 72 bytes per node; cached
    1.5 and 1.7 times its cost, the adjoint streamed 5.3."""
    nx, ny = 3, 100000
    _, lat = _lat(nx, ny)
    f = lat.state()
    adj, out = lat.adjoint_buffer(), torch.empty_like(f)
    get = lambda: L.lbm_get_state(lat.ctx, out, lat.n)
    nb = L.lbm_adjoint_bytes(lat.params)
    _assert_ratio(lambda: L.lbm_set_state(lat.ctx, f, lat.n), get, 2.3)
    _assert_ratio(lambda: L.lbm_adjoint_seed(lat.ctx, f, adj, lat.n, nb), get, 2.8)
    lat.close()


def test_shifted_rows_are_merged_in_the_caches():
    """3600^2: an initial state with velocities (48 bytes per node) against
    loading a state (72); cached 0.82 of its cost, streamed 1.16."""
    n = 3600
    rho, lat = _lat(n, n)
    u = torch.full_like(rho, 0.01)
    f = lat.state()
    _assert_ratio(lambda: L.lbm_init(lat.ctx, rho, u, u, lat.n), lambda: L.lbm_set_state(lat.ctx, f, lat.n), 1.05, 5)
    lat.close()


# FP32: below and above 256 MiB of populations and state, from where the loads
# are shifted instead of the stores; below and above the size from which
# states are streamed (row length a multiple of 64 bytes and a state above 144
# MiB), and rows off 64 bytes.
@pytest.mark.parametrize("nx,ny", [(3, 1000), (560, 600), (1863, 2001), (1864, 2001), (2064, 2031), (2064, 2040),
                                   (2101, 2048)])
def test_loaded_states_agree(nx, ny):
    """A loaded state is exported unchanged, and a state at zero velocity
    given as populations equals the initial one, bit for bit."""
    rho, lat = _lat(nx, ny)
    zero = torch.zeros_like(rho)
    used = 36 * nx * ny
    first = lat.init(rho, zero, zero).save_state()[:used]
    f = lat.state()
    assert torch.equal(lat.set_state(f).save_state()[:used], first)
    assert torch.equal(lat.state(), f)
    lat.close()


def _single(lat, n):
    for _ in range(n):
        L.lbm_step(lat.ctx, 1)


# 600 x 600: 250 tiles of 64 x 24; 1000 x 350: 240.
@pytest.mark.parametrize("nx,ny", [(600, 600), (1000, 350)])
def test_several_steps_cost_no_more_than_single_steps_fp32(nx, ny):
    """lbm_step(20) against 20 calls of one step: 0.9 of their cost with one
    64 x 24 two-step tile per CU, 1.1 on 16 x 16 tiles."""
    _, lat = _lat(nx, ny)
    _assert_ratio(lambda: L.lbm_step(lat.ctx, 20), lambda: _single(lat, 20), 1.0, 5)
    lat.close()


# 16 x 16 tiles that hold more rows past the lattice than 64 x 8 tiles do.
@pytest.mark.parametrize("nx,ny,storage", [(20000, 4, "fp16"), (10000, 24, "bf16")])
def test_several_steps_cost_no_more_than_single_steps_2_byte(nx, ny, storage):
    """lbm_step(20) against 20 calls of one step: the same kernel, 1.26 and
    1.31 of their cost on 16 x 16 tiles."""
    _, lat = _lat(nx, ny, storage)
    _assert_ratio(lambda: L.lbm_step(lat.ctx, 20), lambda: _single(lat, 20), 1.12, 5)
    lat.close()


def test_flat_lattices_share_halo_lines():
    """50000 x 6, two rows of 781 tiles: a step against the export of the
    state, which moves the same 72 bytes per node: 1.5 times its cost in
    strips of 32 tiles, 2.2 in longer ones."""
    _, lat = _lat(50000, 6)
    out = lat.state()
    _assert_ratio(lambda: L.lbm_step(lat.ctx, 1), lambda: L.lbm_get_state(lat.ctx, out, lat.n), 1.85)
    lat.close()


# Strips of 32 tiles of 64 nodes and a narrower last one, or a single tile
# column beyond them; 2-byte lattices below and from eight rows of tiles on.
@pytest.mark.parametrize("nx,ny,storage", [(2112, 9, "fp32"), (50000, 6, "fp32"), (2100, 30, "fp16"), (4100, 56, "bf16"),
                                           (4100, 57, "bf16")])
def test_strips_of_one_step_agree(nx, ny, storage):
    """One step of a flat lattice, which visits its tiles in strips, bitwise
    the repeated step of the lattice it repeats in y, visited in others."""
    rho, lat = _lat(nx, ny, storage)
    one = lat.step(1).state()
    lat.close()
    with_copies = pkg.Lattice(nx, 8 * ny, tr=0.7, storage=storage).init(rho.repeat(8, 1))
    many = with_copies.step(1).state()
    assert torch.equal(many, one.repeat(1, 8, 1))
    with_copies.close()


def _adjoint(nx, ny, copies=1):
    """Forward state and adjoint of a lattice and its copies in y, seeded
    alike; the lattice sized nx x (copies ny)."""
    _, co = params_pair(nx, ny, tr=0.7)
    gen = torch.Generator(device="cuda").manual_seed(nx)
    rho = 0.5 * (co.rho_g + co.rho_l) + 0.02 * (torch.rand((ny, nx), generator=gen, device="cuda") - 0.5)
    lam = torch.randn((9, ny, nx), generator=gen, device="cuda")
    lat = pkg.Lattice(nx, copies * ny, tr=0.7).init(rho.repeat(copies, 1))
    return lat, lat.save_state(), lat.adjoint_seed(lam.repeat(1, copies, 1)), lat.adjoint_buffer()


def test_narrow_adjoints_cost_less_than_wider_ones():
    """An adjoint step on 8 x 20000 against 33 x 20000, two tile columns of 32:
    0.6 of its cost on 32 x 8 tiles, 1.1 on 64 x 8."""
    call = []
    for nx in (8, 33):
        lat, f, a, b = _adjoint(nx, 20000)
        sb, ab = L.lbm_checkpoint_bytes(lat.params), L.lbm_adjoint_bytes(lat.params)
        call.append(lambda lat=lat, f=f, a=a, b=b, sb=sb, ab=ab: L.lbm_adjoint_step(lat.ctx, f, a, b, sb, ab))
    _assert_ratio(*call, 0.85)


# 775 tiles of 32 x 8 in one column, lattices 32 and 33 wide on either side of
# it; and a state above 4 GiB, read relative to each tile's row band and, in
# the tile rows that wrap, with 64-bit addresses.
@pytest.mark.parametrize("nx,ny,copies", [(1, 200, 31), (3, 200, 31), (32, 200, 31), (33, 200, 31), (32, 1900, 2000)])
def test_narrow_adjoints_agree(nx, ny, copies):
    """One adjoint step of copies in y, more than three small tiles per CU,
    bitwise the repeated step of one copy; the parameter sums in proportion,
    to 1e-6 (FP32 sums of two terms, paired alike, then FP64)."""
    lat, f, a, b = _adjoint(nx, ny)
    lat.adjoint_step(f, a, b)
    one, theta = lat.adjoint_get(b), np.array(lat.adjoint_theta())
    lat.close()
    lat, f, a, b = _adjoint(nx, ny, copies)
    lat.adjoint_step(f, a, b)
    assert torch.equal(lat.adjoint_get(b), one.repeat(1, copies, 1))
    assert np.abs(np.array(lat.adjoint_theta()) / copies - theta).max() <= 1e-6 * np.abs(theta).max()
    lat.close()


# Two steps per launch on either side of the lines between 16 x 16, 64 x 16 and
# 64 x 24 tiles (256 CUs): 2.8 and 3.1 tiles of 16 x 16 per CU; one 64 x 16
# tile and more; one 64 x 24 tile and more; two 64 x 16 tiles and more.
@pytest.mark.parametrize("nx,ny", [(432, 432), (448, 448), (512, 512), (520, 520), (600, 600), (608, 608), (6000, 24),
                                   (100, 3000), (200, 1800), (700, 700), (712, 712), (576, 576), (4064, 89)])
def test_two_step_tiles_agree(nx, ny):
    """Three steps in one call, and as a chain of stored states, bitwise three
    calls of one step."""
    _, lat = _lat(nx, ny)
    used = 36 * nx * ny
    bufs = [lat.checkpoint_buffer().zero_() for _ in range(4)]
    lat.save_state(bufs[0])
    lat.step_saved_chain(bufs)
    once = lat.step(3).save_state()[:used].clone()
    lat.load_state(bufs[0])
    for j in range(1, 4):
        assert torch.equal(lat.step(1).save_state()[:used], bufs[j][:used])
    assert torch.equal(bufs[3][:used], once)
    lat.close()


# 2-byte lattices on either side of the line between 16 x 16 tiles and single
# steps: 2.2 and 2.4 tiles per 64 x 8 tile, below and above three per CU.
@pytest.mark.parametrize("storage", ["fp16", "bf16"])
@pytest.mark.parametrize("nx,ny", [(2000, 72), (4000, 40), (4800, 40), (20000, 4), (16000, 9)])
def test_flat_2_byte_steps_agree(nx, ny, storage):
    """Five steps in one call bitwise five calls of one step, the reference
    densities included."""
    rho, lat = _lat(nx, ny, storage)
    once = lat.step(5).state()
    ref = lat.save_state()[-2 * nx * ny:]
    lat.init(rho)
    _single(lat, 5)
    assert torch.equal(lat.state(), once) and torch.equal(lat.save_state()[-2 * nx * ny:], ref)
    lat.close()


# 2-byte single steps on 64 x 4 and 64 x 8 tiles: last tile columns of 8, 9 and
# 64 nodes; 128 tiles of 64 x 8 and 132.
@pytest.mark.parametrize("storage", ["fp16", "bf16"])
@pytest.mark.parametrize("nx,ny", [(72, 72), (73, 71), (64, 65), (256, 256), (256, 260), (9, 3)])
def test_small_2_byte_steps_agree(nx, ny, storage):
    """Four steps, one call at a time, bitwise the four steps of one launch."""
    rho, lat = _lat(nx, ny, storage)
    once = lat.step(4).state()
    ref = lat.save_state()[-2 * nx * ny:]
    lat.init(rho)
    _single(lat, 4)
    assert torch.equal(lat.state(), once) and torch.equal(lat.save_state()[-2 * nx * ny:], ref)
    lat.close()


# 2-byte exports below and above 256 MiB of populations.
@pytest.mark.parametrize("storage", ["fp16", "bf16"])
@pytest.mark.parametrize("nx,ny", [(2736, 2725), (2736, 2727)])
def test_exports_agree(nx, ny, storage):
    """The exported state of a lattice that repeats a smaller one is the
    repeated export."""
    k = {2725: 25, 2727: 27}[ny]
    rho, one = _lat(48, k, storage)
    f = one.step(1).state()
    one.close()
    many = pkg.Lattice(nx, ny, tr=0.7, storage=storage).init(rho.repeat(ny // k, nx // 48))
    assert torch.equal(many.step(1).state(), f.repeat(1, ny // k, nx // 48))
    many.close()
