"""The schedules that lbfe_create chooses."""
import ctypes

import pytest
import torch

from gpu_util import droplet_rho, make_sim, say
from oracle import eos
from paper_2504_03819_amd import lbfe

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape", [(96, 96, 96), (100, 70, 130)])
def test_reported_parameters_give_the_same_schedule(shape):
    """One launch for chain and collision, and a march where the chain runs
    alone, whose length lbfe_get_params reports.  Inside the collide kernel the
    chain's interval holds no launch: a small part of the moments pass, on
    grids whose moments pass is long against the events themselves."""
    nz, ny, nx = shape
    T = eos.temperature(0.8)
    a = make_sim(nx=nx, ny=ny, nz=nz, T=T)
    b = make_sim(params=a.params)
    rho0 = torch.tensor(droplet_rho(shape, T))
    part = []
    for s in (a, b):
        s.init_density(rho0)
        s.step(10)
        t = min((s.step_timed(20) for _ in range(5)), key=lambda v: v["chain"])
        part.append(t["chain"] / t["moments"])
    say(f"chain / moments {shape}: {part[0]:.3f} chosen, {part[1]:.3f} from the reported parameters")
    assert bytes(a.params) == bytes(b.params)
    assert torch.equal(a.get_state(), b.get_state())
    assert max(part) < 0.5


OM = [1.0, 1.0, 1.0, 0.5] + [1.0] * 7


@pytest.mark.parametrize("wall_u", [(0.0, 0.0, 0.0, 0.0), (0.02, 0.0, -0.01, 0.01)])
@pytest.mark.parametrize("shape,precision,adjoint", [
    ((90, 88, 90), "fp64", 0),              # one launch, non-temporal population loads
    ((26, 150, 145), "fp32", 1),            # the same (a reverse context counts its lattices twice)
    ((3, 701, 700), "fp32", 0),             # two launches: one plane beside both walls
    ((3, 300, 201), "fp32", 0),             # one
    ((5, 400, 400), "fp64", 0),             # two: mostly blocks beside a wall
    ((4, 350, 701), "fp16dev_f0fp32", 0)])  # chunks of the grid's two planes
def test_walled_routes_equal_the_march(shape, precision, adjoint, wall_u):
    nz, ny, nx = shape
    T = eos.temperature(0.8)
    say(f"walled route: {shape} {precision} {wall_u}")
    rho0 = torch.tensor(droplet_rho(shape, T, walls=True, radius=8.0))
    out = []
    for chunk in (0, 64):
        sim = make_sim(nx=nx, ny=ny, nz=nz, T=T, walls_z=1, wet_mode=1, wet_value=1.2, omega=OM, precision=precision,
                       wall_u=wall_u, chain_chunk=chunk, adjoint=adjoint)
        sim.init_density(rho0)
        sim.step(3)
        out.append((sim.get_state(), sim.field(2)))
    assert torch.equal(out[0][0], out[1][0]) and torch.equal(out[0][1], out[1][1])


@pytest.mark.parametrize("shape,precision", [((1, 300, 700), "fp64"), ((2, 301, 701), "fp32"), ((5, 512, 512), "fp64")])
def test_thin_periodic_routes_equal_the_march(shape, precision):
    nz, ny, nx = shape
    T = eos.temperature(0.8)
    say(f"thin route: {shape} {precision}")
    rho0 = torch.tensor(droplet_rho(shape, T, radius=8.0))
    out = []
    for chunk in (0, 64):
        sim = make_sim(nx=nx, ny=ny, nz=nz, T=T, precision=precision, chain_chunk=chunk)
        sim.init_density(rho0)
        sim.step(3)
        out.append((sim.get_state(), sim.field(2)))
    assert torch.equal(out[0][0], out[1][0]) and torch.equal(out[0][1], out[1][1])


@pytest.mark.parametrize("nx,ny,nz,precision,path", [
    (256, 256, 256, "fp64", 2), (160, 150, 245, "fp64", 2), (200, 90, 327, "fp64", 2), (80, 226, 762, "fp64", 2),
    (50, 95, 1300, "fp64", 2),
    (70, 300, 280, "fp64", 2), (33, 200, 890, "fp64", 2),                          # part lines, large planes
    (300, 14, 1399, "fp64", 1), (40, 40, 3671, "fp64", 1), (65, 65, 1390, "fp64", 1), (96, 27, 2266, "fp64", 1),
    (512, 512, 512, "fp32", 2), (320, 320, 320, "fp32", 2), (301, 205, 330, "fp32", 2), (97, 708, 442, "fp32", 2),
    (65, 65, 4964, "fp32", 1), (40, 40, 13108, "fp32", 1), (32, 544, 1982, "fp32", 1), (160, 150, 874, "fp32", 1),
    (160, 160, 160, "fp64", 1), (256, 256, 256, "fp32", 1), (512, 512, 512, "fp16dev_f0fp32", 1)])
def test_step_path_of_large_grids(nx, ny, nz, precision, path):
    """The path chosen: fused where the columns fill its tiles, or where their
    rows are no whole lines and their planes exceed an XCD's L2."""
    p = lbfe.default_params(nx=nx, ny=ny, nz=nz, precision=precision)
    ctx, q = ctypes.c_void_p(), lbfe.Params()
    assert lbfe.lib().lbfe_create(ctypes.byref(p), None, ctypes.byref(ctx)) == lbfe.OK
    assert lbfe.lib().lbfe_get_params(ctx, ctypes.byref(q)) == lbfe.OK
    lbfe.lib().lbfe_destroy(ctx)
    assert q.step_path == path


@pytest.mark.parametrize("wall_u", [(0.0, 0.0, 0.0, 0.0), (0.02, 0.0, -0.01, 0.01)])
@pytest.mark.parametrize("shape,precision", [((3, 14, 33), "fp64"), ((4, 9, 65), "fp32"), ((11, 27, 40), "fp64"),
                                             ((9, 10, 64), "fp16dev_f0fp32")])
def test_fused_step_with_the_march_between_walls(shape, precision, wall_u):
    """On large grids the march, not the fused step, leaves the solid planes'
    density: until the chain runs they hold what the step kept there.  State,
    every field and the reductions against the two-pass block form."""
    nz, ny, nx = shape
    T = eos.temperature(0.8)
    say(f"fused step and march: {shape} {precision} {wall_u}")
    rho0 = torch.tensor(droplet_rho(shape, T, walls=True, radius=4.0))
    kw = dict(nx=nx, ny=ny, nz=nz, T=T, walls_z=1, wet_mode=1, wet_value=1.2, omega=OM, precision=precision, wall_u=wall_u)
    ref = make_sim(step_path=lbfe.PATH_TWO_PASS, **kw)
    sims = [make_sim(step_path=lbfe.PATH_FUSED, chain_chunk=c, **kw) for c in (3, 64)]
    for s in (ref, *sims):
        s.init_density(rho0)
    for n in (1, 2):
        ref.step(n)
        for s in sims:
            s.step(n)
            red = s.reduce()  # the first reader after a step
            assert red == ref.reduce()
            for which in range(6):
                assert torch.equal(s.field(which), ref.field(which)), (n, which)
            assert torch.equal(s.get_state(), ref.get_state())


@pytest.mark.parametrize("value", [float("nan"), float("inf")])
@pytest.mark.parametrize("precision", ["fp64", "fp32"])
def test_bad_density_stays_on_its_side_of_the_walls(precision, value):
    """A NaN or an infinity beside the top wall: the step reports it, every
    route spreads it alike, and nothing crosses to the bottom wall through the
    periodic wrap of the planes."""
    shape = nz, ny, nx = (14, 18, 70)
    T = eos.temperature(0.8)
    rho0 = torch.tensor(droplet_rho(shape, T, walls=True, radius=4.0))
    out = []
    for chunk in (0, 64, 3):
        sim = make_sim(nx=nx, ny=ny, nz=nz, T=T, walls_z=1, wet_mode=1, wet_value=1.2, omega=OM, precision=precision,
                       chain_chunk=chunk, step_path=lbfe.PATH_TWO_PASS)
        sim.init_density(rho0)
        f = sim.populations()
        f[5, nz - 2, 9, 33] = value
        sim.set_populations(f)
        with pytest.raises(lbfe.LBFEError) as e:
            sim.step(1)
        assert e.value.code == lbfe.E_DIVERGED
        out.append(sim.populations())
    for g in out[1:]:
        assert torch.equal(torch.isfinite(g), torch.isfinite(out[0]))
    assert bool(torch.isfinite(out[0][:, :7]).all()) and not bool(torch.isfinite(out[0]).all())
