"""The block form of the stencil chain (grids below 2^19 fluid nodes), alone and
with the collision in the same launch, against the marching forms (periodic,
between walls), bit for bit: all sum every stencil in the same order, so the
states after a few steps and the fields must be equal.  The sizes sit at the edges of the 16 x 8 blocks, the 64 x 16 tiles
and their halos: one node, extents below the halo, one more and one less than
a block or tile, one and two fluid planes between walls, chunks of one plane
and longer than the grid, a ragged last block in every direction."""
import numpy as np
import pytest
import torch

from gpu_util import droplet_rho, make_sim, say
from oracle import eos

pytestmark = pytest.mark.gpu

OM = [1.0, 1.0, 1.0, 0.5] + [1.0] * 7
MARCH = (64, 3, 5)  # chunk lengths that only the marching forms have
SHAPES = [(1, 1, 1), (2, 3, 1), (5, 2, 3), (4, 8, 16), (5, 9, 17), (9, 7, 15), (3, 17, 33), (6, 40, 31),
          (7, 16, 64), (4, 17, 65), (11, 15, 63), (8, 33, 130)]


@pytest.mark.parametrize("walls", [False, True])
@pytest.mark.parametrize("precision", ["fp64", "fp32", "fp16dev_f0fp32"])
def test_block_chain_equals_the_march(walls, precision):
    T = eos.temperature(0.8)
    for shape in SHAPES:
        nz, ny, nx = shape
        if walls:
            nz += 2
        say(f"chain block: {(nz, ny, nx)} walls={walls} {precision}")
        kw = dict(nx=nx, ny=ny, nz=nz, T=T, walls_z=int(walls), precision=precision, step_path=1)
        if walls:
            kw.update(wet_mode=1, wet_value=1.3, omega=OM)
        rho0 = torch.tensor(droplet_rho((nz, ny, nx), T, walls=walls, radius=max(2.0, min(ny, nx) / 3.0)))
        g = np.random.Generator(np.random.PCG64(4))
        u0 = torch.tensor(0.02 * g.uniform(-1, 1, (3, nz, ny, nx)))
        sims = [make_sim(chain_chunk=c, **kw) for c in (*MARCH, 0, 1, 2, 4)]
        for s in sims:
            s.init_density(rho0, u0)
            s.step(3)
        ref, fr = sims[0].get_state(), sims[0].fields()
        for s in sims[1:]:
            assert torch.equal(s.get_state(), ref), (shape, s.params.chain_chunk)
            f = s.fields()
            for name in ("rho", "u", "mu", "F"):
                assert torch.equal(f[name], fr[name]), (shape, s.params.chain_chunk, name)


@pytest.mark.parametrize("precision", ["fp64", "fp32", "fp16dev", "fp16dev_f0fp32"])
@pytest.mark.parametrize("shape", [(3, 9, 17), (4, 8, 16), (6, 17, 33), (11, 7, 65)])
def test_block_step_between_moving_walls(shape, precision):
    """The moving-wall term reads the mu that the block kernel leaves beside
    the walls; nz = 3 and 4 put both walls in one block."""
    nz, ny, nx = shape
    T = eos.temperature(0.8)
    say(f"block step, moving walls: {shape} {precision}")
    rho0 = torch.tensor(droplet_rho(shape, T, walls=True, radius=3.0))
    out = []
    for chunk in (64, 3, 0, 1, 2, 4):
        s = make_sim(nx=nx, ny=ny, nz=nz, T=T, walls_z=1, wet_mode=1, wet_value=0.7, omega=OM, precision=precision,
                     step_path=1, chain_chunk=chunk, wall_u=(-0.01, 0.004, 0.02, 0.0))
        s.init_density(rho0)
        s.step(4)
        out.append(s.get_state())
    for st in out[1:]:
        assert torch.equal(st, out[0])


@pytest.mark.parametrize("precision", ["fp64", "fp32", "fp16dev_f0fp32"])
def test_large_periodic_grid_steps_like_its_small_copy(precision):
    """From 6 (FP64) or 12 (narrow forms) x 2^20 nodes a periodic chain forms
    mu0(rho) itself: a state repeated to 17.8e6 nodes must step as the small
    box does (stored mu0), node by node the same bits."""
    shape, reps = (13, 27, 66), (6, 8, 16)
    T = eos.temperature(0.85)
    rho0 = torch.tensor(droplet_rho(shape, T, radius=4.0), device="cuda:0")
    g = np.random.Generator(np.random.PCG64(6))
    u0 = torch.tensor(0.02 * g.uniform(-1, 1, (3,) + shape), device="cuda:0")
    out = []
    for r in ((1, 1, 1), reps):
        nz, ny, nx = (a * b for a, b in zip(shape, r))
        sim = make_sim(nx=nx, ny=ny, nz=nz, T=T, precision=precision)
        sim.init_density(rho0.repeat(r), u0.repeat((1,) + r))
        sim.step(4)
        mu = sim.field(2)
        out.append((sim.populations(), mu))
        sim.close()
    (fs, ms), (fb, mb) = out
    assert torch.equal(ms.repeat(reps), mb)
    for i in range(27):
        assert torch.equal(fs[i].repeat(reps), fb[i]), i
