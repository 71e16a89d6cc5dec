"""The FP64 stencil marches of the solid-mask path at the edges of their tiles
(32 x 16 for mu; 32 x 12 and, from 2^20 nodes, 64 x 13 for F, phi and Q).

Narrow tiles: fields and populations of one step against the oracle on extents
one less, equal to and one more than a tile.  Wide tiles: a periodic state and
mask repeated to more than 2^20 nodes step as the repeated small box does, node
by node the same sums, so the populations must be equal bit for bit."""
import numpy as np
import pytest
import torch

from gpu_util import droplet_rho, gpu_fields, make_sim, oracle_fields, oracle_params, rel_err, say
from oracle import eos, lbm
from paper_2504_03819_amd import inputs

pytestmark = pytest.mark.gpu


def _box(shape, seed):
    T = eos.temperature(0.85)
    nz, ny, nx = shape
    mask = inputs.mask_obstacles(shape)
    sim = make_sim(nx=nx, ny=ny, nz=nz, T=T, solid=torch.tensor(mask), wet_mode=1, wet_value=1.3)
    g = np.random.Generator(np.random.PCG64(seed))
    rho0 = torch.tensor(droplet_rho(shape, T, radius=max(2.0, min(shape) / 3)))
    u0 = torch.tensor(0.02 * g.uniform(-1, 1, (3,) + shape))
    return sim, torch.tensor(mask), rho0, u0


@pytest.mark.parametrize("shape", [(8, 11, 31), (9, 12, 32), (8, 13, 33), (10, 16, 32), (8, 17, 65), (19, 25, 30)], ids=str)
def test_tile_edges_match_the_oracle(shape):
    say(f"mask tiles {shape}")
    sim, mask, rho0, u0 = _box(shape, 3)
    p = oracle_params(sim)
    f = lbm.init(rho0, p, u0)
    f = f + torch.tensor(inputs.uniform_noise(tuple(f.shape), 2e-4, 3)) * (f != 0)
    sim.set_populations(f)
    fg, fo = gpu_fields(sim), oracle_fields(f, p)
    for k in ("rho", "mu", "F", "u", "Q"):
        assert rel_err(fg[k], fo[k]) < 1e-11, k
    sim.step(1)
    assert rel_err(sim.populations().cpu(), lbm.step(f, p)) < 1e-11


def test_repeated_state_steps_like_the_small_box():
    shape, reps = (13, 27, 66), (4, 7, 2)
    sim, mask, rho0, u0 = _box(shape, 5)
    sim.init_density(rho0, u0)
    sim.step(4)
    nz, ny, nx = (a * b for a, b in zip(shape, reps))
    big = make_sim(nx=nx, ny=ny, nz=nz, T=eos.temperature(0.85), solid=mask.repeat(reps), wet_mode=1, wet_value=1.3)
    big.init_density(rho0.repeat(reps), u0.repeat((1,) + reps))
    big.step(4)
    assert torch.equal(sim.populations().repeat((1,) + reps), big.populations())
    assert torch.equal(sim.field(4).repeat((1,) + reps), big.field(4))  # Q
