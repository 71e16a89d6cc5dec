"""Two contexts of the same parameters that use one workspace in turn: each
starts its runs from a density and its reverse sweeps from a seed, so nothing
the other left there may count.  Gradients bit for bit those of a context with
a workspace of its own."""
import ctypes

import pytest
import torch

from gpu_util import droplet_rho, make_sim, say
from oracle import eos
from paper_2504_03819_amd import inputs, lbfe

pytestmark = pytest.mark.gpu

OM = [1.0, 1.0, 1.0, 0.5] + [1.0] * 7
SHAPE = (9, 14, 19)


def sweep(sim, rho0, steps=3):
    sim.init_density(rho0)
    states = []
    for _ in range(steps):
        states.append(sim.get_state())
        sim.step(1)
    sim.adjoint_seed(sim.fields()["rho"])
    for st in reversed(states):
        sim.adjoint_step(st)
    g = sim.adjoint_init_density()
    return g, sim.adjoint_state(), sim.adjoint_grads()


@pytest.mark.parametrize("boundary", ["periodic", "walls", "mask"])
@pytest.mark.parametrize("precision", ["fp64", "fp32"])
def test_contexts_share_a_workspace(boundary, precision):
    nz, ny, nx = SHAPE
    T = eos.temperature(0.8)
    kw = dict(nx=nx, ny=ny, nz=nz, T=T, precision=precision, adjoint=1)
    if boundary != "periodic":
        kw.update(wet_mode=1, wet_value=1.2, omega=OM)
    if boundary == "walls":
        kw.update(walls_z=1)
    if boundary == "mask":
        kw.update(solid=torch.from_numpy(inputs.mask_planes(SHAPE)))
    say(f"shared workspace: {boundary} {precision}")
    walls = boundary != "periodic"
    rho_a = torch.tensor(droplet_rho(SHAPE, T, walls=walls, radius=4.0))
    rho_b = torch.tensor(droplet_rho(SHAPE, T, walls=walls, radius=5.0, seed=3))
    ga, la, pa = sweep(make_sim(**kw), rho_a)
    gb, lb, pb = sweep(make_sim(**kw), rho_b)

    a, b = make_sim(**kw), make_sim(**kw)
    base = (a.workspace.data_ptr() + 255) & ~255
    n = ctypes.c_size_t()
    assert lbfe.lib().lbfe_workspace_bytes(ctypes.byref(b.params), ctypes.byref(n)) == lbfe.OK
    assert lbfe.lib().lbfe_bind_workspace(b._ctx, ctypes.c_void_p(base), n) == lbfe.OK
    if boundary == "mask":
        b.set_solid(kw["solid"])
        a.set_solid(kw["solid"])
    for sim, rho, g, lam, p in ((b, rho_b, gb, lb, pb), (a, rho_a, ga, la, pa), (b, rho_b, gb, lb, pb)):
        h, mu, q = sweep(sim, rho)
        assert torch.equal(h, g) and torch.equal(mu, lam) and q == p
