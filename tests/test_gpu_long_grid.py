"""A periodic column so long that four-plane blocks would need more workgroups
than a launch's y dimension holds (65535): the same bits as the 64-plane
march."""
import pytest
import torch

from gpu_util import make_sim
from oracle import eos
from paper_2504_03819_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("walls", [False, True])
@pytest.mark.parametrize("precision", ["fp64", "fp32"])
def test_long_column(walls, precision):
    nz = 4 * 65535 + 8
    T = eos.temperature(0.9)
    rl, rv = eos.maxwell(eos.PAPER["a"], eos.PAPER["b"], eos.PAPER["R"], T)
    rho0 = torch.full((nz, 1, 1), rv, dtype=torch.float64)
    rho0[nz // 4:3 * nz // 4] = rl
    rho0 += torch.tensor(inputs.uniform_noise((nz, 1, 1), 1e-3, 2))
    out = []
    for chunk in (64, 0):
        sim = make_sim(nx=1, ny=1, nz=nz, T=T, precision=precision, walls_z=int(walls), chain_chunk=chunk)
        sim.init_density(rho0)
        sim.step(2)
        out.append((sim.get_state(), sim.field(2), sim.reduce()))
    assert torch.equal(out[0][0], out[1][0]) and torch.equal(out[0][1], out[1][1]) and out[0][2] == out[1][2]
