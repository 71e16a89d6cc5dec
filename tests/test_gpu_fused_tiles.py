"""The fused step kernel at the edges of its tiles (32 x 13 columns in FP64,
64 x 9 in the narrow forms) and chunks, against the two-pass path: the same
bits.  Extents of one node, one less, equal and one more than a tile, a ragged
last tile in both directions, fewer planes than the shortest chunk of 8, and a
grid whose chunks do not divide it."""
import numpy as np
import pytest
import torch

from gpu_util import droplet_rho, make_sim, say
from oracle import eos
from paper_2504_03819_amd import lbfe

pytestmark = pytest.mark.gpu

OM = [1.0, 1.0, 1.0, 0.5] + [1.0] * 7
SHAPES = [(1, 1, 1), (3, 2, 5), (7, 12, 31), (8, 13, 32), (9, 14, 33), (4, 8, 63), (17, 9, 64), (5, 10, 65),
          (26, 27, 97), (40, 19, 130)]


@pytest.mark.parametrize("walls", ["none", "still", "moving"])
@pytest.mark.parametrize("precision", ["fp64", "fp32", "fp16dev", "fp16dev_f0fp32"])
def test_fused_tiles_equal_the_two_passes(walls, precision):
    T = eos.temperature(0.8)
    for shape in SHAPES:
        nz, ny, nx = shape
        kw = dict(T=T, precision=precision)
        if walls != "none":
            nz += 2
            kw.update(walls_z=1, wet_mode=1, wet_value=1.2, omega=OM)
        if walls == "moving":
            kw.update(wall_u=(0.01, -0.02, 0.015, 0.0))
        say(f"fused tiles: {(nz, ny, nx)} walls={walls} {precision}")
        rho0 = torch.tensor(droplet_rho((nz, ny, nx), T, walls=walls != "none", radius=max(2.0, min(ny, nx) / 3.0)))
        g = np.random.Generator(np.random.PCG64(8))
        u0 = torch.tensor(0.02 * g.uniform(-1, 1, (3, nz, ny, nx)))
        out = []
        for path in (lbfe.PATH_TWO_PASS, lbfe.PATH_FUSED):
            s = make_sim(nx=nx, ny=ny, nz=nz, step_path=path, **kw)
            s.init_density(rho0, u0)
            s.step(3)
            out.append((s.get_state(), s.field(2)))
        assert torch.equal(out[0][0], out[1][0]) and torch.equal(out[0][1], out[1][1]), shape


@pytest.mark.parametrize("walls", ["none", "still", "moving"])
@pytest.mark.parametrize("path", [lbfe.PATH_TWO_PASS, lbfe.PATH_FUSED, lbfe.PATH_STATE])
def test_fields_after_steps_are_those_of_the_stored_state(path, walls):
    """The fields read the density and momentum that the fused and state paths
    leave behind, twice the same, and the same as a context that only got the
    populations."""
    if path == lbfe.PATH_STATE and walls == "moving":
        pytest.skip("the state path has no moving walls")
    shape = (11, 14, 33)
    T = eos.temperature(0.8)
    kw = dict(nx=33, ny=14, nz=11, T=T, precision="fp64")
    if walls != "none":
        kw.update(walls_z=1, wet_mode=1, wet_value=1.2)
    if path != lbfe.PATH_STATE and walls != "none":
        kw.update(omega=OM)
    if walls == "moving":
        kw.update(wall_u=(0.01, -0.02, 0.015, 0.0))
    a, b = make_sim(step_path=path, **kw), make_sim(step_path=path, **kw)
    a.init_density(torch.tensor(droplet_rho(shape, T, walls=walls != "none", radius=4.0)))
    for n in (1, 2, 3):
        a.step(n)
        b.set_state(a.get_state())
        fb = b.fields()
        for _ in range(2):
            fa = a.fields()
            for name in fb:
                assert torch.equal(fa[name], fb[name]), (n, name)
        assert a.reduce() == b.reduce()
