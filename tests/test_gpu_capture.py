"""lbfe_reduce_into captured into a graph: every replay reduces the state that
the lattice holds then, also where the eager call would use the density and
momentum that the last step left (fused and state paths)."""
import pytest
import torch

from gpu_util import droplet_rho, make_sim, say
from oracle import eos
from paper_2504_03819_amd import lbfe

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("walls", [0, 1])
@pytest.mark.parametrize("path", [lbfe.PATH_TWO_PASS, lbfe.PATH_FUSED, lbfe.PATH_STATE])
def test_replays_reduce_the_state_of_the_moment(path, walls):
    shape = nz, ny, nx = (12, 14, 33)
    T = eos.temperature(0.85)
    say(f"captured reduction: path {path} walls {walls}")
    stream = torch.cuda.Stream()
    out = torch.zeros(8, dtype=torch.float64, device="cuda:0")
    with torch.cuda.stream(stream):
        sim = make_sim(nx=nx, ny=ny, nz=nz, T=T, walls_z=walls, step_path=path)
        states = []
        for seed in (1, 2, 3):
            sim.init_density(torch.tensor(droplet_rho(shape, T, walls=bool(walls), radius=3.0 + seed, seed=seed)))
            sim.step(2)
            states.append(sim.get_state())
        sim.reduce_into(out)  # the scratch's address is found outside the capture
        stream.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=stream):
            sim.reduce_into(out)
        for k in (0, 1, 2, 1, 0):
            sim.set_state(states[k])
            out.zero_()
            graph.replay()
            stream.synchronize()
            got = out.cpu().tolist()
            assert got == sim.reduce(), k
            # back on the same lattice: the paths take the two in turn, the
            # state path holds its own form in one until the last step
            sim.step(3 if path == lbfe.PATH_STATE else 2)
            graph.replay()
            stream.synchronize()
            assert out.cpu().tolist() == sim.reduce(), k
