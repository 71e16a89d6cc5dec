"""lbfe_step_record refuses states and records that overlap each other or the
context's workspace, and leaves the context as it was."""
import ctypes

import pytest
import torch

from gpu_util import droplet_rho, make_sim
from oracle import eos
from paper_2504_03819_amd import lbfe

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision", ["fp64", "fp16dev_f0fp32"])
def test_overlaps_are_refused(precision):
    nz, ny, nx = 6, 7, 16
    T = eos.temperature(0.8)
    sim = make_sim(nx=nx, ny=ny, nz=nz, T=T, precision=precision)
    sim.init_density(torch.tensor(droplet_rho((nz, ny, nx), T, radius=2.0)))
    L = lbfe.lib()
    sb = sim.state_bytes()
    n = ctypes.c_size_t()
    assert L.lbfe_aux_bytes(sim._ctx, ctypes.byref(n)) == lbfe.OK
    ab = n.value
    up = lambda v: (v + 255) & ~255
    pool = torch.zeros(up(2 * sb) + up(sb) + up(ab) + 1024, dtype=torch.uint8, device="cuda:0")
    base = up(pool.data_ptr())
    s_in, s_out, rec = base, base + up(sb), base + 2 * up(sb)
    ws = up(sim.workspace.data_ptr())
    assert L.lbfe_workspace_bytes(ctypes.byref(sim.params), ctypes.byref(n)) == lbfe.OK
    f0, f1, rho = ws, ws + up(sb), ws + 2 * up(sb)
    last = ws + up(n.value) - 256
    V = ctypes.c_void_p
    assert L.lbfe_get_state(sim._ctx, V(s_in)) == lbfe.OK
    before = sim.get_state()

    def step(i, o, r):
        return L.lbfe_step_record(sim._ctx, V(i), ctypes.c_int64(5), V(o), V(r))

    bad = [(s_in, s_in, rec), (s_in, s_in + 256, rec), (s_in + 256, s_in, rec),  # the states
           (s_in, s_out, s_in), (s_in, s_out, s_out + 256), (s_in, None, s_in + 256),  # the record
           (s_in, f0, rec), (s_in, f1, rec), (s_in, last, rec),  # the workspace
           (s_in, s_out, rho), (s_in, None, last), (rho, s_out, rec), (f0 + 256, None, rec)]
    for args in bad:
        assert step(*args) == lbfe.E_INVAL, args
    assert torch.equal(sim.get_state(), before) and sim.step_count == 0
    # adjacent buffers (their padding zero, as in a workspace), and a lattice of the context as the input, are fine
    assert step(s_in, s_out, rec) == lbfe.OK
    assert torch.equal(sim.get_state(), before) and sim.step_count == 0
    assert step(f0, None, rec) == lbfe.OK and sim.step_count == 6
    got = torch.empty(sb, dtype=torch.uint8, device="cuda:0")
    got.copy_(pool[s_out - pool.data_ptr():][:sb])
    assert torch.equal(sim.get_state(), got)
