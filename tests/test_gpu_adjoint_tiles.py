"""The transposed-stencil marches of the adjoint at the edges of their tiles
(32 x 12 and, from 2^20 nodes, 64 x 13; 32 x 16 for the density part).

Narrow tiles: one adjoint step against oracle reverse mode on extents of one
node, one less, equal to and one more than a tile.  Wide tiles: a periodic
state repeated to more than 2^20 nodes has the repeated adjoint, node by node
the same sums, so lambda must be equal bit for bit to that of the small box
(narrow tiles), and the parameter gradients are the number of copies times
those of the small box (to the rounding of the reductions)."""
import numpy as np
import pytest
import torch

from gpu_util import droplet_rho, make_sim, oracle_params, rel_err, say
from oracle import eos, lbm
from paper_2504_03819_amd import inputs, lbfe
from test_gpu_adjoint import _oracle_vjp

pytestmark = pytest.mark.gpu

SHAPES = [((1, 1, 1), False), ((2, 13, 33), False), ((5, 12, 32), False), ((4, 11, 31), False), ((3, 25, 65), False),
          ((5, 13, 33), True), ((4, 17, 31), True)]


@pytest.mark.parametrize("shape,walls", SHAPES, ids=[f"{s}{'w' if w else ''}" for s, w in SHAPES])
def test_tile_edges_match_oracle_reverse_mode(shape, walls):
    say(f"adjoint tiles {shape} walls={walls}")
    T = eos.temperature(0.8)
    nz, ny, nx = shape
    extra = dict(wet_mode=1, wet_value=1.3) if walls else {}
    sim = make_sim(nx=nx, ny=ny, nz=nz, T=T, walls_z=int(walls), adjoint=1, **extra)
    p = oracle_params(sim)
    g = np.random.Generator(np.random.PCG64(7))
    f0 = lbm.init(torch.tensor(droplet_rho(shape, T, walls=walls, radius=max(1.0, min(shape) / 3))), p,
                  torch.tensor(0.03 * g.uniform(-1, 1, (3,) + shape)))
    f = f0 + torch.tensor(inputs.uniform_noise(tuple(f0.shape), 2e-4, 3)) * (f0 != 0)
    lam = torch.tensor(g.uniform(-1, 1, (27,) + shape))
    sl = slice(1, -1) if walls else slice(None)
    if walls:
        lam[:, 0] = lam[:, -1] = 0
    sim.set_populations(f)
    sim.adjoint_seed_populations(lam)
    sim.adjoint_step(None)
    lo, ko, _, no = _oracle_vjp(f, lam, p)
    gg = sim.adjoint_grads()
    assert rel_err(sim.adjoint_state().cpu()[:, sl], lo[:, sl]) < 1e-11
    # a one-node box has no gradient with respect to kappa (its Laplacian vanishes)
    assert abs(gg["kappa"] - ko) < 1e-9 * max(abs(ko), 1e-3) and abs(gg["nu"] - no) < 1e-9 * max(abs(no), 1e-3)


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
def test_repeated_state_has_the_repeated_adjoint(precision):
    shape, reps = (13, 27, 66), (4, 7, 2)
    T = eos.temperature(0.85)
    g = np.random.Generator(np.random.PCG64(11))
    rho0 = torch.tensor(droplet_rho(shape, T, radius=4.0))
    u0 = torch.tensor(0.03 * g.uniform(-1, 1, (3,) + shape))
    seed = torch.tensor(g.uniform(-1, 1, shape))
    out = []
    for r in ((1, 1, 1), reps):
        nz, ny, nx = (a * b for a, b in zip(shape, r))
        sim = make_sim(nx=nx, ny=ny, nz=nz, T=T, adjoint=1, precision=precision, step_path=1)
        sim.init_density(rho0.repeat(r), u0.repeat((1,) + r))
        sim.step(2)
        st = sim.get_state()
        sim.adjoint_seed(seed.repeat(r))
        sim.adjoint_step(st)
        sim.adjoint_step(st)
        out.append((sim.adjoint_state(), sim.adjoint_grads()))
        sim.close()
    (a, ga), (b, gb) = out
    assert torch.equal(a.repeat((1,) + reps), b)
    n = reps[0] * reps[1] * reps[2]
    for k in ("kappa", "nu"):  # sums of 1.3e6 signed terms of magnitudes up to ~1e2 of the mean
        assert abs(gb[k] - n * ga[k]) < 1e-9 * abs(n * ga[k]), (k, ga[k], gb[k])


@pytest.mark.parametrize("walls", ["none", "still", "moving"])
@pytest.mark.parametrize("form", ["fp64", "fp32", "fp16dev_f0fp32"])
def test_step_record_is_step_aux_without_the_copies(form, walls):
    """Steps between stored states (and at last into the context) against
    set_state, step_aux and get_state: the same states at the fluid nodes, the
    same records and lambda."""
    nz, ny, nx = shape = (9, 10, 21)
    T = eos.temperature(0.8)
    kw = dict(nx=nx, ny=ny, nz=nz, T=T, precision=form, adjoint=1)
    if walls != "none":
        kw.update(walls_z=1, wet_mode=1, wet_value=1.2)
    if walls == "moving":
        kw.update(wall_u=(0.01, -0.02, 0.015, 0.0))
    a, b = make_sim(**kw), make_sim(**kw)
    a.init_density(torch.tensor(droplet_rho(shape, T, walls=walls != "none", radius=3.0)))
    first = a.get_state()
    sa, ra, sb, rb = [first], [], [first], []
    for t in range(3):
        ra.append(a.aux_record().zero_())
        a.step_aux(ra[-1])
        sa.append(a.get_state())
        rb.append(b.aux_record().zero_())
        sb.append(None if t == 2 else torch.zeros_like(first))
        b.step_record(sb[t], t, rb[-1], sb[-1])
    assert torch.equal(a.get_state(), b.get_state()) and b.step_count == 3
    for t in range(3):
        assert torch.equal(sa[t], sb[t]) and torch.equal(ra[t], rb[t]), t
    assert torch.equal(a.fields()["mu"], b.fields()["mu"])
    bad = torch.zeros(first.numel() + 8, dtype=torch.uint8, device="cuda:0")[8:]
    for args in ((first, 0, rb[0], first), (bad, 0, rb[0]), (first, -1, rb[0]), (first, 0, rb[0], bad)):
        with pytest.raises(lbfe.LBFEError) as e:
            b.step_record(*args)
        assert e.value.code == lbfe.E_INVAL


@pytest.mark.parametrize("form", ["fp64", "fp32"])
def test_init_gradient_with_the_last_term_pending(form):
    """lbfe_adjoint_init_density adds the last term of lambda(0) as it reads
    it; reading lambda out first (which completes it in place) gives the same
    gradients, a second call the same again, and a second seed of a used
    workspace those of a fresh one."""
    nz, ny, nx = shape = (8, 9, 19)
    T = eos.temperature(0.8)
    rho0 = torch.tensor(droplet_rho(shape, T, walls=True, radius=3.0))
    g = torch.tensor(inputs.uniform_noise(shape, 1.0, 5), device="cuda:0")
    kw = dict(nx=nx, ny=ny, nz=nz, T=T, precision=form, adjoint=1, walls_z=1, wet_mode=1, wet_value=1.2)
    out = []
    for read_first in (False, True):
        s = make_sim(**kw)
        for _ in range(2):  # the second time on used arrays
            s.init_density(rho0)
            f = s.get_state()
            s.adjoint_seed(g)
            s.adjoint_step(f)
            if read_first:
                s.adjoint_state()
            a = s.adjoint_init_density()
            out.append((a, s.adjoint_grads()))
        assert torch.equal(s.adjoint_init_density(), a)
    for a, gr in out[1:]:
        assert torch.equal(a, out[0][0]) and gr == out[0][1]
