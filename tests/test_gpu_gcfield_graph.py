"""A damage solve captured in a HIP graph keeps the toughness field that it was captured with (or
without) when the handle's field is set or cleared afterwards, and clearing enqueues nothing, so
that it can stand inside a capture.  Every replay against the bits of the eager solve."""
import numpy as np
import pytest
import torch

import workloads as w

pytestmark = pytest.mark.gpu


def _setup(dtype):
    from paper_2606_23458_amd import Simulator, State
    from paper_2606_23458_amd.sim import CgConfig, default_tol
    p = w.small_plate(60, 30, jitter=0.15, seed=4, model=2, random_diag=True)
    sim = Simulator(p, dtype=dtype, cg=CgConfig(tol=default_tol(dtype), start=0, check_every=0, rounds=40))
    r = np.random.default_rng(3)
    z = np.zeros((p.n_nodes, 2))
    s = State.from_user(sim.mesh, [{"u": z, "v": z, "a": z, "d": p.d0, "H": r.uniform(0, 8000.0, p.n_elems)}])
    return p, sim, s, r.uniform(0.4, 2.5, p.n_elems)


def _solve(sim, s, d):
    sim.damage(s.H, s.d, d, sim.active)


@pytest.mark.parametrize("dtype", ["f64", "f32"])
@pytest.mark.parametrize("with_field", [False, True])
def test_captured_solve_keeps_its_field(dtype, with_field):
    p, sim, s, phi = _setup(dtype)
    if with_field:
        sim.set_gc_field([phi])
    d = torch.zeros_like(s.d)
    _solve(sim, s, d)
    torch.cuda.synchronize()
    want = d.clone()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        _solve(sim, s, d)
    sim.set_gc_field(None if with_field else [phi])
    other = torch.zeros_like(d)
    for _ in range(3):
        d.zero_()
        g.replay()
        _solve(sim, s, other)
        torch.cuda.synchronize()
        assert torch.equal(d, want)
        assert not torch.equal(other, want)
    st = sim.cg_stats()[0]
    assert st["flags"] == 0, st


def test_field_cleared_inside_a_capture():
    p, sim, s, phi = _setup("f64")
    d = torch.zeros_like(s.d)
    _solve(sim, s, d)
    torch.cuda.synchronize()
    want = d.clone()
    sim.set_gc_field([phi])
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        sim.set_gc_field(None)
        _solve(sim, s, d)
    for _ in range(2):
        d.zero_()
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(d, want)
