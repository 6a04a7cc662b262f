"""A solve that a resumed call continues with another preconditioner degree than it was begun
with: the rows that the set-up assembled bound the degree, and the exact minimiser of the QP is
reached as from a solve of one degree.  Tolerances: the solver's stopping residual (1e-12 FP64,
1e-6 FP32) times the operator's condition number (about 30 at l0 = 2h), with a factor of three."""
import numpy as np
import pytest
import torch

import workloads as w
from oracle.damage import DamageQP
from oracle.step import Sim as OSim

pytestmark = pytest.mark.gpu

TOL = {"f64": 1e-10, "f32": 1e-4}


@pytest.mark.parametrize("dtype", ["f64", "f32"])
@pytest.mark.parametrize("first,then", [(1, 4), (1, 0), (2, 4), (2, 0), (4, 1), (0, 1), (0, 2)])
def test_resumed_solve_of_another_degree(dtype, first, then):
    from paper_2606_23458_amd import Mesh, Simulator, State
    from paper_2606_23458_amd.sim import CgConfig, default_tol
    p = w.small_plate(120, 60, jitter=0.15, seed=4, model=2, random_diag=True)
    r = np.random.default_rng(8)
    H = r.uniform(0, 8000.0, p.n_elems) * (r.random(p.n_elems) < 0.5)
    lb = np.where(r.random(p.n_nodes) < 0.2, r.uniform(0, 0.9, p.n_nodes), 0.0)
    mesh = Mesh([p], dtype, 256)
    sim = Simulator(p, dtype=dtype, mesh=mesh)
    z = np.zeros((p.n_nodes, 2))
    one, two = (State.from_user(mesh, [{"u": z, "v": z, "a": z, "d": x, "H": h}])
                for x, h in ((0 * lb, 1e3 * H[::-1] + 1e6), (lb, H)))
    d = torch.zeros_like(two.d)
    tol = default_tol(dtype)
    # rows of another solve, with entries a thousand times larger, stand in the handle before
    sim.damage(one.H, one.d, d, cg=CgConfig(tol=tol, start=0))
    sim.damage(two.H, two.d, d, sim.active, cg=CgConfig(tol=tol, start=0, check_every=0, rounds=4, precond=first))
    torch.cuda.synchronize()
    begun = sim.cg_stats()[0]
    sim.damage(two.H, two.d, d, sim.active, cg=CgConfig(tol=tol, start=0, resume=1, precond=then, max_iter=400))
    torch.cuda.synchronize()
    st = sim.cg_stats()[0]
    got = mesh.nodes_from_internal(d.double())[0]
    ref = DamageQP(OSim(p).mesh, p.l0, 2).solve(H, p.Gc, lb)[0]
    assert begun["iters"] == 4 and st["flags"] == 0, (begun, st)
    assert np.max(np.abs(got - ref)) < TOL[dtype], st
