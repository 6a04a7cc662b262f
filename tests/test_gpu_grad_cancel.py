"""dL/dGc where its terms cancel: an AT1 plate before the waves reach the notch (H = 0 at every
free node).  A and b both scale with Gc there, the minimiser does not depend on Gc, and dL/dGc is
exactly 0; the elements' terms, which do not vanish one by one, sum to lambda'(A d - b)/Gc on the
free nodes.  The forward solve leaves |r_i| <= tol A_ii there, so

    |dL/dGc| <= (tol / Gc) sum_i |lambda_i| A_ii + rounding of the sum's terms,

with nothing left of the digits of single terms.  The bound is evaluated in 64 bits by the oracle."""
import numpy as np
import pytest
import scipy.sparse.linalg as spla
import torch

import workloads as w
from oracle.damage import assemble_damage, node_area, stiffness_matrix
from oracle.step import Sim as OSim

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("tol", [1e-8, 1e-12])
@pytest.mark.parametrize("nx,ny,diag", [(90, 40, False), (61, 43, True), (100, 35, True)])
def test_cancelling_gradient_is_bounded_by_the_solve(tol, nx, ny, diag):
    from paper_2606_23458_amd import Simulator, State
    from paper_2606_23458_amd.grad import backward_step
    from paper_2606_23458_amd.sim import CgConfig
    p = w.small_plate(nx, ny, jitter=0.15, seed=nx, model=1, split="voldev", random_diag=diag)
    sim = Simulator(p, dtype="f64", cg=CgConfig(tol=tol), cg_adj=CgConfig(tol=1e-14))
    s0 = State.from_user(sim.mesh, [{"u": p.u0, "v": p.v0, "a": p.a0, "d": p.d0, "H": p.H0}])
    s1, act = State(sim.mesh), torch.zeros(sim.mesh.n_nodes, dtype=torch.uint8, device="cuda")
    s1.d.copy_(s0.d)
    sim.step_into(s0, s1, act, None)
    dbar = 1e-2 * (1.5 + np.cos(p.xy[:, 0] / (9 * 2.5e-4)) * np.sin(p.xy[:, 1] / (7 * 2.5e-4)))
    adj1, adj0 = State(sim.mesh), State(sim.mesh)
    adj1.nodes[6].copy_(torch.tensor(sim.mesh.nodes_to_internal([dbar])))
    dgc = torch.zeros(1, dtype=torch.float64, device="cuda")
    backward_step(sim, s0, s1, act, adj1, adj0, dgc)
    torch.cuda.synchronize()

    mesh = OSim(p).mesh
    got = s1.to_user()[0]
    held = sim.mesh.nodes_from_internal(act)[0] != 0
    free = np.flatnonzero(~held)
    A, _ = assemble_damage(mesh, got["H"], p.Gc, p.l0, 1)
    # the regime: no history at any element of a free node, and free nodes there are
    assert len(free) > nx // 4
    at_free = (~held)[p.tri].any(1)
    assert np.all(got["H"][at_free] == 0.0)
    lam = np.zeros(p.n_nodes)
    lam[free] = spla.spsolve(A[free][:, free].tocsc(), dbar[free])
    # the terms' sizes, node by node (every one of a row's products counted)
    K, wn = stiffness_matrix(mesh), node_area(mesh)
    terms = np.abs(lam) @ (0.75 * p.l0 * (abs(K) @ np.abs(got["d"])) + 0.375 / p.l0 * wn)
    bound = tol / p.Gc * np.sum(np.abs(lam) * A.diagonal()) + 64 * np.finfo(float).eps * terms
    print(f"|dL/dGc| {abs(float(dgc[0])):.2e}, bound {bound:.2e}, terms {terms:.2e}")
    assert abs(float(dgc[0])) <= bound
    assert bound < 1e-4 * terms
