"""What a damage solve delivers passes its own stopping test: a second solve that starts at the
delivered d (d_prev = 0, and -d in the output array, so the extrapolated start is d itself) ends
with its set-up round.  In FP32 the CG's iterate has more digits than d; tolerances down to the
rounding of d, so that testing the one and delivering the other would show.  d in [1/2, 1] is
rounded by up to 3e-8, which moves a scaled residual by up to (1 + sum |A_ij|/A_ii) 3e-8, about
9e-8: below that a solve may say that it has not converged, but not that it has."""
import numpy as np
import pytest
import torch

import workloads as w

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,tol", [("f64", 1e-12), ("f32", 1e-6), ("f32", 2e-7), ("f32", 6e-8)])
@pytest.mark.parametrize("precond", [0, 1, 3])
@pytest.mark.parametrize("seed", [1, 2])
def test_delivered_damage_passes_the_stopping_test(dtype, tol, precond, seed):
    from paper_2606_23458_amd import Simulator, State
    from paper_2606_23458_amd._lib import PF_ERR_NOT_CONVERGED, PfError
    from paper_2606_23458_amd.sim import CgConfig
    p = w.small_plate(150, 75, jitter=0.15, seed=seed, model=2, random_diag=True)
    sim = Simulator(p, dtype=dtype, cg=CgConfig(tol=tol, precond=precond, max_iter=500))
    r = np.random.default_rng(seed)
    z = np.zeros((p.n_nodes, 2))
    # history everywhere: the minimiser lies inside the bounds, so no node is clamped at the end
    s = State.from_user(sim.mesh, [{"u": z, "v": z, "a": z, "d": z[:, 0], "H": r.uniform(3000.0, 30000.0, p.n_elems)}])
    d = torch.zeros_like(s.d)
    try:
        sim.damage(s.H, s.d, d, sim.active)
    except PfError as e:
        assert e.status == PF_ERR_NOT_CONVERGED and dtype == "f32" and tol < 9e-8
        return
    torch.cuda.synchronize()
    first = sim.cg_stats()[0]
    again = -d
    sim.damage(s.H, s.d, again, sim.active, sim.active)
    torch.cuda.synchronize()
    second = sim.cg_stats()[0]
    assert first["flags"] == 0 and first["iters"] > 3 and 0.0 < float(d.min()) and float(d.max()) < 1.0, first
    assert second["iters"] == 1 and second["resid"] <= tol, (first, second)
    assert torch.equal(again, d)
