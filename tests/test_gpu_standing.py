"""A damage field that stands still: at a constant history, repeated FP32 steps with the extrapolated
start settle within a dozen solves, and from then on each ends with its set-up round and gives the
same bits.  (A start that carries movements below the tolerance on creeps upward instead: d cannot
come back down, and every few steps a solve has to bring the residual back under the
tolerance; FP64 starts carry every movement on.)"""
import numpy as np
import pytest
import torch

import workloads as w

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["f32"])
@pytest.mark.parametrize("model", [1, 2])
@pytest.mark.parametrize("nx,ny", [(200, 100), (400, 200)])
def test_standing_damage_settles(dtype, model, nx, ny):
    from paper_2606_23458_amd import Simulator
    p = w.small_plate(nx, ny, jitter=0.2, seed=2, model=model, split="voldev", random_diag=True)
    sim = Simulator(p, dtype=dtype)
    cen = p.xy[p.tri].mean(1)
    # a hill of history ahead of the notch, above AT1's threshold at its top
    hc = 3 * p.Gc / (16 * p.l0)
    tip = np.array([nx // 2 * 2.5e-4, ny // 2 * 2.5e-4])
    H = 3 * hc * np.exp(-((cen - tip) ** 2).sum(1) / (8 * 2.5e-4) ** 2)
    H = torch.tensor(sim.mesh.elems_to_internal([H]), dtype=sim.mesh.dtype, device="cuda")
    prev, cur, act = torch.zeros_like(sim.state.d), sim.state.d.clone(), sim.active.clone()
    rounds, same = [], []
    for _ in range(60):
        out, act2 = prev.clone(), torch.zeros_like(act)
        sim.damage(H, cur, out, act2, act)
        torch.cuda.synchronize()
        rounds.append(sim.cg_stats()[0]["iters"])
        same.append(torch.equal(out, cur))
        prev, cur, act = cur, out, act2
    assert rounds[0] > 3
    assert rounds[12:] == [1] * 48 and all(same[12:]), rounds


@pytest.mark.parametrize("dtype", ["f64", "f32"])
def test_non_finite_start_is_reported(dtype):
    """A NaN in the output array, which holds the damage before d_prev on entry, is not hidden."""
    from paper_2606_23458_amd import Simulator
    from paper_2606_23458_amd._lib import PF_ERR_NONFINITE, PfError
    p = w.small_plate(60, 30, seed=2, model=2)
    sim = Simulator(p, dtype=dtype)
    H = torch.full((p.n_elems,), 500.0, dtype=sim.mesh.dtype, device="cuda")
    out = torch.zeros_like(sim.state.d)
    out[7] = float("nan")
    with pytest.raises(PfError) as e:
        sim.damage(H, sim.state.d, out, torch.zeros_like(sim.active), sim.active)
    assert e.value.status == PF_ERR_NONFINITE
