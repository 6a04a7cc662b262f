"""How many launches a round takes follows the row tiles of the damage passes, not the explicit
step's tiles: the pass's last workgroup combines up to 1024 row tiles of an instance and 3072 of
a handle, and a launch of its own does so above, at any tile_nodes from 128 up; both orders of
launches reach the same minimiser.  Tolerance: the stopping residual of 1e-12 times the
operator's condition number (about 30 at l0 = 2h), with a factor of three."""
import numpy as np
import pytest
import torch

import workloads as w

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nx,ny,plates,many", [(400, 370, 1, False), (700, 372, 1, False), (760, 380, 1, True),
                                               (256, 128, 11, False), (256, 128, 12, True)])
def test_launches_per_round_follow_the_row_tiles(nx, ny, plates, many):
    from paper_2606_23458_amd import Mesh, Simulator, State
    from paper_2606_23458_amd.sim import CgConfig
    p = w.small_plate(nx, ny, jitter=0.1, seed=2, model=2)
    r = np.random.default_rng(1)
    H, z = r.uniform(0.0, 8000.0, p.n_elems), np.zeros((p.n_nodes, 2))
    got = []
    for tile in (256, 1024):
        mesh = Mesh([p] * plates, "f64", tile)
        sim = Simulator([p] * plates, dtype="f64", mesh=mesh, cg=CgConfig(tol=1e-12, start=0))
        s = State.from_user(mesh, [{"u": z, "v": z, "a": z, "d": p.d0, "H": H}] * plates)
        d = torch.zeros_like(s.d)
        sim.timer(True)
        sim.damage(s.H, s.d, d)
        _, passes = sim.timer_read(1)
        _, reductions = sim.timer_read(4)
        sim.timer(False)
        st = sim.cg_stats()
        assert all(x["flags"] == 0 for x in st)
        assert reductions == (passes if many else 0), (tile, passes, reductions)
        got.append(mesh.nodes_from_internal(d))
    for a, b in zip(*got):
        assert np.max(np.abs(a - b)) < 1e-10
