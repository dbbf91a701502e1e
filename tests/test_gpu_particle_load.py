"""Particles go in in the caller's order and come back in it, through the sort at
loading and the sorts between steps, for counts at the edges of a wavefront and of
a sort tile, clustered in few cells or spread, at grids whose keys take one to four
passes.  Positions and velocities are moved, not computed: bit for bit.
"""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [16, 64, 96, (16, 16, 512)])
@pytest.mark.parametrize("count", [1, 2, 63, 257, 1023, 1024, 1025, 5000])
def test_round_trip(wdm, n, count):
    rng = np.random.default_rng(count)
    plan = wdm.Plan(wdm.make_config(n, four_pi_G=0.0, n_particles=count, particle_mass=1.0))
    shape = (n,) * 3 if isinstance(n, int) else n
    psi = torch.zeros(shape, dtype=torch.complex64, device="cuda")
    pos = rng.random((count, 3)).astype(np.float32)
    pos[::2] = 0.3 + 1e-3 * pos[::2]                     # half of them in a few cells
    vel = (1e-3 * rng.standard_normal((count, 3))).astype(np.float32)
    p, v = torch.empty((count, 3), device="cuda"), torch.empty((count, 3), device="cuda")
    for shift in (0.0, 2.0):                             # outside the box: wrapped
        wdm.wdm_set_state(plan.handle, 0, psi, torch.from_numpy(pos + np.float32(shift)).cuda(),
                          torch.from_numpy(vel).cuda())
        wdm.wdm_particles(plan.handle, 0, p, v)
        want = (pos + np.float32(shift)).astype(np.float64) % 1.0
        assert np.array_equal(p.cpu().numpy(), want.astype(np.float32) % np.float32(1.0))
        assert np.array_equal(v.cpu().numpy(), vel)
    wdm.wdm_set_sort_interval(plan.handle, 1)
    wdm.wdm_step(plan.handle, 3, 1e-3)
    wdm.wdm_particles(plan.handle, 0, p, v)
    assert np.array_equal(v.cpu().numpy(), vel)          # no force: the velocities as given
