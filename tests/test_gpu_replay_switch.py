"""Calls of one plan that change between direct launches (one or two steps, on
the caller's stream) and graph replay (more, on the plan's own stream): the same
bits as a plan without graphs.

Moving particles make a run replay; with the deterministic deposit every sum is
exact or in a fixed order, so no tolerance is needed.
"""
import numpy as np
import pytest

from paper_2606_25026_amd import inputs

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

CALLS = (1, 3, 2, 20, 1, 1, 10, 2, 7)


def make(wdm, halos, graphs):
    plan = wdm.Plan([wdm.make_config(w.n, n_particles=w.pos.shape[0], particle_mass=w.particle_mass,
                                     flags=wdm.WDM_DETERMINISTIC_DEPOSIT) for w in halos])
    wdm.wdm_use_graphs(plan.handle, graphs)
    wdm.wdm_set_sort_interval(plan.handle, 8)
    for k, w in enumerate(halos):
        wdm.wdm_set_state(plan.handle, k, torch.from_numpy(w.psi.astype(np.complex64)).cuda(),
                          torch.from_numpy(w.pos.astype(np.float32)).cuda(),
                          torch.from_numpy(w.vel.astype(np.float32)).cuda())
    return plan


def fields(wdm, plan, halos):
    out = []
    for k, w in enumerate(halos):
        psi = torch.empty((w.n,) * 3, dtype=torch.complex64, device="cuda")
        p = torch.empty((w.pos.shape[0], 3), dtype=torch.float32, device="cuda")
        v = torch.empty_like(p)
        wdm.wdm_get_psi(plan.handle, k, psi)
        wdm.wdm_particles(plan.handle, k, p, v)
        out += [psi, p, v]
    return [x.cpu().numpy() for x in out]


@pytest.mark.parametrize("side_stream", [False, True])
@pytest.mark.parametrize("sizes", [(32,), (64, 32, 64)], ids=str)
def test_mixed_call_lengths(wdm, sizes, side_stream):
    halos = [inputs.coupled_halo(n=n, n_particles=3000 + 500 * i, seed=20 + i, steps=0)
             for i, n in enumerate(sizes)]
    dt = min(w.dt for w in halos)
    s = torch.cuda.Stream() if side_stream else torch.cuda.current_stream()
    with torch.cuda.stream(s):
        replay, direct = make(wdm, halos, True), make(wdm, halos, False)
        for i, k in enumerate(CALLS):
            wdm.wdm_step(replay.handle, k, dt)
            wdm.wdm_step(direct.handle, k, dt)
            if i % 2:    # every other call follows the last without a wait
                a, b = fields(wdm, replay, halos), fields(wdm, direct, halos)
                assert all(np.array_equal(x, y) for x, y in zip(a, b)), f"call {i} of {k} steps"
        wdm.wdm_energy(replay.handle, 0)
        a, b = fields(wdm, replay, halos), fields(wdm, direct, halos)
        assert all(np.array_equal(x, y) for x, y in zip(a, b))
        assert not np.array_equal(a[1], halos[0].pos.astype(np.float32))
    replay.close()
    direct.close()
