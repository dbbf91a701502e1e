"""Which form a step takes, and the four-pass kernels that only boxes with many
plane tiles reach: every plane pass (nx, R2) and every z pass (nz, R1) that is
built runs in a box of this list, is seen to run (the per-pass timing names the
passes) and agrees with the FP64 oracle; boxes below the tile rule or without
the form take the eight passes.

Tolerances: a transform of N points in single precision is off by about
eps log2 N = 6e-8 * 23, of which a step has four, so three steps stay below
5e-6; in double precision the same count gives 1e-14.
"""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

TOL = {0: 5e-6, 1: 1e-13}

# y length -> (R1, R2)
RADIX = {16: (4, 4), 32: (8, 4), 64: (8, 8), 96: (12, 8), 128: (16, 8), 192: (12, 16),
         256: (16, 16)}
SIDES = (16, 32, 64, 96, 128, 192, 256)

FOUR = [(16, 16, 16), (16, 32, 32), (16, 64, 128), (16, 96, 128), (16, 128, 192), (16, 192, 32),
        (32, 16, 32), (32, 32, 256), (32, 64, 64), (32, 96, 256), (32, 128, 256), (32, 192, 192),
        (64, 16, 64), (64, 32, 96), (64, 96, 32), (64, 128, 96), (64, 256, 128), (96, 32, 16),
        (96, 96, 96), (96, 192, 96), (96, 192, 128), (128, 32, 32), (128, 64, 192), (128, 192, 64), (128, 256, 32),
        (192, 32, 128), (192, 128, 64), (192, 192, 192), (256, 32, 192), (256, 64, 96),
        (256, 128, 128), (256, 256, 32)]
# too few plane tiles; a pair (nz, R1) that is not built; a side that is not
EIGHT = [(192, 32, 32), (256, 32, 16), (256, 64, 32), (96, 256, 32), (192, 192, 32), (16, 256, 16),
         (32, 96, 16), (16, 16, 256), (32, 384, 32), (384, 32, 32), (192, 192, 128)]
# the form depends on the precision: four passes in complex64 alone
SINGLE = [(128, 16, 32), (192, 192, 96)]


def test_boxes_reach_every_kernel():
    planes = {(nx, RADIX[ny][1]) for nx, ny, _ in FOUR}
    assert planes == {(nx, r2) for nx in SIDES for r2 in (4, 8, 16)}
    rows = {(nz, RADIX[ny][0]) for _, ny, nz in FOUR}
    assert rows == ({(nz, 4) for nz in (16, 32, 64)} | {(nz, 8) for nz in SIDES} |
                    {(nz, r1) for nz in SIDES[1:] for r1 in (12, 16)})


def rel_l2(a, b):
    return float(np.linalg.norm((a - b).ravel()) / np.linalg.norm(b.ravel()))


@pytest.mark.gpu
@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("n", FOUR + EIGHT + SINGLE, ids=lambda n: "x".join(map(str, n)))
def test_form_and_result(wdm, orc, n, prec):
    rng = np.random.default_rng(sum(n))
    L = (1.0, 0.75, 1.25)
    psi = (rng.standard_normal(n) + 1j * rng.standard_normal(n)).astype(
        np.complex128 if prec else np.complex64)
    # the drift turns the fastest mode by about a radian a step, the kick by about 0.1
    dt = 2.0 / (np.pi ** 2 * sum((a / b) ** 2 for a, b in zip(n, L)))
    g = 0.1 / dt * (2 * np.pi) ** 2
    plan = wdm.Plan(wdm.make_config(n, L=L, four_pi_G=g, precision=prec))
    x = torch.from_numpy(psi).cuda()
    wdm.wdm_set_state(plan.handle, 0, x)
    wdm.wdm_profile(plan.handle, True)
    wdm.wdm_step(plan.handle, 3, dt)
    names = {s["name"] for s in wdm.wdm_profile_read(plan.handle)}
    wdm.wdm_profile(plan.handle, False)
    four = n in FOUR or (n in SINGLE and prec == 0)
    assert ({"xy_kinetic", "xy_green"} <= names) == four, names
    assert ({"x_kinetic", "x_green"} <= names) == (not four), names
    out = torch.empty_like(x)
    wdm.wdm_get_psi(plan.handle, 0, out)
    got = out.cpu().numpy().astype(np.complex128)
    plan.close()
    start = psi.astype(np.complex128)
    ref = orc.kdk(orc.make_config(n, L=L, four_pi_G=g), start, nsteps=3, dt=dt)[0]
    assert rel_l2(ref, start) > 0.1
    assert rel_l2(got, ref) < TOL[prec]


@pytest.mark.gpu
def test_particles_raise_the_tile_rule(wdm):
    n = (192, 32, 128)     # 64 tiles: in complex128 eight passes beside many moving particles
    pos = torch.rand((50_000, 3), generator=torch.Generator().manual_seed(1)).cuda()
    psi = torch.ones(n, dtype=torch.complex128, device="cuda")
    for npart, mode, four in ((50_000, wdm.WDM_BARYON_DYNAMIC, False),
                              (49_999, wdm.WDM_BARYON_DYNAMIC, True),
                              (50_000, wdm.WDM_BARYON_STATIC, True)):
        plan = wdm.Plan(wdm.make_config(n, n_particles=npart, particle_mass=1e-6, precision=1,
                                        baryon_mode=mode))
        wdm.wdm_set_state(plan.handle, 0, psi, pos, torch.zeros_like(pos))
        wdm.wdm_profile(plan.handle, True)
        wdm.wdm_step(plan.handle, 1, 1e-6)
        names = {s["name"] for s in wdm.wdm_profile_read(plan.handle)}
        assert ("xy_kinetic" in names) == four
        plan.close()


@pytest.mark.gpu
def test_members_count_in_the_tile_rule(wdm):
    n = (96, 192, 128)     # 384 tiles a member: in complex128 four passes up to 768
    for members, four in ((2, True), (3, False)):
        plan = wdm.Plan([wdm.make_config(n, precision=1)] * members)
        psi = torch.ones(n, dtype=torch.complex128, device="cuda")
        for k in range(members):
            wdm.wdm_set_state(plan.handle, k, psi)
        wdm.wdm_profile(plan.handle, True)
        wdm.wdm_step(plan.handle, 1, 1e-6)
        names = {s["name"] for s in wdm.wdm_profile_read(plan.handle)}
        assert ("xy_kinetic" in names) == four
        plan.close()
