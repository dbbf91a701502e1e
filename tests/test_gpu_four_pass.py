"""The four-pass step (the y transform divided between the z and the plane
passes) against the FP64 oracle: every factor pair of the y axis with every x
plan and z length at small sizes, ragged boxes and boxes it is not built for,
and the half spectrum's change of form when another FFT plan is chosen.

Tolerances: a transform of N points in single precision is off by about
eps log2 N = 6e-8 * 20, of which a step has four, so three steps stay below
5e-6 (the unit round-off errors do not all add up: 1e-6 is seen at 128^3);
in double precision the same count gives 1e-14.
"""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

TOL = {0: 5e-6, 1: 1e-13}


def rel_l2(a, b):
    return float(np.linalg.norm((a - b).ravel()) / np.linalg.norm(b.ravel()))


def field(n, seed):
    rng = np.random.default_rng(seed)
    return rng.standard_normal(n) + 1j * rng.standard_normal(n)


def oracle_run(orc, n, L, psi, steps, dt, g):
    cfg = orc.make_config(n, L=L, four_pi_G=g)
    return orc.kdk(cfg, psi, nsteps=steps, dt=dt)[0]


def gpu_state(wdm, plan, prec, psi):
    x = torch.from_numpy(psi).to(torch.complex64 if prec == 0 else torch.complex128).cuda()
    wdm.wdm_set_state(plan.handle, 0, x)
    return x


def gpu_psi(wdm, plan, like):
    out = torch.empty_like(like)
    wdm.wdm_get_psi(plan.handle, 0, out)
    torch.cuda.synchronize()
    return out.cpu().numpy().astype(np.complex128)


# (nx, ny, nz): ny = R1 R2 with R2 = 4 (16, 32), 8 (64, 96, 128), 16 (192, 256);
# every x plan of each R2; every z length with every R1; (16, 256, 16) and
# (32, 96, 16) have no four-pass form, (16, 16, 256) no z pass at R1 = 4
SHAPES = [(16, 16, 16), (64, 16, 32), (96, 32, 16), (32, 32, 128), (128, 16, 64), (192, 32, 32),
          (256, 32, 16), (16, 64, 192), (32, 96, 32), (64, 128, 64), (96, 64, 96), (128, 64, 16),
          (192, 96, 64), (256, 64, 32), (16, 192, 96), (32, 256, 32), (64, 192, 128),
          (96, 256, 32), (128, 256, 32), (192, 192, 32), (256, 256, 32), (16, 128, 256),
          (16, 256, 16), (32, 96, 16), (16, 16, 256)]


@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("n", SHAPES, ids=lambda n: "x".join(map(str, n)))
def test_steps_match_oracle(wdm, orc, n, prec):
    L = (1.0, 0.75, 1.25)
    psi = field(n, n[0] + n[1] + n[2])
    # both factors matter: the drift turns the fastest mode by about a radian a
    # step, the potential's kick by about 0.1
    dt, g, steps = 1.0 / (np.pi ** 2 * sum((a / b) ** 2 for a, b in zip(n, L))) * 2.0, 0.0, 3
    k2 = (2 * np.pi) ** 2
    g = 0.1 / dt * k2
    plan = wdm.Plan(wdm.make_config(n, L=L, four_pi_G=g, precision=prec))
    x = gpu_state(wdm, plan, prec, psi)
    start = x.cpu().numpy().astype(np.complex128)
    wdm.wdm_step(plan.handle, steps, dt)
    got = gpu_psi(wdm, plan, x)
    ref = oracle_run(orc, n, L, start, steps, dt, g)
    assert rel_l2(ref, start) > 0.1
    err = rel_l2(got, ref)
    print(f"{n} prec={prec}: rel L2 {err:.2e}")
    assert err < TOL[prec]
    plan.close()


@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("n", [(32, 16, 32), (32, 64, 32), (32, 96, 32), (32, 128, 64)])
def test_plan_change_between_calls_keeps_the_potential(wdm, orc, n, prec):
    """The half spectrum a call leaves is read by the next one: choosing another
    FFT plan in between (eight passes) and going back continues the run."""
    L = (1.0, 1.0, 1.0)
    psi = field(n, 7)
    dt = 1e-4
    g = 0.1 / dt * (2 * np.pi) ** 2
    plan = wdm.Plan(wdm.make_config(n, L=L, four_pi_G=g, precision=prec))
    x = gpu_state(wdm, plan, prec, psi)
    start = x.cpu().numpy().astype(np.complex128)
    other = [0, 0, 1, 0, 0, 0]    # P3's second plan: nx = 32 has one
    for table in ([0] * 6, other, other, [0] * 6):
        wdm.wdm_set_tuning(plan.handle, table)
        wdm.wdm_step(plan.handle, 1, dt)
    got = gpu_psi(wdm, plan, x)
    ref = oracle_run(orc, n, L, start, 4, dt, g)
    assert rel_l2(got, ref) < TOL[prec] * 2
    plan.close()
