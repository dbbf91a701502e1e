"""Diagnostics, mass radii, shell power and energies at grids whose sides cut the
kernels' tiles, fold or do not fold their octants, against numpy in 64 bits.

Tolerances: the FP64 sums of the same FP64 terms differ by their order only
(1e-12 of the sum of magnitudes); the spectrum and the kinetic energy carry the
transform's rounding, below 4 log2(N) ulps of a mode's power.
"""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

GRIDS = [(16, 16, 16), (32, 16, 96), (16, 96, 32), (96, 96, 96), (64, 128, 192)]


def state(wdm, n, prec, seed=3):
    rng = np.random.default_rng(seed)
    h = 1.0 / max(n)
    plan = wdm.Plan(wdm.make_config(n, L=tuple(a * h for a in n), precision=prec))
    psi = (rng.standard_normal(n) + 1j * rng.standard_normal(n)) * (1.0 + rng.random(n))
    psi = psi.astype(np.complex128 if prec else np.complex64)
    dev = torch.from_numpy(psi).cuda()
    wdm.wdm_set_state(plan.handle, 0, dev)
    return plan, psi.astype(np.complex128), h


def squared_distance(n, centre):
    d = [np.minimum((np.arange(a) - c) % a, (c - np.arange(a)) % a) ** 2
         for a, c in zip(n, centre)]
    return d[0][:, None, None] + d[1][None, :, None] + d[2][None, None, :]


@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("n", GRIDS)
def test_diagnostics_and_radii(wdm, n, prec):
    plan, psi, h = state(wdm, n, prec)
    phi = torch.empty(n, dtype=torch.float64 if prec else torch.float32, device="cuda")
    wdm.wdm_potential(plan.handle, 0, phi)
    phi = phi.cpu().numpy().astype(np.float64)
    rho = psi.real ** 2 + psi.imag ** 2
    j2, q, mom = 0.0, 0.0, []
    for a in range(3):
        g = (np.roll(psi, -1, a) - np.roll(psi, 1, a)) / (2 * h)
        ja = (psi.conj() * g).imag    # hbar/m = 1
        s = (np.roll(np.abs(psi), -1, a) - np.roll(np.abs(psi), 1, a)) / (2 * h)
        j2, q = j2 + ja * ja, q + s * s
        mom.append((ja.sum(), np.abs(ja).sum()))
    dv = h ** 3
    for centre in (None, (0, n[1] - 1, n[2] // 2 - 1)):
        d = wdm.wdm_diagnostics(plan.handle, 0, centre)
        assert d["K"] == pytest.approx((0.5 * j2 / rho).sum() * dv, rel=1e-10)
        assert d["Q"] == pytest.approx(q.sum() * dv, rel=1e-10)
        assert d["mass"] == pytest.approx(rho.sum() * dv, rel=1e-12)
        assert abs(d["V"] - (rho * phi).sum() * dv) <= 1e-12 * (rho * np.abs(phi)).sum() * dv
        for got, (want, scale) in zip(d["momentum"], mom):
            assert abs(got - want * dv) <= 1e-12 * scale * dv
        c = centre or tuple(a // 2 for a in n)
        r2 = squared_distance(n, c)
        mass = np.bincount(r2.ravel(), weights=rho.ravel())
        cum = np.cumsum(mass)
        want = [h * np.sqrt(np.flatnonzero((cum >= 0.1 * f * cum[-1]) & (mass > 0))[0])
                for f in range(1, 10)]
        assert np.allclose(d["radii"], want, rtol=1e-14, atol=0)


def test_radii_of_no_mass(wdm):
    plan = wdm.Plan(wdm.make_config(16))
    psi = torch.zeros((16,) * 3, dtype=torch.complex64, device="cuda")
    wdm.wdm_set_state(plan.handle, 0, psi)
    assert list(wdm.wdm_diagnostics(plan.handle, 0)["radii"]) == [-1.0] * 9


@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("n,nbins", [(16, 1), (16, 14), (64, 32), (96, 96), (128, 1024)])
def test_shell_power(wdm, n, nbins, prec):
    plan, psi, _ = state(wdm, (n,) * 3, prec)
    pk, counts = wdm.wdm_power_spectrum(plan.handle, 0, nbins)
    rho = psi.real ** 2 + psi.imag ** 2
    p = np.abs(np.fft.fftn(rho / rho.mean() - 1.0)) ** 2 / float(n) ** 6
    m = np.fft.fftfreq(n, 1.0 / n)
    k = np.rint(np.sqrt(m[:, None, None] ** 2 + m[None, :, None] ** 2 + m[None, None, :] ** 2))
    k = k.astype(int).ravel()
    cnt = np.bincount(k, minlength=nbins)[:nbins]
    ref = np.bincount(k, weights=p.ravel(), minlength=nbins)[:nbins]
    assert np.array_equal(counts, cnt)
    ulp = 2.0 ** -52 if prec else 2.0 ** -23
    lg = np.log2(float(n) ** 3)
    for b in range(1, nbins):    # the mean of the contrast is rounding alone
        if cnt[b]:
            assert abs(pk[b] * cnt[b] - ref[b]) <= 4 * lg * ulp * ref[b]
        else:
            assert pk[b] == 0.0


@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("n", GRIDS)
def test_energies(wdm, n, prec):
    plan, psi, h = state(wdm, n, prec)
    e = wdm.wdm_energy(plan.handle, 0)
    phi = torch.empty(n, dtype=torch.float64 if prec else torch.float32, device="cuda")
    wdm.wdm_potential(plan.handle, 0, phi)
    phi = phi.cpu().numpy().astype(np.float64)
    rho = psi.real ** 2 + psi.imag ** 2
    dv = h ** 3
    assert e["mass"] == pytest.approx(rho.sum() * dv, rel=1e-12)
    assert e["max_rho"] == pytest.approx(rho.max(), rel=1e-15)
    assert e["max_abs_phi"] == np.abs(phi).max()
    assert abs(e["e_pot"] - 0.5 * (rho * phi).sum() * dv) <= 1e-12 * (rho * np.abs(phi)).sum() * dv
    k2 = sum(np.meshgrid(*[(2 * np.pi / h * np.fft.fftfreq(a)) ** 2 for a in n], indexing="ij"))
    ref = 0.5 * (k2 * np.abs(np.fft.fftn(psi)) ** 2).sum() * dv / psi.size
    ulp = 2.0 ** -52 if prec else 2.0 ** -23
    assert e["e_kin"] == pytest.approx(ref, rel=4 * np.log2(psi.size) * ulp)
