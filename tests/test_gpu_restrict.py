"""Restriction to a coarser grid, every ratio of sides that cuts the pencils
differently, against numpy in 64 bits; the result at an address that is no
multiple of an element.

Tolerance: two transforms' rounding, 4 log2(N) ulps of the field's norm each.
"""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def restricted(psi, nc):
    nf = psi.shape[0]
    m = np.concatenate([np.arange(nc // 2), [0], np.arange(-nc // 2 + 1, 0)])
    f = np.fft.fftn(psi)[np.ix_(m % nf, m % nf, m % nf)] * (nc / nf) ** 3
    for a in range(3):
        f[(slice(None),) * a + (nc // 2,)] = 0
    return np.fft.ifftn(f)


@pytest.mark.parametrize("nf,nc,prec", [(32, 16, 0), (96, 16, 0), (96, 64, 1), (128, 96, 0),
                                        (128, 64, 1), (192, 128, 0), (256, 192, 0)])
def test_restriction_matches_numpy(wdm, nf, nc, prec):
    rng = np.random.default_rng(nf + nc)
    dtype = np.complex128 if prec else np.complex64
    psi = (rng.standard_normal((nf,) * 3) + 1j * rng.standard_normal((nf,) * 3)).astype(dtype)
    fine, coarse = (wdm.Plan(wdm.make_config(n, precision=prec)) for n in (nf, nc))
    wdm.wdm_set_state(fine.handle, 0, torch.from_numpy(psi).cuda())
    ref = restricted(psi.astype(np.complex128), nc)
    tol = 8 * np.log2(nf ** 3) * (2.0 ** -52 if prec else 2.0 ** -23)
    words = torch.zeros(2 * nc ** 3 + 2, dtype=torch.float64 if prec else torch.float32,
                        device="cuda")
    for shift in (0, 1):
        words.zero_()
        wdm.wdm_restrict(fine.handle, 0, coarse.handle, 0, words[shift:])
        out = words.cpu().numpy()
        assert (out[:shift] == 0).all() and (out[shift + 2 * nc ** 3:] == 0).all()
        got = out[shift:shift + 2 * nc ** 3].astype(np.float64).view(np.complex128)
        assert np.linalg.norm(got - ref.ravel()) <= tol * np.linalg.norm(ref)


def test_members_of_one_plan(wdm):
    rng = np.random.default_rng(1)
    psi = (rng.standard_normal((64,) * 3) + 1j * rng.standard_normal((64,) * 3)).astype(np.complex64)
    plan = wdm.Plan([wdm.make_config(64), wdm.make_config(32)])
    wdm.wdm_set_state(plan.handle, 0, torch.from_numpy(psi).cuda())
    out = torch.empty((32,) * 3, dtype=torch.complex64, device="cuda")
    wdm.wdm_restrict(plan.handle, 0, plan.handle, 1, out)
    ref = restricted(psi.astype(np.complex128), 32)
    tol = 8 * np.log2(64 ** 3) * 2.0 ** -23
    assert np.linalg.norm(out.cpu().numpy() - ref) <= tol * np.linalg.norm(ref)
