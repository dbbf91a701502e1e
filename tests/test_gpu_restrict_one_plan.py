"""Restriction between two members of one plan, which share their scratch, into
an address that is and one that is no multiple of an element, against numpy in 64
bits; nothing around the result is written.

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


@pytest.mark.parametrize("shift", [0, 4, 8])
@pytest.mark.parametrize("nf,nc,prec", [(64, 32, 0), (96, 64, 0), (96, 16, 1), (128, 96, 1)])
def test_addresses(wdm, nf, nc, prec, shift):
    rng = np.random.default_rng(nf + nc)
    dtype = np.complex128 if prec else np.complex64
    psi = (rng.standard_normal((nf,) * 3) + 1j * rng.standard_normal((nf,) * 3)).astype(dtype)
    plan = wdm.Plan([wdm.make_config(n, precision=prec) for n in (nf, nc)])
    wdm.wdm_set_state(plan.handle, 0, torch.from_numpy(psi).cuda())
    size = nc ** 3 * psi.itemsize
    room = torch.full((size + 64,), 7, dtype=torch.uint8, device="cuda")
    wdm.wdm_restrict(plan.handle, 0, plan.handle, 1, room[shift:])
    out = room.cpu().numpy()
    assert (out[:shift] == 7).all() and (out[shift + size:] == 7).all()
    got = out[shift:shift + size].copy().view(dtype).astype(np.complex128)
    ref = restricted(psi.astype(np.complex128), nc).ravel()
    tol = 8 * np.log2(nf ** 3) * (2.0 ** -52 if prec else 2.0 ** -23)
    assert np.linalg.norm(got - ref) <= tol * np.linalg.norm(ref)
    plan.close()
