"""The particle deposit's per-run sums: runs of equal cells of every length up to
several wavefronts, starting anywhere in a wavefront and crossing its 16-lane
rows, in compact boxes (summed in LDS) and in boxes too large for it, against
numpy's CIC in 64 bits.

Tolerance: a node sums at most 2000 positive float32 terms in some order, so it
is off by less than 2000 * 2^-24 of itself; in fixed point by one rounding.
"""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

N = 64


def cic(pos, q):
    s = pos.astype(np.float64) * N
    i = np.floor(s).astype(int)
    f = s - i
    rho = np.zeros((N, N, N))
    for a in (0, 1):
        for b in (0, 1):
            for c in (0, 1):
                w = (np.abs(1 - a - f[:, 0]) * np.abs(1 - b - f[:, 1]) * np.abs(1 - c - f[:, 2]))
                np.add.at(rho, tuple((i + [a, b, c]).T % N), q * w)
    return rho


def particles(kind, rng):
    counts = [1, 2, 3, 5, 8, 15, 16, 17, 1, 31, 32, 33, 47, 1, 1, 63, 64, 65, 9, 130, 257, 600, 4]
    cells = []
    for k, n in enumerate(counts):
        # compact: neighbouring cells; spread: cells all over the box, its faces too
        c = (20 + k % 3, 21 + (k // 3) % 3, 22 + k // 9) if kind == "compact" else \
            tuple(rng.integers(0, N, 3)) if k % 4 else (N - 1, k % N, N - 1)
        cells += [c] * n
    pos = (np.array(cells) + rng.uniform(0.02, 0.98, (len(cells), 3))) / N
    return pos[rng.permutation(len(pos))].astype(np.float32)


@pytest.mark.parametrize("kind", ["compact", "spread"])
@pytest.mark.parametrize("prec,det", [(0, 0), (1, 0), (0, 1)])
def test_deposit_of_runs_matches_cic(wdm, kind, prec, det):
    rng = np.random.default_rng(5)
    pos = particles(kind, rng)
    mass = 1e-3
    plan = wdm.Plan(wdm.make_config(N, n_particles=len(pos), particle_mass=mass, precision=prec,
                                    flags=wdm.WDM_DETERMINISTIC_DEPOSIT if det else 0))
    psi = torch.zeros((N,) * 3, dtype=torch.complex128 if prec else torch.complex64, device="cuda")
    p = torch.from_numpy(pos).cuda()
    wdm.wdm_set_state(plan.handle, 0, psi, p, torch.zeros_like(p))
    rho = torch.empty((N,) * 3, dtype=torch.float64 if prec else torch.float32, device="cuda")
    ref = cic(pos, mass * N ** 3)
    tol = 2000 * 2.0 ** -24 if prec == 0 else 2000 * 2.0 ** -53 + 1e-12
    for _ in range(2):    # the second call meets the LDS box the first one left
        wdm.wdm_density(plan.handle, 0, rho)
        got = rho.cpu().numpy().astype(np.float64)
        assert np.max(np.abs(got - ref)) <= tol * ref.max()
    plan.close()
