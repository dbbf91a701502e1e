"""The eight-pass step on its default plans where the four-pass form exists: it
can be chosen, read back, cached and left again, and a state survives the change.

Tolerances as in the four-pass parity test: 5e-6 in single precision, 1e-13 in
double for a few steps.
"""
import json

import numpy as np
import pytest

torch = pytest.importorskip("torch")

TOL = {0: 5e-6, 1: 1e-13}


class FakePlan:
    """The tuning calls of a plan of two size classes."""

    def __init__(self, monkeypatch, w, tuned=None):
        self.table, self.forms = [0] * 12, [0, 0]

        def set_tuning(_, t):
            self.table, self.forms = list(t), [0, 0]

        monkeypatch.setattr(w, "wdm_tuning_entries", lambda _: 12)
        monkeypatch.setattr(w, "wdm_set_tuning", set_tuning)
        monkeypatch.setattr(w, "wdm_get_tuning", lambda _: list(self.table))
        monkeypatch.setattr(w, "wdm_set_step_form", lambda _, f: setattr(self, "forms", list(f)))
        monkeypatch.setattr(w, "wdm_get_step_form", lambda _: list(self.forms))
        monkeypatch.setattr(w, "wdm_autotune", lambda _, reps: setattr(self, "forms", list(tuned)))


def test_cache_keeps_the_form(monkeypatch, tmp_path):
    from paper_2606_25026_amd import wdm as w

    cfgs = [w.make_config(64), w.make_config(32)]
    cache = tmp_path / "tune.json"
    FakePlan(monkeypatch, w, tuned=[0, 1])
    assert w.autotune(None, cfgs, cache=str(cache)) == [0] * 12
    again = FakePlan(monkeypatch, w)
    w.autotune(None, cfgs, cache=str(cache))
    assert again.forms == [0, 1]
    # a cache that names no forms (the tables alone) means the default ones
    store = json.loads(cache.read_text())
    cache.write_text(json.dumps({w.tuning_key(cfgs): store[w.tuning_key(cfgs)]}))
    again.forms = [1, 1]
    w.autotune(None, cfgs, cache=str(cache))
    assert again.forms == [0, 0]


def names_of_step(wdm, plan, dt):
    wdm.wdm_profile(plan.handle, True)
    wdm.wdm_step(plan.handle, 1, dt)
    names = {s["name"] for s in wdm.wdm_profile_read(plan.handle)}
    wdm.wdm_profile(plan.handle, False)
    return names


@pytest.mark.gpu
@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("n", [(32, 16, 32), (64, 96, 32), (96, 128, 64), (32, 192, 96)],
                         ids=lambda n: "x".join(map(str, n)))
def test_eight_default_passes(wdm, orc, n, prec):
    rng = np.random.default_rng(5)
    psi = (rng.standard_normal(n) + 1j * rng.standard_normal(n)).astype(
        np.complex128 if prec else np.complex64)
    dt = 1e-4
    g = 0.1 / dt * (2 * np.pi) ** 2
    plan = wdm.Plan(wdm.make_config(n, four_pi_G=g, precision=prec))
    x = torch.from_numpy(psi).cuda()
    wdm.wdm_set_state(plan.handle, 0, x)
    for form in (0, 1, 1, 0):
        wdm.wdm_set_step_form(plan.handle, [form])
        assert wdm.wdm_get_step_form(plan.handle) == [form]
        assert wdm.wdm_get_tuning(plan.handle) == [0] * 6
        names = names_of_step(wdm, plan, dt)
        assert ("x_kinetic" in names) == bool(form) and ("xy_kinetic" in names) == (not form)
    for bad in ([2], [-1], [0, 0], []):
        with pytest.raises(wdm.WdmError):
            wdm.wdm_set_step_form(plan.handle, bad)
    # the table's own meaning stays: all 0 is the default form again
    wdm.wdm_set_step_form(plan.handle, [1])
    wdm.wdm_set_tuning(plan.handle, [0] * 6)
    assert wdm.wdm_get_step_form(plan.handle) == [0]
    assert "xy_kinetic" in names_of_step(wdm, plan, dt)
    out = torch.empty_like(x)
    wdm.wdm_get_psi(plan.handle, 0, out)
    got = out.cpu().numpy().astype(np.complex128)
    ref = orc.kdk(orc.make_config(n, four_pi_G=g), psi.astype(np.complex128), nsteps=5, dt=dt)[0]
    assert np.linalg.norm(got - ref) < 2 * TOL[prec] * np.linalg.norm(ref)
    plan.close()


@pytest.mark.gpu
def test_autotune_resets_the_form(wdm):
    """The tuner times both forms and leaves a table and a form that agree."""
    plan = wdm.Plan([wdm.make_config(96), wdm.make_config((32, 384, 32))])
    wdm.wdm_set_step_form(plan.handle, [1, 1])
    wdm.wdm_autotune(plan.handle, 3)
    table, forms = wdm.wdm_get_tuning(plan.handle), wdm.wdm_get_step_form(plan.handle)
    assert forms[0] == 0              # no four-pass form: nothing to choose
    assert forms[1] in (0, 1)
    plan.close()
    wdm_again = wdm.Plan([wdm.make_config(96), wdm.make_config((32, 384, 32))])
    wdm.wdm_set_tuning(wdm_again.handle, table)
    wdm.wdm_set_step_form(wdm_again.handle, forms)
    assert wdm.wdm_get_tuning(wdm_again.handle) == table
    assert wdm.wdm_get_step_form(wdm_again.handle) == forms
    wdm_again.close()
