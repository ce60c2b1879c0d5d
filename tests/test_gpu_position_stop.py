"""A stop raised by a step's position check, which runs in the same launch as
the forcing of that step: whatever the other blocks of the launch have done,
the run ends with the state of the last completed step, bit for bit.  Two large
capsules give the launch some two hundred blocks beside the small one that its
first update damages; the reference is a run of that one step."""
import numpy as np
import pytest
import torch

import synth

pytestmark = pytest.mark.gpu

DAMAGED = 5


def _workload(precision):
    d = synth.pipe(52, 34, 34, 15.2, u_max=0.0, tau=0.8, init="rest", body_force=(1e-5, 0.0, 0.0))
    c = np.array([4.2, 16.3, 16.6])
    X, F = synth.icosphere(1, 0.5, tuple(c), tilt=True)
    bodies = [synth.Body(X, F, rigid=False, ca=0.05, r_ref=0.5, u_ref=0.02, v0=-2.4 * (X - c))]
    for cx in (16.3, 36.1):
        X, F = synth.icosphere(4, 8.0, (cx, 16.7, 16.2), tilt=True)
        bodies.append(synth.Body(X, F, rigid=False, ca=0.05, eb=1e-4, rho_ratio=1.1, r_ref=8.0, u_ref=0.02))
    return synth.Workload("damage", d, bodies, 0.8, 0.02, precision, 4)


def _state(lat):
    out = [lat.populations(), *lat.fields(), lat.force()]
    for b in range(len(lat.bodies)):
        out += list(lat.body(b))
    return out


@pytest.mark.parametrize("form", ["graph", "eager", "batch", "two passes"])
@pytest.mark.parametrize("precision", ["f64", "f32", "f16s"])
def test_the_state_of_the_last_completed_step_survives(precision, form, monkeypatch):
    from paper_2207_06043_amd import Batch, from_workload
    print(precision, form, flush=True)
    if form == "two passes":
        monkeypatch.setenv("LBM_SPREAD_TWO_PASS", "1")
    w = _workload(precision)
    one = from_workload(w)
    one.step(1)
    ref = _state(one)
    lat = from_workload(w)
    if form == "batch":
        Batch([lat]).step(20)
    else:
        lat.set_graph(form != "eager")
        lat.step(20)
    assert lat.sync(raise_on_stop=False) == DAMAGED
    assert lat.info()["steps_done"] == 1
    for a, b in zip(_state(lat), ref):
        assert torch.equal(a, b)
    lat.step(3)
    assert lat.sync(raise_on_stop=False) == DAMAGED
    assert lat.info()["steps_done"] == 1
