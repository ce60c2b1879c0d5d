"""A mesh whose faces lie more than 2^31 lattice spacings apart, far outside the
box: its markers have no supports, so the fluid, and the adjoint of the fluid,
are those of a lattice without it.  (The box of a block's supports, which is
formed in 32 bits, must not pass for a small one.)"""
import numpy as np
import pytest
import torch

import synth

pytestmark = pytest.mark.gpu

TAU, U = 0.8, 0.03


def _workload(axis, fixed, precision):
    d = synth.pipe(20, 11, 11, 4.6, u_max=U, tau=TAU, init="poiseuille")
    X, F = synth.icosphere(1, 2.0, (0.0, 0.0, 0.0), tilt=True)
    X = X.copy()
    X[:, axis] *= 1e9  # within the range of a 32-bit integer, on both sides
    b = synth.Body(X, F, rigid=fixed, fixed=fixed, ca=0.5, eb=1e-3, rho_ratio=1.1, r_ref=2.0, u_ref=U)
    return synth.Workload("far", d, [b], TAU, U, precision, 4)


@pytest.mark.parametrize("two_pass", [False, True])
@pytest.mark.parametrize("precision", ["f64", "f32"])
@pytest.mark.parametrize("axis", [0, 1, 2])
def test_far_markers_leave_the_fluid_alone(axis, precision, two_pass, monkeypatch):
    from paper_2207_06043_amd import from_workload
    print(axis, precision, two_pass, flush=True)
    monkeypatch.setenv("LBM_SPREAD_TWO_PASS", "1" if two_pass else "0")
    w = _workload(axis, True, precision)
    c = w.bodies[0].x[w.bodies[0].faces].mean(axis=1)[:, axis]
    assert c.max() - c.min() > 2.0**31 and np.abs(c).max() < 2.0**31
    lat, free = from_workload(w), from_workload(w, with_bodies=False)
    for s in (lat, free):
        s.step(4)
        s.sync()
    assert torch.equal(lat.populations(), free.populations())
    assert not lat.force().any()
    assert np.array_equal(lat.body(0)[0].cpu().numpy(), w.bodies[0].x)


@pytest.mark.parametrize("axis", [0, 2])
def test_far_markers_leave_the_adjoint_alone(axis):
    from paper_2207_06043_amd import from_workload
    print(axis, flush=True)
    w = _workload(axis, False, "f64")
    lat, free = from_workload(w), from_workload(w, with_bodies=False)
    rng = np.random.default_rng(3)
    lam = torch.from_numpy(rng.normal(size=(19, w.domain.n_nodes)))
    g, grad, _, _ = lat.adjoint_run(3, lam, checkpoint_every=2)
    gf, gradf = free.adjoint(3, lam, checkpoint_every=2)
    assert (g - gf).abs().max() <= 1e-12 * gf.abs().max()
    assert (grad[:5] - gradf).abs().max() <= 1e-12 * gradf.abs().max()
