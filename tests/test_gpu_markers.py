"""Forcing markers and probes where their launches branch, through the C ABI
against the FP64 oracle: supports at wall nodes with one batch of links and
more (a sphere close to the wall of a narrow pipe), supports at the inlet and
outlet nodes, a chunk whose box exceeds the on-chip capacity (a coarse mesh:
every marker takes the direct path), and a periodic axis of two nodes.

Bounds: the repository's FP64 bar 1e-12, for the force field relative to its
largest value, for positions to the largest coordinate; FP32 2e-5 on the force."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu

U = 0.03


def _body(subdiv, r, c, **kw):
    X, F = synth.icosphere(subdiv, r, c, tilt=True)
    return synth.Body(X, F, rigid=kw.pop("rigid", True), ca=0.5, eb=1e-3, rho_ratio=1.1, r_ref=r, u_ref=U, **kw)


def _workload(name):
    if name in ("wall", "inlet", "outlet"):
        d = synth.pipe(20, 11, 11, 4.6, u_max=U, tau=0.8, init="poiseuille")
        c = {"wall": (9.8, 5.9, 5.2), "inlet": (3.3, 5.1, 4.9), "outlet": (16.2, 5.1, 4.9)}[name]
        bodies = [_body(1, 2.0, c)]
    elif name == "direct":
        d = synth.periodic_box(26, 24, 23, body_force=(1e-4, 0.0, 2e-5))
        bodies = [_body(0, 8.0, (12.3, 11.6, 10.9))]
    else:  # "two"
        d = synth.periodic_box(14, 12, 2, body_force=(1e-4, 0.0, 0.0))
        bodies = [_body(1, 2.2, (6.3, 5.6, 0.8))]
    return synth.Workload(name, d, bodies, 0.8, U, "f64", 6)


@pytest.mark.parametrize("precision", ["f64", "f32"])
@pytest.mark.parametrize("name", ["wall", "inlet", "outlet", "direct", "two"])
def test_markers(name, precision):
    import oracle
    from paper_2207_06043_amd import from_workload
    w = _workload(name)
    orc = oracle.from_workload(w)
    lat = from_workload(w, precision=precision)
    bar = 1e-12 if precision == "f64" else 2e-5
    print(name, precision, flush=True)
    for steps in (1, 5):
        assert orc.step(steps) == 0
        lat.step(steps)
        lat.sync()
        f, fo = lat.force().cpu().numpy().ravel(), np.asarray(orc.force()).ravel()
        assert np.abs(f - fo).max() <= bar * np.abs(fo).max()
        for k in range(len(w.bodies)):
            x, xo = lat.body(k)[0].cpu().numpy(), orc.body(k)[0]
            assert np.abs(x - xo).max() <= bar * np.abs(xo).max()
    assert np.abs(fo).max() > 0  # (a fluid at rest has no force in its first step)
    assert lat.info()["mls_singular"] == orc.mls_singular
