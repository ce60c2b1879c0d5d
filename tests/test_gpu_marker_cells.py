"""The cells that a chunk of forcing markers computes, through the C ABI against
the FP64 oracle: a box of at most 256 cells (all of them), larger boxes (a list
of the cells that some marker uses), the largest that fit on chip and one that
does not, in a periodic box and across its faces.

Bounds: the repository's FP64 bar 1e-12, for the force field relative to its
largest value, for positions to the largest coordinate; FP32 2e-5 on the force."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu

U = 0.03


@pytest.mark.parametrize("precision", ["f64", "f32"])
@pytest.mark.parametrize("r,c", [(1.4, (9.8, 9.9, 9.2)), (2.6, (10.3, 9.1, 9.9)), (4.2, (10.1, 10.4, 9.7)),
                                 (4.9, (10.0, 10.2, 10.1)), (3.1, (0.4, 18.7, 10.2))])
def test_box_sizes(r, c, precision):
    import oracle
    from paper_2207_06043_amd import from_workload
    X, F = synth.icosphere(1, r, c, tilt=True)
    b = synth.Body(X, F, rigid=True, ca=0.5, eb=1e-3, rho_ratio=1.1, r_ref=r, u_ref=U)
    w = synth.Workload("cells", synth.periodic_box(22, 20, 21, body_force=(1e-4, 0.0, 2e-5)), [b], 0.8, U, "f64", 4)
    orc = oracle.from_workload(w)
    lat = from_workload(w, precision=precision)
    bar = 1e-12 if precision == "f64" else 2e-5
    print(r, precision, flush=True)
    assert orc.step(4) == 0
    lat.step(4)
    lat.sync()
    f, fo = lat.force().cpu().numpy().ravel(), np.asarray(orc.force()).ravel()
    assert np.abs(f - fo).max() <= bar * np.abs(fo).max() and np.abs(fo).max() > 0
    x, xo = lat.body(0)[0].cpu().numpy(), orc.body(0)[0]
    assert np.abs(x - xo).max() <= bar * np.abs(xo).max()
