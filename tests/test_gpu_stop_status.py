"""The status of a run whose last step became unstable and left positions that
the damage check would refuse as well, through the C ABI: it is that of the
step, unstable, whether or not another step was enqueued after it, in every
launch form, at either parity, and after a checkpoint.  The capsule starts
with vertex velocities so large that the first forcing leaves the fixed-point
range, and that the first update stretches its edges far beyond twice their
length."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu

UNSTABLE = 4


def _lattice(first):
    from paper_2207_06043_amd import from_workload
    w = synth.tiny_pipe(with_body=True, rigid=False)
    b = w.bodies[0]
    b.v0 = -40.0 * (b.x - b.x.mean(axis=0))
    lat = from_workload(w, precision="f64", with_bodies=False)
    lat.step(first)
    lat.add_body(b)
    return lat, b


def _stretch(lat, b):
    e = np.unique(np.sort(np.vstack([b.faces[:, [0, 1]], b.faces[:, [1, 2]], b.faces[:, [2, 0]]]), axis=1), axis=0)
    x = lat.body(0)[0].cpu().numpy()
    return (np.linalg.norm(x[e[:, 0]] - x[e[:, 1]], axis=1) / np.linalg.norm(b.x[e[:, 0]] - b.x[e[:, 1]], axis=1)).max()


@pytest.mark.parametrize("form", ["graph", "eager", "batch"])
@pytest.mark.parametrize("first", [0, 1])
@pytest.mark.parametrize("steps", [1, 2, 5])
def test_status_of_an_unstable_last_step(steps, first, form, tmp_path):
    from paper_2207_06043_amd import Batch
    print(steps, first, form, flush=True)
    lat, b = _lattice(first)
    if form == "batch":
        Batch([lat]).step(steps)
    else:
        lat.set_graph(form == "graph")
        lat.step(steps)
    assert lat.sync(raise_on_stop=False) == UNSTABLE
    assert lat.info()["steps_done"] == first + 1
    assert _stretch(lat, b) > 2.0
    lat.diagnostics()
    assert lat.sync(raise_on_stop=False) == UNSTABLE
    lat.save(tmp_path / "c")
    other, _ = _lattice(first)
    other.load(tmp_path / "c")
    other.step(2)
    assert other.sync(raise_on_stop=False) == UNSTABLE
    assert other.info()["steps_done"] == first + 1
