"""Closing a step: the step count and the stop after an unstable step, through
the C ABI.  A bit raised during a step stops the next one whatever the step's
parity, the launch form (graphs, one launch at a time, a batch) and whether
bodies are present: a run of many steps at once ends where a run checked after
every step ends, with the same state, bit for bit.  And the vertex update's
incidence tables: a capsule with vertices of up to eight neighbours (the wide
table) against the FP64 oracle (1e-12, the repository's bar for short runs)."""
import numpy as np
import pytest
import torch

import synth

pytestmark = pytest.mark.gpu


def _lattice(bodies, precision, first):
    from paper_2207_06043_amd import from_workload
    # an inlet far beyond the stability bound of |u|: the run stops within a few steps
    w = synth.tiny_pipe(precision=precision, with_body=bodies, rigid=False)
    w.domain.inlet_u = np.asarray(w.domain.inlet_u) * 0.0
    lat = from_workload(w, precision=precision, with_bodies=bodies)
    if first:
        lat.step(first)
    return lat


def _hit(lat):
    # a jet at one node drives |u| past the bound two steps later
    f = lat.populations()
    n = 11 + 24 * (5 + 12 * 5)
    f[1, n] += 0.9
    lat.set_populations(f)


@pytest.mark.parametrize("bodies", [False, True])
@pytest.mark.parametrize("precision", ["f64", "f32", "f16s"])
@pytest.mark.parametrize("first", [0, 1])
def test_unstable_stop(bodies, precision, first):
    from paper_2207_06043_amd import Batch
    print(bodies, precision, first, flush=True)
    one = _lattice(bodies, precision, first)
    _hit(one)
    for _ in range(40):
        one.step(1)
        if one.sync(raise_on_stop=False):
            break
    ref = one.info()["steps_done"]
    assert first < ref < first + 40
    runs = []
    for form in ("graph", "eager", "batch"):
        lat = _lattice(bodies, precision, first)
        _hit(lat)
        if form == "batch":
            Batch([lat]).step(40)
        else:
            lat.set_graph(form == "graph")
            lat.step(40)
        assert lat.sync(raise_on_stop=False) == one.sync(raise_on_stop=False) != 0
        assert lat.info()["steps_done"] == ref
        lat.step(3)
        assert lat.info()["steps_done"] == ref
        runs.append(lat.populations())
    for f in runs:
        assert torch.equal(torch.nan_to_num(f), torch.nan_to_num(one.populations()))


@pytest.mark.parametrize("sides", [5, 7, 8])
def test_vertex_valence(sides):
    import oracle
    from paper_2207_06043_amd import from_workload
    # a bipyramid over a regular polygon: apexes with `sides` neighbours
    a = 2 * np.pi * np.arange(sides) / sides + 0.3
    X = np.vstack([np.stack([np.cos(a), np.sin(a), 0 * a], 1), [[0, 0, 0.9], [0, 0, -0.9]]]) * 2.6 + (8.23, 5.71, 5.37)
    k = np.arange(sides)
    up = np.stack([k, (k + 1) % sides, np.full(sides, sides)], 1)
    dn = np.stack([(k + 1) % sides, k, np.full(sides, sides + 1)], 1)
    b = synth.Body(X, np.vstack([up, dn]).astype(np.int32), ca=5.0, eb=1e-3, rho_ratio=1.1, r_ref=2.6, u_ref=0.05)
    d = synth.periodic_box(17, 12, 11, body_force=(1e-4, 2e-5, 0.0))
    w = synth.Workload("bipyramid", d, [b], 0.8, 0.05, "f64", 12)
    orc = oracle.from_workload(w)
    assert orc.step(12) == 0
    lat = from_workload(w)
    lat.step(12)
    lat.sync()
    x, xo = lat.body(0)[0].cpu().numpy(), orc.body(0)[0]
    assert np.abs(x - xo).max() <= 1e-12 * np.abs(xo).max()
