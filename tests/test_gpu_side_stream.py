"""A lattice on a stream of its own that does not wait for the default stream:
what the library clears when a body is added, or at the first spread, is
cleared in that stream's order.  The capsule's probes and markers reach solid
nodes, which the fits tell by a mark in the macroscopic field, written right
after that field is cleared; the lattice is large, so that the clear takes
time.  Bit for bit the results on the default stream, and the spread's."""
import numpy as np
import pytest
import torch

import synth

pytestmark = pytest.mark.gpu


def _run(stream, precision):
    from paper_2207_06043_amd import Lattice
    d = synth.pipe(512, 64, 64, 30.2, u_max=0.02, tau=0.8, init="poiseuille")
    X, F = synth.icosphere(2, 5.0, (20.3, 54.4, 31.2), tilt=True)
    pts = torch.tensor(X + 0.21, device="cuda")
    one = torch.ones(len(X), 3, dtype=torch.float64, device="cuda") * 0.01
    fib = torch.zeros(3, d.n_nodes, dtype=torch.float64, device="cuda")
    torch.cuda.synchronize()
    lat = Lattice(d, 0.8, 0.02, precision, stream=stream)
    lat.add_body(synth.Body(X, F, rigid=False, ca=0.5, eb=1e-4, rho_ratio=1.1, r_ref=5.0, u_ref=0.02))
    lat.step(3)
    lat.sync()
    lat.ib_spread(pts, one, one[:, 0].contiguous(), fib)
    return [lat.populations(), lat.force(), *lat.body(0), fib]


@pytest.mark.parametrize("precision", ["f64", "f32"])
def test_a_side_stream_gives_the_same(precision):
    print(precision, flush=True)
    ref = _run(None, precision)
    assert ref[1].any() and ref[4].any()
    for _ in range(3):
        with torch.cuda.stream(torch.cuda.Stream()):
            out = _run(torch.cuda.current_stream(), precision)
        for a, b in zip(out, ref):
            assert torch.equal(a, b)
