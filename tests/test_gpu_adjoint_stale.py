"""The coupled adjoint's states in memory that holds NaN, through the C ABI: a
sweep on a lattice of another shape and type fills the memory that the next
sweep takes, once with zeros and once with NaN, and the next sweep's results
must not tell.  The capsule's supports lie at nodes whose wall links have no
fluid node behind them (the interpolated rule's coefficients are zero there),
where what the sweep's states hold at solid nodes is closest to being used.

Bound: a repeat of the same sweep, 1e-12 of each array's largest value (the
transposes are summed in any order)."""
import numpy as np
import pytest
import torch

import synth

pytestmark = pytest.mark.gpu

U, STEPS = 0.02, 5


def _workload(precision):
    d = synth.pipe(30, 10, 10, 3.6, u_max=U, tau=0.8, init="poiseuille")
    X, F = synth.icosphere(1, 1.8, (12.3, 5.0, 4.3), tilt=True)
    c = X.mean(axis=0)
    X = c + (X - c) * np.array([1.1, 1.0, 0.92])
    b = synth.Body(X, F, rigid=False, ca=0.5, eb=1e-3, rho_ratio=1.1, r_ref=2.0, u_ref=U)
    return synth.Workload("pipe", d, [b], 0.8, U, precision, STEPS)


def _nodes_without_a_neighbour(d):
    """Nodes with a wall link whose first or second node behind is not fluid."""
    n = np.array([d.nx, d.ny, d.nz])
    solid = (d.node_type == synth.SOLID).reshape(d.nz, d.ny, d.nx)
    x = np.stack([d.link_node % d.nx, d.link_node // d.nx % d.ny, d.link_node // (d.nx * d.ny)], 1)
    e = synth.D3Q19_DIRS[d.link_dir]
    out = np.zeros(len(x), bool)
    for k in (1, 2):
        y = x - k * e
        inside = ((y >= 0) & (y < n)).all(1)
        y = np.clip(y, 0, n - 1)
        out |= ~inside | solid[y[:, 2], y[:, 1], y[:, 0]]
    return set(d.link_node[out].tolist())


def _supports(w):
    d, b = w.domain, w.bodies[0]
    c = np.floor(b.x[b.faces].mean(axis=1) + 0.5).astype(int)
    o = np.array([(i, j, k) for k in (-1, 0, 1) for j in (-1, 0, 1) for i in (-1, 0, 1)])
    s = (c[:, None] + o[None]).reshape(-1, 3)
    return set((s[:, 0] + d.nx * (s[:, 1] + d.ny * s[:, 2])).tolist())


@pytest.mark.parametrize("every", [2, 5])
@pytest.mark.parametrize("precision", ["f64", "f32", "f16s"])
def test_a_coupled_sweep_uses_nothing_that_another_left(precision, every):
    from paper_2207_06043_amd import Lattice, from_workload
    w = _workload(precision)
    assert len(_nodes_without_a_neighbour(w.domain) & _supports(w)) >= 10
    rng = np.random.default_rng(5)
    fl = w.domain.node_type != synth.SOLID
    lam = torch.from_numpy(rng.normal(size=(19, w.domain.n_nodes)) * fl)
    obs = torch.from_numpy(rng.normal(size=(19, w.domain.n_nodes)) * fl)
    print(precision, every, flush=True)
    lat = from_workload(w, precision=precision)
    other = Lattice(synth.periodic_box(32, 32, 32), 0.8, U, "f64")

    def sweep(left):
        fill = torch.full((19, other.N), left, dtype=torch.float64)
        other.adjoint(3, fill, fill, checkpoint_every=3)
        out = lat.adjoint_run(STEPS, lam, obs, taylor_weight=2.0, taylor_body=0, checkpoint_every=every,
                              body_grad=True)
        return [t.cpu().numpy() for t in out[:3]] + [np.array(out[3])]

    ref, got = sweep(0.0), sweep(float("nan"))
    for r, g in zip(ref, got):
        assert np.isfinite(r).all() and np.abs(r).max() > 0.0
        assert np.abs(g - r).max() <= 1e-12 * np.abs(r).max()
