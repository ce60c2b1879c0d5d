"""The device memory that the adjoint keeps from one sweep to the next: it is
given back on request and with the last lattice, and a sweep after that gives
the same gradient."""
import gc

import pytest
import torch

import synth

pytestmark = pytest.mark.gpu

MIB = 1 << 20


def _free():
    torch.cuda.synchronize()
    return torch.cuda.mem_get_info()[0]


def test_the_kept_memory_is_given_back():
    from paper_2207_06043_amd import Lattice
    gc.collect()
    d = synth.periodic_box(96, 96, 96, body_force=(1e-5, 0.0, 0.0))
    lat, other = Lattice(d, 0.8, 0.02, "f64"), Lattice(synth.periodic_box(8, 8, 8), 0.8, 0.02, "f64")
    lam = torch.ones(19, lat.N, dtype=torch.float64, device="cuda")
    kept = 6 * 19 * lat.N * 8  # at least: the sweep's fields
    lat.adjoint(2, lam, checkpoint_every=2)
    lat.trim()
    ref = lat.adjoint(2, lam, checkpoint_every=2)
    lat.trim()
    torch.cuda.empty_cache()
    before = _free()
    got = lat.adjoint(2, lam, checkpoint_every=2)
    for a, b in zip(got, ref):
        assert torch.equal(a, b)
    del got, a
    torch.cuda.empty_cache()
    assert before - _free() >= kept
    other.trim()  # any lattice of the device
    assert before - _free() < 64 * MIB
    other.trim()  # nothing left: no error
    lat.adjoint(2, lam, checkpoint_every=2)
    del lat
    torch.cuda.empty_cache()
    other.adjoint(2, torch.ones(19, other.N, dtype=torch.float64), checkpoint_every=2)
    del other
    torch.cuda.empty_cache()
    gc.collect()
    assert _free() >= before
