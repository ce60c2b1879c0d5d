"""The status words of a checkpoint file: their order in the file is fixed
(stop, two pending words that are zero at a save, overflow between them, the
step count, the singular fits, zero), whatever their order on the device, so
that a file written before the device's words were reordered loads as it was.
The run stops on a spread contribution beyond the fixed-point range, which sets
the overflow word."""
import struct

import pytest

import synth

pytestmark = pytest.mark.gpu

UNSTABLE = 4
HEADER = 8 + 8 * 4 + 8  # magic, eight 32-bit words, the step count


def _lattice():
    from paper_2207_06043_amd import from_workload
    w = synth.tiny_pipe(with_body=True, rigid=False)
    w.bodies[0].v0 = -40.0 * (w.bodies[0].x - w.bodies[0].x.mean(axis=0))
    return from_workload(w, precision="f64")


def test_status_words_in_a_checkpoint(tmp_path):
    lat = _lattice()
    lat.step(3)
    assert lat.sync(raise_on_stop=False) == UNSTABLE
    lat.save(tmp_path / "c")
    data = (tmp_path / "c").read_bytes()
    stop, pend0, overflow, pend1, steps, singular, last = struct.unpack_from("<IIIIqiI", data, HEADER)
    assert (stop, pend0, overflow, pend1, steps, last) == (1, 0, 1, 0, lat.info()["steps_done"], 0)
    other = _lattice()
    other.load(tmp_path / "c")
    with pytest.raises(Exception, match="contribution"):
        other.sync()
    other.save(tmp_path / "d")
    assert (tmp_path / "d").read_bytes() == data
