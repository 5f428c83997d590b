"""The binding in a forked child: torch refuses to use an initialised GPU there, and so does a call without
a stream.  The getters of an initialised torch are stood in for, so that no device is needed."""
import os

from paper_2606_20917_amd import nir


def test_a_forked_child_asks_torch_again(monkeypatch):
    monkeypatch.setattr(nir, "_current", (lambda: 0, lambda device: 4321))
    assert nir._stream(None) == 4321
    r, w = os.pipe()
    pid = os.fork()
    if pid == 0:
        os.write(w, b"1" if nir._current is None else b"0")
        os._exit(0)
    os.waitpid(pid, 0)
    os.close(w)
    answer = os.read(r, 1)
    os.close(r)
    assert answer == b"1"
    assert nir._stream(None) == 4321   # the parent keeps them
