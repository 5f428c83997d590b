"""The binding enqueues on torch's current stream of the moment, call by call."""
import threading

import pytest

torch = pytest.importorskip("torch")

from paper_2606_20917_amd import nir

pytestmark = pytest.mark.gpu


def test_current_stream_is_asked_for_at_every_call():
    def now():
        return nir._stream(None), torch.cuda.current_stream().cuda_stream

    assert len(set(now())) == 1
    side, other = torch.cuda.Stream(), torch.cuda.Stream()
    with torch.cuda.stream(side):
        assert now() == (side.cuda_stream, side.cuda_stream)
        with torch.cuda.stream(other):
            assert now()[0] == other.cuda_stream
        seen = []
        t = threading.Thread(target=lambda: seen.append(now()))   # another thread: its own current stream
        t.start()
        t.join()
        assert seen[0][0] == seen[0][1]
        assert now()[0] == side.cuda_stream
    assert len(set(now())) == 1
    assert nir._stream(side) == side.cuda_stream and nir._stream(1234) == 1234
