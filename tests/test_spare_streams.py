"""The streams of closed contexts: a context collected while their lock is held
closes without waiting for it, a stream that could not be waited for is not
handed on, and one whose outputs are alive is not destroyed.  CPU only (made-up
handles)."""
import threading

import pytest

torch = pytest.importorskip("torch")
from paper_2607_14513_amd import gsbc  # noqa: E402


class _Lib:
    def __init__(self, status):
        self.status = status

        self.destroyed = []

    def gsbc_destroy(self, h):
        return self.status

    def hipStreamDestroy(self, h):
        self.destroyed.append(h.value)


def _context(handle):
    c = object.__new__(gsbc.Context)
    c._h, c._own, c.device = 1, handle, torch.device("cuda", 0)
    return c


def test_closing_a_context_inside_the_lock(monkeypatch):
    monkeypatch.setattr(gsbc, "load", lambda: _Lib(gsbc.OK))

    class Collects(dict):
        def setdefault(self, key, value):          # as a collection here would
            spare = super().setdefault(key, value)
            if not spare:
                spare.append(0)
                _context(11).close()
            return spare

    monkeypatch.setattr(gsbc, "_spare_streams", Collects())
    t = threading.Thread(target=lambda: _context(12).close(), daemon=True)
    t.start()
    t.join(20)
    assert not t.is_alive()
    assert sorted(gsbc._spare_streams[0]) == [0, 11, 12]


@pytest.mark.parametrize("status,spare", [(gsbc.OK, [21]), (gsbc.E_DEVICE, [])])
def test_only_streams_that_were_waited_for(monkeypatch, status, spare):
    monkeypatch.setattr(gsbc, "load", lambda: _Lib(status))
    monkeypatch.setattr(gsbc, "_spare_streams", {})
    c = _context(21)
    c.close()
    assert gsbc._spare_streams.get(0, []) == spare
    assert c._h is None and c._own is None


def test_stream_of_a_living_output_is_kept(monkeypatch):
    lib, waited = _Lib(gsbc.OK), []
    most = gsbc._SPARE_STREAMS
    segments = [{"stream": 100 + k, "device": 0, "blocks": [{"state": "active_allocated"}, {"state": "inactive"}]}
                for k in range(most + 3)]
    monkeypatch.setattr(gsbc, "load", lambda: lib)
    monkeypatch.setattr(gsbc, "_spare_streams", {})
    monkeypatch.setattr(gsbc, "_held_streams", {}, raising=False)
    monkeypatch.setattr(torch.cuda, "memory_snapshot", lambda: segments)
    monkeypatch.setattr(torch.cuda, "default_stream",
                        lambda d: type("S", (), {"synchronize": lambda self: waited.append(list(lib.destroyed))})())
    for k in range(most + 2):
        _context(100 + k).close()
    assert lib.destroyed == [] and len(gsbc._spare_streams[0]) == most
    segments[most]["blocks"] = [{"state": "inactive"}]       # its outputs are gone
    _context(100 + most + 2).close()
    assert lib.destroyed == [100 + most] and waited == [[]]
    kept = {gsbc._take_stream(0) for _ in range(most + 2)}   # the others go to the next contexts
    assert kept == {100 + k for k in range(most + 3)} - {100 + most}
