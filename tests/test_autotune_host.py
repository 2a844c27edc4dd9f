"""The tuner's host side: a cached tuning belongs to the library that it was
timed with.  CPU only."""
import types

import pytest

torch = pytest.importorskip("torch")
from paper_2607_14513_amd import autotune, gsbc  # noqa: E402


def _descs(nblk, formats):
    d = gsbc.StreamDesc()
    d.n_streams, d.blocks_per_stream, d.arrangement = 16, nblk, gsbc.ARR_BANDS
    for k in range(16):
        d.format[k] = formats[k % len(formats)]
    return [d]


def test_key_names_the_library(monkeypatch, tmp_path):
    gsbc.load()                                    # (the tuning calls below use the built one)
    monkeypatch.setattr(torch.cuda, "current_device", lambda: 0)
    monkeypatch.setattr(torch.cuda, "get_device_properties",
                        lambda i: types.SimpleNamespace(name="card", multi_processor_count=256))
    keys = []
    for text in (b"one build", b"another", b"one build"):
        p = tmp_path / f"lib{len(keys)}.so"
        p.write_bytes(text)
        monkeypatch.setattr(gsbc, "LIB_PATH", str(p))
        keys.append(autotune.workload_key(_descs(100, [1, 7])))
    assert keys[0] == keys[2] != keys[1]
