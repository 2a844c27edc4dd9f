"""The tuner's host side: a cached tuning belongs to the library that it was
timed with, and settings that launch the same kernels are timed once.  CPU only."""
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


@pytest.mark.parametrize("nblk,shared", [(1000, True), (70_000, False)])
def test_same_launches_are_timed_once(monkeypatch, nblk, shared):
    timed = []

    def time_batch(ctx, textures, descs, blocks, tuning, params, repeats):
        timed.append(tuning.as_dict())
        return 1.0 + 0.001 * (len(timed) * 7919 % 13)     # noise

    monkeypatch.setattr(autotune, "time_batch", time_batch)
    monkeypatch.setattr(autotune, "workload_key", lambda *a: "k")
    autotune.tune(None, None, _descs(nblk, [1, 1, 7]), None, use_cache=False)

    def launches(t):
        plain = t["item_rounds"] == 1 and t["wgs_per_cu"] == 0
        return (t["item_rounds"], t["wgs_per_cu"], 0 if plain and shared else t["bc1_lanes"],
                min(t["bc7_split"], 2), t["concurrent"])

    assert len({launches(t) for t in timed}) == len(timed) > 5
