"""Tuning entries hold for the library they were timed on, and for no other."""

from paper_1503_06189_amd import tune

# as written when both batch kernels ran on the int8 matrix instructions
OLD = {"version": 2, "chunk_steps": 867, "geometry": "super", "ms": 1.35,
       "timings_ms": {"super/867": 1.35, "halves/867": 1.38}, "instances": 128}


def _lookup(monkeypatch, tmp_path, entry):
    path = str(tmp_path / "tune.json")
    monkeypatch.setattr(tune, "_key", lambda items: ("gfx950/256cu|k", []))
    tune._store("gfx950/256cu|k", entry, path)
    return tune.lookup([None], path)


def test_entries_of_replaced_kernels_are_not_used(monkeypatch, tmp_path):
    assert _lookup(monkeypatch, tmp_path, OLD) is None
    assert _lookup(monkeypatch, tmp_path, dict(OLD, version=tune.CACHE_VERSION)) is None


def test_entries_of_another_library_are_not_used(monkeypatch, tmp_path):
    entry = dict(OLD, version=tune.CACHE_VERSION, library=tune.library_digest())
    assert _lookup(monkeypatch, tmp_path, entry) == entry
    assert _lookup(monkeypatch, tmp_path, dict(entry, library="0" * 20)) is None
    copy = tmp_path / "libxengine.so"
    copy.write_bytes(open(tune.xengine.LIB_PATH, "rb").read() + b"\0")
    monkeypatch.setattr(tune.xengine, "LIB_PATH", str(copy))
    assert _lookup(monkeypatch, tmp_path, entry) is None
