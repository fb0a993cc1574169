"""Which entries of the apply_H tuner's cache file are installed (no GPU): those of
this build of the library that weighed the automatic shape, and no others."""
import torch

from paper_2002_05725_amd import autotune

ARCH = "gfx950"
OLD_KEY = f"{ARCH}|N=32|c128|nvec=1"           # without the library build
OLD = {"tile_bits": 9, "xcd_remap": 1, "cols_per_group": 1, "ms": 0.38}


def _tune(monkeypatch, path):
    """What tune_apply installs from the cache alone, None if it starts timing."""
    class Timed(Exception):
        pass

    class Handle:
        N, dim = 32, 1 << 16

    installed = []
    monkeypatch.setattr(autotune, "_arch", lambda: ARCH)
    monkeypatch.setattr(autotune.api, "set_apply_tuning", lambda t, *a: installed.append(a))

    def generator(*a, **k):
        raise Timed()
    monkeypatch.setattr(autotune.torch, "Generator", generator)
    try:
        autotune.tune_apply(Handle(), torch.complex128, 1, cache=path)
    except Timed:
        assert not installed
        return None
    return installed


def test_entries_of_earlier_builds_are_timed_again(tmp_path, monkeypatch):
    path = str(tmp_path / "tune.json")
    autotune.write_cache(path, OLD_KEY, OLD)
    assert _tune(monkeypatch, path) is None
    # the same entry under today's key: the automatic shape was never weighed
    autotune.write_cache(path, autotune.cache_key(ARCH, 32, torch.complex128, 1), OLD)
    assert _tune(monkeypatch, path) is None
    # another build's key
    monkeypatch.setattr(autotune, "_build_id", lambda p: "0" * 16)
    autotune.write_cache(path, autotune.cache_key(ARCH, 32, torch.complex128, 1), dict(OLD, automatic_ms=1.0))
    monkeypatch.undo()
    assert _tune(monkeypatch, path) is None


def test_entries_of_this_build_are_installed(tmp_path, monkeypatch):
    path = str(tmp_path / "tune.json")
    key = autotune.cache_key(ARCH, 32, torch.complex128, 1)
    autotune.write_cache(path, key, dict(OLD, automatic_ms=0.05))
    assert _tune(monkeypatch, path) == [(0, 1, 0)]
    autotune.write_cache(path, key, dict(OLD, automatic_ms=0.5))
    assert _tune(monkeypatch, path) == [(9, 1, 1)]
