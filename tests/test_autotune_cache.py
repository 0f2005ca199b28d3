"""The autotuner's cache keys: measurements hold for the library they were
taken with."""
import os

from paper_2410_11625_amd import _lib, autotune


def test_keys_follow_the_built_library(tmp_path, monkeypatch):
    monkeypatch.setattr(autotune, "arch", lambda device=None: "gfx950")
    a, b = tmp_path / "a.so", tmp_path / "b.so"
    a.write_bytes(b"kernels")
    b.write_bytes(b"other kernels")

    def keys(path):
        monkeypatch.setattr(_lib, "LIB_PATH", str(path))
        return autotune.frame_key(64, 96, 8, 3, 8), autotune._target()
    first = keys(a)
    assert first == keys(a) and set(first).isdisjoint(keys(b))
    a.write_bytes(b"rebuilt kernels")
    os.utime(a, ns=(1, 1))
    assert set(first).isdisjoint(keys(a))
