"""The batch autotuner's cache on the host: entries of another library build
are not read, those of this one are."""
import hashlib
import json

from paper_2202_11819_amd import autotune, j3d


def test_entries_of_another_build_are_not_read(tmp_path, monkeypatch):
    probs = [j3d.Problem((40, 33, 27), pid=i) for i in range(4)]
    monkeypatch.setattr(autotune, "device_arch", lambda: "gfx950")
    timed = []

    def time_batch(problems, iters, tune, stream=None):
        timed.append(tune)
        return 1.0 if tune == autotune.LIBRARY else 2.0

    monkeypatch.setattr(autotune, "time_batch", time_batch)
    # the same version and one-sweep shapes, another build
    table = hashlib.sha256(repr(j3d.variants()).encode()).hexdigest()[:12]
    stale = f"gfx950|{j3d.j3d_version()}|{table}|batch|{autotune.size_class(probs)}"
    path = tmp_path / "tune.json"
    path.write_text(json.dumps({stale: {"tune": [25, 32, 0], "seconds": 1.0}}))
    assert autotune.tune_batch(probs, [100] * 4, cache_path=str(path)) == autotune.LIBRARY
    assert timed
    timed.clear()
    assert autotune.tune_batch(probs, [100] * 4, cache_path=str(path)) == autotune.LIBRARY
    assert not timed  # its own entry is

    other = tmp_path / "other.so"
    other.write_bytes(b"another build")
    assert autotune.library_digest(str(other)) != autotune.library_digest()
