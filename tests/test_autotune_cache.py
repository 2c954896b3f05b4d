"""The autotuner's saved choices hold for the library they were timed with."""
import json
import shutil
import types

import pytest

torch = pytest.importorskip("torch")


def test_a_choice_of_another_library_is_not_taken(tmp_path, monkeypatch):
    from paper_2307_03404_amd import batch, pxm
    pxm.lib()
    grid = types.SimpleNamespace(reso=(8, 8, 8), n_alloc=3)
    rays = types.SimpleNamespace(n_rays=10, n_frames=1)
    opts = types.SimpleNamespace(flags=0, color_act=0)
    sig = batch._signature(grid, rays, opts, 3)
    assert batch._signature(grid, rays, opts, 3) == sig
    # a choice saved without its library, as older versions did, and one of this library
    path = tmp_path / "tune.json"
    old = "r8x8x8_n3_rays10_f1_w3_fl0_act0"
    path.write_text(json.dumps({old: {"best": [64, 1], "ms": {}}, sig: {"best": [128, 2], "ms": {}}}))
    tuner = batch.Autotuner(str(path))
    assert sig in tuner.cache and sig != old
    applied = []
    monkeypatch.setattr(pxm, "set_tuning", lambda b, v: applied.append((b, v)))
    assert tuner.tune(grid, rays, opts, None, None, None, 3)[0] == (128, 2) and applied == [(128, 2)]
    # the same problem under another build
    other = tmp_path / "other.so"
    shutil.copy(pxm.LIB_PATH, other)
    with open(other, "ab") as fh:
        fh.write(b"\0")
    monkeypatch.setattr(pxm, "LIB_PATH", str(other))
    assert batch._signature(grid, rays, opts, 3) not in tuner.cache


def test_every_launch_shape_is_timed_once():
    from paper_2307_03404_amd import batch
    # the plain launches (variant 0) take no block
    shapes = {(None if v == 0 else b, v) for b, v in batch.CANDIDATES}
    assert len(shapes) == len(batch.CANDIDATES) == 7
