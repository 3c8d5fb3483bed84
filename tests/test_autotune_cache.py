"""The autotuner's file cache (no GPU): shapes tuned for another kernel are not taken."""
import hashlib
import json
from types import SimpleNamespace

import torch

from paper_2511_21535_amd import api, autotune


def _tree():
    return SimpleNamespace(grids=[api.Grid(8, 0.125, 1.0)], n=512, leaf_start=torch.zeros(1))


def _tune(monkeypatch, tmp_path, cache):
    path = tmp_path / "cache.json"
    path.write_text(json.dumps(cache))
    monkeypatch.setenv("P2P_AUTOTUNE_CACHE", str(path))
    monkeypatch.setattr(torch.cuda, "get_device_name", lambda device: "card")
    monkeypatch.setattr(autotune, "time_call", lambda fn, reps: 1.0)
    q = torch.zeros(512, 32, dtype=torch.complex64)
    tile, _ = autotune.tune_helmholtz(_tree(), None, q=q, candidates=[(2, 1, 32)], copies=(1,))
    return tile, json.loads(path.read_text())


def test_entries_of_an_earlier_kernel_are_measured_again(monkeypatch, tmp_path):
    key = f"card|grids=1:{hashlib.sha1(b'8').hexdigest()[:16]}|nrhs=32|gather|fp32"
    tile, _ = _tune(monkeypatch, tmp_path, {key: {"tile": [4, 8, 32, 8], "ms": {}}})
    assert tile == (2, 1, 32, 1)


def test_own_entries_are_kept(monkeypatch, tmp_path):
    _, cache = _tune(monkeypatch, tmp_path, {})
    (key,) = cache
    tile, _ = _tune(monkeypatch, tmp_path, {key: {"tile": [4, 2, 32, 1], "ms": {}}})
    assert tile == (4, 2, 32, 1)


def test_no_launch_is_timed_twice():
    """Four tiles of 32 columns to a workgroup with a first entry of 4, else two."""
    shapes = [(4 if w == 4 else 2, c, r) for w, c, r in autotune.CANDIDATES]
    assert len(set(shapes)) == len(shapes)
