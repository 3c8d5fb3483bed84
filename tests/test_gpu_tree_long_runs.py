"""Particle trees with runs of more than 64 points that share the top 32 bits of
their keys (a cell of 2^-32 of the domain): their points are sorted among themselves,
in tiles of 1024 up to 65536 of them and of 4096 beyond; and grid trees of so many
instances that the boxes' runs would be long.  perm is stable, so points that coincide stand in
caller order.  Bit-exact against the oracle."""
import numpy as np
import pytest
import torch

import oracle
from paper_2511_21535_amd import api
from paper_2511_21535_amd import workloads as W

pytestmark = pytest.mark.gpu


def _check(x, y, z, cap=8):
    t = api.Tree.build_particles(*[torch.as_tensor(np.ascontiguousarray(v), device="cuda") for v in (x, y, z)],
                                 depth=20, leaf_cap=cap)
    o = oracle.build_tree_particles(x, y, z, depth=20, leaf_cap=cap)
    assert t.n_leaves == o.n_leaves and t.max_level == int(o.leaf_level.max())
    assert np.array_equal(t.perm.cpu().numpy(), o.perm)
    assert np.array_equal(t.iperm.cpu().numpy()[o.perm], np.arange(len(x)))
    assert np.array_equal(t.leaf_start.cpu().numpy(), o.leaf_start)
    assert np.array_equal(t.leaf_key.cpu().numpy().view(np.uint64), o.leaf_key.astype(np.uint64))
    assert np.array_equal(t.leaf_level.cpu().numpy(), o.leaf_level)


def _points(runs, background, seed):
    """Clusters of the given sizes, each inside one cell of 2^-32, some of whose points coincide, in mixed order among
    uniform points.  The first cluster lies at the domain's first corner, the last at its last."""
    rng = np.random.default_rng(seed)
    parts = [rng.random((background, 3))]
    for c, n in enumerate(runs):
        at = 0.0 if c == 0 else 1.0 - 2.0 ** -10 if c == len(runs) - 1 else 2.0 ** -10 * rng.integers(1, 1000, 3)
        # a cell of 2^-30 (edge 2^-10): its first quarter in y and z is one of 2^-32
        parts.append(at + rng.integers(0, 4096, (n, 3)) * 2.0 ** -22 * np.array([1.0, 0.25, 0.25]))
    p = np.concatenate(parts)
    return rng.permutation(p)


@pytest.mark.parametrize("runs", [[65], [100, 65, 66], [1024], [1025, 65], [4097, 8191, 127], [65536], [65000, 70, 65500],
                                  [66] * 300])
def test_long_runs(runs):
    print(f"case long runs {runs[:4]} of {len(runs)}", flush=True)
    _check(*_points(runs, 9000, len(runs)).T)


@pytest.mark.parametrize("n", [8193, 65536, 65537, 300000])
def test_all_points_in_one_run(n):
    print(f"case one run of {n}", flush=True)
    _check(*_points([n], 0, n).T)


def test_tight_sphere():
    """One Plummer sphere of scale radius 0.002: runs of hundreds of points."""
    print("case tight sphere", flush=True)
    rng = np.random.default_rng(3)
    n = 1 << 17
    r = 0.002 / np.sqrt((1.0 - rng.random(n)) ** (-2.0 / 3.0) - 1.0 + 1e-300)
    d = rng.standard_normal((n, 3))
    p = 0.4 + d / np.linalg.norm(d, axis=1)[:, None] * np.minimum(r, 0.3)[:, None]
    _check(*p.T, cap=64)


def test_grid_of_many_instances():
    """One grid of side 132 among 16,385 of side 4: 39 key bits, of which the top 32 are shared by 128 points."""
    print("case grid tree of many instances", flush=True)
    sides = [4] * 9000 + [132] + [4] * 7385
    t = api.Tree.build_grids([api.Grid(s, *W.grid_geometry(s)) for s in sides], device="cuda")
    o = oracle.build_tree_grids(sides)
    assert t.n_leaves == o.n_leaves
    assert np.array_equal(t.perm.cpu().numpy(), o.perm)
    assert np.array_equal(t.leaf_start.cpu().numpy(), o.leaf_start)
    assert np.array_equal(t.leaf_key.cpu().numpy().view(np.uint64), o.leaf_key.astype(np.uint64))
