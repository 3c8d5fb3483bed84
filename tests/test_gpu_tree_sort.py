"""Particle trees at the sizes where the sort and the leaf steps change path:
places by counting up to 8192 points, tiles of 1024 up to 65536, of 4096
beyond (their counts added up to 64 tiles, scanned beyond), runs of equal top
key bits of at most 64 keys, leaf counts scanned beyond 4M slots.  perm is
stable, so points that coincide stand in caller order.  Bit-exact against the
oracle."""
import ctypes

import numpy as np
import pytest
import torch

import oracle
from paper_2511_21535_amd import _lib as L
from paper_2511_21535_amd import api
from paper_2511_21535_amd import workloads as W

pytestmark = pytest.mark.gpu


def _check(x, y, z, depth, cap):
    g = [torch.as_tensor(np.ascontiguousarray(v), device="cuda") for v in (x, y, z)]
    print(f"case tree n={len(x)} depth={depth} cap={cap}", flush=True)
    t = api.Tree.build_particles(*g, depth=depth, leaf_cap=cap)
    o = oracle.build_tree_particles(x, y, z, depth=depth, leaf_cap=cap)
    assert t.n_leaves == o.n_leaves and t.max_level == int(o.leaf_level.max())
    perm = t.perm.cpu().numpy()
    assert np.array_equal(perm, o.perm)
    assert np.array_equal(t.iperm.cpu().numpy()[perm], np.arange(len(x)))
    assert np.array_equal(t.leaf_start.cpu().numpy(), o.leaf_start)
    assert np.array_equal(t.leaf_key.cpu().numpy().view(np.uint64), o.leaf_key.astype(np.uint64))
    assert np.array_equal(t.leaf_level.cpu().numpy(), o.leaf_level)


@pytest.mark.parametrize("n", [1, 2, 15, 16, 17, 255, 257, 1025, 8191, 8192, 8193, 65535, 65536, 65537, 262144, 262145])
def test_sizes(n):
    x, y, z, _ = (W.plummer_mixture if n >= 100 else W.uniform_particles)(n, 900 + n % 97)
    _check(x, y, z, 20, 32)


@pytest.mark.parametrize("cap", [0, 1, 64, 65, 2048, 2049])
@pytest.mark.parametrize("n", [3001, 20000])
def test_leaf_caps(n, cap):
    x, y, z, _ = W.plummer_mixture(n, 77)
    _check(x, y, z, 4 if cap == 0 else 20, cap)


@pytest.mark.parametrize("run", [1, 63, 64, 65, 66, 5000])
def test_equal_top_bits(run):
    """Clusters inside one cell of 2^-32 of the domain: `run` points each, some of them coinciding, in mixed order."""
    x, y, z, _ = W.uniform_particles(9000, 5)
    rng = np.random.default_rng(run)
    for c in range(3):
        # the cell of level 10 at c holds several cells of 2^-32; its first corner holds the cluster
        pos = (rng.integers(0, 4, (run, 3)) * 2.0 ** -20) + (0.25 + 0.125 * c)
        x, y, z = (np.concatenate([v, pos[:, d]]) for d, v in enumerate((x, y, z)))
    p = rng.permutation(len(x))
    _check(x[p], y[p], z[p], 20, 8)


def test_one_point_many_times():
    x, y, z, _ = W.uniform_particles(300, 6)
    x, y, z = (np.tile(v, 100) for v in (x, y, z))
    _check(x, y, z, 20, 64)


def test_many_slots():
    x, y, z, _ = W.uniform_particles((1 << 22) + 1, 8)
    _check(x, y, z, 20, 64)


@pytest.mark.parametrize("n", [500, 20000])
def test_refused_builds_write_nothing(n):
    x, y, z, _ = W.plummer_mixture(n, 3)
    for bad in (False, True):
        if bad:
            x = x.copy()
            x[n // 2] = 1.0
        g = [torch.as_tensor(v, device="cuda") for v in (x, y, z)]
        arrs = [torch.full((n + 1,), -7, dtype=d, device="cuda") for d in
                (torch.int32, torch.int32, torch.int32, torch.int64, torch.int8)]
        t = L.p2p_tree()
        t.n, t.cap_leaves = n, n if bad else 3
        t.perm, t.iperm, t.leaf_start, t.leaf_key, t.leaf_level = (a.data_ptr() for a in arrs)
        nb = ctypes.c_size_t(0)
        args = [ctypes.c_void_p(v.data_ptr()) for v in g] + [None, 0, 20, 64, ctypes.byref(t)]
        L.check(L.p2p_build_tree(*args, None, ctypes.byref(nb), None))
        ws = torch.empty(nb.value, dtype=torch.uint8, device="cuda")
        torch.cuda.synchronize()
        print(f"case refused build n={n} bad={bad}", flush=True)
        st = L.p2p_build_tree(*args, ctypes.c_void_p(ws.data_ptr()), ctypes.byref(nb), None)
        assert st == (L.P2P_EDOMAIN if bad else L.P2P_ECAPACITY)
        assert t.n_leaves == (0 if bad else oracle.build_tree_particles(x, y, z, depth=20, leaf_cap=64).n_leaves)
        torch.cuda.synchronize()
        assert all(bool((a == -7).all()) for a in arrs)
