"""Near lists where their search changes path: leaves taken together by parent
(roots, first levels, grids of single boxes), leaves of many candidates (a large
leaf beside finely split ones: one workgroup each, more chunks than it holds at
a time), lists of 64 entries and more, and capacities that do not suffice.
Bit-exact against the oracle."""
import ctypes

import numpy as np
import pytest
import torch

import oracle
from paper_2511_21535_amd import _lib as L
from paper_2511_21535_amd import api
from paper_2511_21535_amd import workloads as W

pytestmark = pytest.mark.gpu


def _beside(n_fine, n_coarse, seed, edge=0.5):
    """n_fine points in the half [0.5, 0.5 + edge) x [0,1)^2, n_coarse in the other half."""
    rng = np.random.default_rng(seed)
    p = rng.random((n_fine + n_coarse, 3))
    p[:n_fine, 0] = 0.5 + edge * p[:n_fine, 0]
    p[n_fine:, 0] *= 0.5
    return p[:, 0].copy(), p[:, 1].copy(), p[:, 2].copy()


SETS = {
    "one point": lambda: W.uniform_particles(1, 1)[:3],
    "one leaf": lambda: W.uniform_particles(8, 2)[:3],
    "two levels": lambda: W.uniform_particles(60, 3)[:3],
    "uniform": lambda: W.uniform_particles(6000, 4)[:3],
    "plummer": lambda: W.plummer_mixture(30000, 5)[:3],
    # leaves of a quarter of the domain beside thousands of fine ones
    "coarse beside fine": lambda: _beside(40000, 24, 6),
    "slab": lambda: W.slab_particles(30000, 40, 0.01, 7)[:3],
}
# more chunks of 64 candidates than a workgroup holds at a time (4096)
SETS["many chunks"] = lambda: _beside(1200000, 9, 8)


@pytest.mark.parametrize("periodic", [False, True])
@pytest.mark.parametrize("name", SETS)
def test_particles(name, periodic):
    x, y, z = SETS[name]()
    cap = 2 if name == "many chunks" else 8
    g = [torch.as_tensor(np.ascontiguousarray(v), device="cuda") for v in (x, y, z)]
    print(f"case near lists {name} periodic={periodic}", flush=True)
    t = api.Tree.build_particles(*g, depth=20, leaf_cap=cap)
    nb = t.neighbors(periodic=periodic)
    o = oracle.build_tree_particles(x, y, z, depth=20, leaf_cap=cap)
    start = nb.nbr_start.cpu().numpy()
    # the lists of the largest leaves and of a sample, where there are many
    sel = np.arange(o.n_leaves)
    if o.n_leaves > 20000:
        sel = np.unique(np.concatenate([np.argsort(o.leaf_level, kind="stable")[:4], sel[:: o.n_leaves // 200]]))
    if periodic:
        ws, wi, wc = oracle.neighbors_periodic(o, targets=sel)
    else:
        ws, wi = oracle.neighbors(o, targets=sel)
    idx = nb.nbr_idx.cpu().numpy()
    code = nb.nbr_shift.cpu().numpy() if periodic else None
    assert start[0] == 0 and start[-1] == nb.count
    for k, A in enumerate(sel):
        assert np.array_equal(idx[start[A]:start[A + 1]], wi[ws[k]:ws[k + 1]]), f"leaf {A}"
        if periodic:
            assert np.array_equal(code[start[A]:start[A + 1]], wc[ws[k]:ws[k + 1]]), f"leaf {A}"
    occ = np.diff(o.leaf_start).astype(np.int64)
    assert nb.red_entries == int(occ[idx].sum())


# 512 boxes and 513: no leaf has more candidates than one wavefront takes, or may
# have; 16,354 and 16,625: starts by one workgroup, or by many
@pytest.mark.parametrize("sides", [[4], [4] * 9, [4, 8, 4, 12], [8] * 3, [16, 4], [16], [32], [32, 4], [100, 36], [100, 40]])
def test_grids(sides):
    grids = [api.Grid(s, *W.grid_geometry(s)) for s in sides]
    print(f"case near lists grids {sides}", flush=True)
    nb = api.Tree.build_grids(grids, device="cuda").neighbors()
    ws, wi = oracle.neighbors(oracle.build_tree_grids(sides))
    assert np.array_equal(nb.nbr_start.cpu().numpy(), ws)
    assert np.array_equal(nb.nbr_idx.cpu().numpy(), wi)


@pytest.mark.parametrize("a,b", [("plummer", "coarse beside fine"), ("coarse beside fine", "plummer"),
                                 ("one leaf", "uniform"), ("slab", "one point")])
def test_remote(a, b):
    pa, pb = SETS[a](), SETS[b]()
    ga, gb = ([torch.as_tensor(np.ascontiguousarray(v), device="cuda") for v in p] for p in (pa, pb))
    print(f"case remote lists {a}, {b}", flush=True)
    ta, tb = (api.Tree.build_particles(*g, depth=20, leaf_cap=8) for g in (ga, gb))
    nb = api.build_neighbors(ta, src_tree=tb)
    ws, wi = oracle.neighbors_remote(*(oracle.build_tree_particles(*p, depth=20, leaf_cap=8) for p in (pa, pb)))[:2]
    assert np.array_equal(nb.nbr_start.cpu().numpy(), ws)
    assert np.array_equal(nb.nbr_idx.cpu().numpy(), wi)


@pytest.mark.parametrize("name", ["plummer", "coarse beside fine"])
def test_capacity_refused_writes_nothing(name):
    x, y, z = SETS[name]()
    g = [torch.as_tensor(np.ascontiguousarray(v), device="cuda") for v in (x, y, z)]
    t = api.Tree.build_particles(*g, depth=20, leaf_cap=8)
    want = t.neighbors().count
    ts = t.struct()
    for cap, has_idx, status in ((want - 1, True, L.P2P_ECAPACITY), (want, False, L.P2P_EINVAL), (want, True, L.P2P_OK)):
        start = torch.full((t.n_leaves + 1,), -7, dtype=torch.int64, device="cuda")
        idx = torch.full((want,), -7, dtype=torch.int32, device="cuda")
        s = L.p2p_nbrs()
        s.cap, s.nbr_start, s.nbr_idx = cap, start.data_ptr(), idx.data_ptr() if has_idx else None
        nb = ctypes.c_size_t(0)
        L.check(L.p2p_build_neighbors(ctypes.byref(ts), ctypes.byref(s), None, ctypes.byref(nb), None))
        ws = torch.empty(nb.value, dtype=torch.uint8, device="cuda")
        torch.cuda.synchronize()
        print(f"case near lists cap={cap} of {want}", flush=True)
        st = L.p2p_build_neighbors(ctypes.byref(ts), ctypes.byref(s), ctypes.c_void_p(ws.data_ptr()),
                                   ctypes.byref(nb), None)
        torch.cuda.synchronize()
        assert st == status
        if status == L.P2P_OK:
            assert s.count == want and int(start[-1]) == want and bool((idx >= 0).all())
        else:
            assert bool((start == -7).all()) and bool((idx == -7).all())
            if status == L.P2P_ECAPACITY:
                assert s.count == want
