"""The per-interaction layout at the leaf sizes where its kernels change path:
records of few and of more than 64 targets or sources, chunks of 64 entries with
more rows than the row map holds, lists over one chunk, points that coincide,
periodic lists.  Records against the oracle bit by bit; sums to 1e-12 (FP64) and
1e-5 (FP32-mixed) of the FP64 oracle."""
import numpy as np
import pytest
import torch

import oracle
from paper_2511_21535_amd import api
from paper_2511_21535_amd import workloads as W

pytestmark = pytest.mark.gpu
TOL = {"fp64": 1e-12, "fp32": 1e-5}


def _rel(a, b):
    return float(np.linalg.norm(np.asarray(a) - np.asarray(b)) / np.linalg.norm(b))


def _sets(name):
    if name.startswith("cap"):
        return W.plummer_mixture(2500, 51), int(name[3:])
    if name == "slab":                       # lists over 64 entries
        return W.slab_particles(3000, 12, 0.01, 52), 8
    x, y, z, m = W.uniform_particles(600, 53)   # 200 points on one spot
    for v in (x, y, z):
        v[::3] = v[0]
    return (x, y, z, m), 4


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("name", ["cap1", "cap16", "cap33", "cap64", "cap200", "slab", "one spot"])
def test_records_and_sums(name, prec):
    (x, y, z, m), cap = _sets(name)
    g = [torch.as_tensor(np.ascontiguousarray(v), device="cuda") for v in (x, y, z, m)]
    t = api.Tree.build_particles(*g[:3], depth=20, leaf_cap=cap)
    o = oracle.build_tree_particles(x, y, z, depth=20, leaf_cap=cap)
    for periodic in (False, True):
        print(f"case interactions edges {name} {prec} periodic={periodic}", flush=True)
        nb = t.neighbors(periodic=periodic)
        on = oracle.neighbors_periodic(o) if periodic else oracle.neighbors(o)
        want = oracle.gravity(x, y, z, m, 1e-2, o, on)
        inter = api.restructure_interactions(t, nb, *g, prec=prec)
        got = [v.cpu().numpy() for v in api.gravity_interactions(t, nb, inter, 1e-2)]
        assert _rel(got[0], want[0]) <= TOL[prec]
        assert _rel(np.stack(got[1:]), np.stack(want[1:])) <= TOL[prec]
        starts, rec = oracle.restructure_interactions(o, on[0], on[1], x, y, z, m, prec=prec,
                                                      **(dict(nbr_shift=on[2]) if periodic else {}))[:2]
        assert np.array_equal(inter.rec_start.cpu().numpy(), starts)
        plane = inter.rows.cpu().numpy()[: inter.count]
        assert np.array_equal(plane.reshape(-1).view(np.uint8), np.ascontiguousarray(rec).reshape(-1).view(np.uint8))
