"""Gravity sums and their adjoint at the leaf sizes where the workgroup's split
changes: leaves of few targets (their many partial sums are added in two steps
up to 16 targets), of many, near lists over more than one chunk of 256
neighbours, odd tile ends and points that coincide.  FP64 to 1e-12 and
FP32-mixed to 1e-5 of the FP64 oracle."""
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
        return W.plummer_mixture(4000, 31), int(name[3:])
    if name == "slab":   # lists of hundreds of leaves
        return W.slab_particles(6000, 20, 0.01, 32), 8
    x, y, z, m = W.uniform_particles(900, 33)   # 300 points on one spot: a leaf of more targets than threads
    for v in (x, y, z):
        v[::3] = v[0]
    return (x, y, z, m), 4


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("name", ["cap1", "cap3", "cap15", "cap16", "cap17", "cap64", "cap300", "slab", "one spot"])
def test_forward_and_adjoint(name, prec):
    (x, y, z, m), cap = _sets(name)
    print(f"case gravity edges {name} {prec}", flush=True)
    g = [torch.as_tensor(np.ascontiguousarray(v), device="cuda") for v in (x, y, z, m)]
    up = [W.normal_like(x.shape, 40 + i) for i in range(4)]
    gu = [torch.as_tensor(v, device="cuda") for v in up]
    eps = 1e-2
    t = api.Tree.build_particles(*g[:3], depth=20, leaf_cap=cap)
    o = oracle.build_tree_particles(x, y, z, depth=20, leaf_cap=cap)
    for periodic in (False, True):
        nb = t.neighbors(periodic=periodic)
        on = oracle.neighbors_periodic(o) if periodic else oracle.neighbors(o)
        want = oracle.gravity(x, y, z, m, eps, o, on)
        got = [v.cpu().numpy() for v in api.gravity(t, nb, eps, *g, prec=prec)]
        assert _rel(got[0], want[0]) <= TOL[prec]
        assert _rel(np.stack(got[1:]), np.stack(want[1:])) <= TOL[prec]
        wm, wx, wy, wz = oracle.gravity_adjoint(x, y, z, m, eps, *up, o, on)
        got = [v.cpu().numpy() for v in api.gravity_adjoint(t, nb, eps, *g, *gu, prec=prec)]
        assert _rel(got[3], wm) <= TOL[prec]
        assert _rel(np.stack(got[:3]), np.stack([wx, wy, wz])) <= TOL[prec]
