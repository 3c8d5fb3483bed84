"""Helmholtz batches of more distinct k h than a call keeps G blocks for (256), or
a plan (4096): the instances are taken in groups.  Against the FP64 oracle at the
project's tolerances (1e-5 and 1e-12), calls and plans to the same bits, and the
memory of a call bounded."""
import numpy as np
import pytest
import torch

import oracle
from paper_2511_21535_amd import api
from paper_2511_21535_amd import workloads as W

pytestmark = pytest.mark.gpu

TOL = {"fp64": 1e-12, "fp32": 1e-5}


def _batch(sides, kh):
    h = np.array([1.0 / s for s in sides])
    kw = np.asarray(kh) / h
    t = api.Tree.build_grids([api.Grid(int(s), float(a), float(k)) for s, a, k in zip(sides, h, kw)], device="cuda")
    return t, t.neighbors(), h, kw


def _rel(a, b):
    return float(np.linalg.norm(a.ravel() - b.ravel()) / np.linalg.norm(b))


# instances of 1 and of 8 boxes; one past a group, exactly two full groups, k h that come back in a later group (600
# among 660 instances)
MEDIA = {"257": 257, "512": 512, "600": 600}


@pytest.mark.parametrize("media", sorted(MEDIA))
@pytest.mark.parametrize("prec,nrhs,tile", [("fp64", 1, None), ("fp64", 3, None), ("fp32", 1, None), ("fp32", 3, None),
                                            ("fp32", 32, None), ("fp32", 32, (2, 1, 32, 2))])
def test_groups(prec, nrhs, tile, media):
    m = MEDIA[media]
    n = 660 if m == 600 else m
    print(f"case many media {m} {prec} nrhs={nrhs} tile={tile}", flush=True)
    sides = [8 if i % 3 else 4 for i in range(n)]
    t, nb, h, kw = _batch(sides, [0.2 + 0.5 * (i * 7 % m) / m for i in range(n)])
    q = W.grid_rhs(t.n, nrhs, seed=5).astype(np.complex128 if prec == "fp64" else np.complex64)
    q = q[:, 0] if nrhs == 1 else q
    gq = torch.as_tensor(np.ascontiguousarray(q), device="cuda")
    ref = oracle.helmholtz(sides, q.reshape(t.n, nrhs), h=h, kw=kw).reshape(q.shape)
    u = api.helmholtz(t, nb, gq, prec=prec, tile=tile)
    assert _rel(u.cpu().numpy(), ref) <= TOL[prec]
    plan = api.HelmholtzPlan(t, nb, prec=prec, nrhs=nrhs, tile=tile)
    assert _rel(api.helmholtz(t, nb, gq, prec=prec, plan=plan).cpu().numpy(), ref) <= TOL[prec]
    red = api.restructure(t, nb, [gq], prec=prec, nrhs=nrhs)
    for p in (None, plan):
        v = api.helmholtz(t, nb, None, layout="redundant", prec=prec, red=red, plan=p, tile=tile if p is None else None)
        assert _rel(v.cpu().numpy(), ref) <= TOL[prec]
    if tile is None:
        a = api.helmholtz_adjoint(t, nb, gq, prec=prec, conjugate=True).cpu().numpy()
        want = np.conj(oracle.helmholtz(sides, np.conj(q).reshape(t.n, nrhs), h=h, kw=kw)).reshape(q.shape)
        assert _rel(a, want) <= TOL[prec]


@pytest.mark.parametrize("prec,nrhs", [("fp64", 2), ("fp32", 1), ("fp32", 2)])
def test_plan_of_more_media_than_it_keeps(prec, nrhs):
    """4100 one-box grids: the plan holds the parameters, its calls form the blocks in groups, also in a graph."""
    n = 4100
    print(f"case plan of {n} media {prec} nrhs={nrhs}", flush=True)
    sides = [4] * n
    t, nb, h, kw = _batch(sides, [0.2 + 0.5 * i / n for i in range(n)])
    q = W.grid_rhs(t.n, nrhs, seed=6).astype(np.complex128 if prec == "fp64" else np.complex64)
    q = q[:, 0] if nrhs == 1 else q
    gq = torch.as_tensor(np.ascontiguousarray(q), device="cuda")
    ref = oracle.helmholtz(sides, q.reshape(t.n, nrhs), h=h, kw=kw).reshape(q.shape)
    plan = api.HelmholtzPlan(t, nb, prec=prec, nrhs=nrhs)
    assert plan.buf.numel() < 1 << 20
    out = torch.empty_like(gq)
    call = lambda: api.helmholtz(t, nb, gq, prec=prec, plan=plan, out=out)
    assert _rel(call().cpu().numpy(), ref) <= TOL[prec]
    first = out.clone()
    g = api.Graph(call)
    for _ in range(3):
        out.zero_()
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, first)


@pytest.mark.parametrize("prec,nrhs", [("fp64", 3), ("fp32", 3)])
def test_memory_of_a_call(prec, nrhs):
    """1000 media: the blocks of 256 at a time, 1.77 MB (FP64) or 1.33 MB a set."""
    n = 1000
    print(f"case memory of {n} media {prec}", flush=True)
    t, nb, _, _ = _batch([4] * n, [0.2 + 0.5 * i / n for i in range(n)])
    q = torch.zeros(t.n, nrhs, dtype=torch.complex128 if prec == "fp64" else torch.complex64, device="cuda")
    out = torch.empty_like(q)
    torch.cuda.synchronize()
    torch.cuda.empty_cache()
    torch.cuda.reset_peak_memory_stats()
    before = torch.cuda.memory_allocated()
    api.helmholtz(t, nb, q, prec=prec, out=out)
    torch.cuda.synchronize()
    assert torch.cuda.max_memory_allocated() - before < 256 * 1.8e6 + 4 * q.numel() * q.element_size() + (1 << 21)
