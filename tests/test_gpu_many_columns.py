"""The Helmholtz product for many columns with few right-hand sides: a
wavefront's 16 columns span several boxes, a tile of 128 columns up to 128 of
them, whose map is then filled in several rounds.  One right-hand side and a few,
whole and partial tiles, one instance and batches, both layouts and directions,
against the FP64 oracle on sampled targets (1e-5).  And calls of two host threads
with different numbers of right-hand sides."""
import threading

import numpy as np
import pytest
import torch

import oracle
from paper_2511_21535_amd import api
from paper_2511_21535_amd import workloads as W

pytestmark = pytest.mark.gpu

TOL = 1e-5


def _rel(a, b):
    return float(np.linalg.norm(a.ravel() - b.ravel()) / np.linalg.norm(b))


# enough columns for rounds of tiles at least three quarters full
CASES = [
    ([120], 1),            # 27,000 columns, 128 boxes to a tile, the last tile partial
    ([32] * 60, 1),        # 60 instances of four whole tiles: uploaded parameters
    ([20] * 200, 1),       # instances of 125 boxes: one tile each, three columns short of it
    ([100], 2),
    ([80], 3),
    ([64], 6),             # 24,576 columns, the fewest
    ([64], 7),
    ([44, 40, 36], 9),
    ([48], 15),
    ([48], 16),            # 16 right-hand sides of one box to a wavefront
    ([44], 20),
]


@pytest.mark.parametrize("prec", ["fp32", "fp32_plain"])
@pytest.mark.parametrize("sides,nrhs", CASES)
def test_few_right_hand_sides(sides, nrhs, prec):
    print(f"case many columns {len(sides)} x {sides[0]} nrhs={nrhs} {prec}", flush=True)
    gt = api.Tree.build_grids([api.Grid(s, *W.grid_geometry(s)) for s in sides], device="cuda")
    gn = gt.neighbors()
    q = W.grid_rhs(gt.n, nrhs, seed=7).astype(np.complex64)
    gq = torch.as_tensor(q if nrhs > 1 else q[:, 0].copy(), device="cuda")
    rng = np.random.default_rng(8)
    tg = np.unique(np.concatenate([rng.choice(gt.n, 1500, replace=False), [0, 63, 64, gt.n - 64, gt.n - 1]]))
    gi = torch.as_tensor(tg, device="cuda")
    ref = oracle.helmholtz(sides, q, targets=tg)
    pick = lambda u: u[gi].cpu().numpy().reshape(len(tg), nrhs)
    assert _rel(pick(api.helmholtz(gt, gn, gq, prec=prec)), ref) <= TOL
    for grain in (1, 2):
        red = api.restructure(gt, gn, [gq], prec=prec, nrhs=nrhs, grain=grain)
        u = pick(api.helmholtz(gt, gn, None, layout="redundant", prec=prec, red=red))
        assert _rel(u, ref) <= TOL and max(_rel(u[:, r], ref[:, r]) for r in range(nrhs)) <= TOL
        del red
    conj = pick(api.helmholtz_adjoint(gt, gn, gq, prec=prec, conjugate=True))
    assert _rel(conj, np.conj(oracle.helmholtz(sides, np.conj(q), targets=tg))) <= TOL


def test_calls_of_two_threads():
    """One kernel, two threads and streams, right-hand sides whose tiles need more and less LDS: each call's result is
    that of a call by itself, bit for bit."""
    print("case two threads", flush=True)
    gt = api.Tree.build_grids([api.Grid(s, *W.grid_geometry(s)) for s in (52, 48, 12)], device="cuda")
    gn = gt.neighbors()
    jobs = []
    for nrhs in (7, 301):
        sides = (52, 48, 12) if nrhs == 7 else (16, 12)
        t = gt if nrhs == 7 else api.Tree.build_grids([api.Grid(s, *W.grid_geometry(s)) for s in sides], device="cuda")
        nb = gn if nrhs == 7 else t.neighbors()
        q = torch.as_tensor(W.grid_rhs(t.n, nrhs, seed=nrhs).astype(np.complex64), device="cuda")
        jobs.append((t, nb, q, api.helmholtz(t, nb, q, prec="fp32")))
    torch.cuda.synchronize()
    bad = []

    def work(t, nb, q, want):
        try:
            s = torch.cuda.Stream()
            with torch.cuda.stream(s):
                outs = [api.helmholtz(t, nb, q, prec="fp32") for _ in range(20)]
            s.synchronize()
            bad.extend(i for i, u in enumerate(outs) if not torch.equal(u, want))
        except Exception as e:   # reported by the test's own thread
            bad.append(e)

    threads = [threading.Thread(target=work, args=j) for j in jobs]
    for th in threads:
        th.start()
    for th in threads:
        th.join()
    assert not bad
