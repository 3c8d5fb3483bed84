"""Helmholtz with (target box, right-hand side) pairs as the columns of the
matrix-core product, against the FP64 oracle: right-hand-side counts around the
16-column tile and that leave a partial last tile, instances of one box, tiles
shared by two workgroups (few columns) and not (many), several G tables, and
more than 8 instances (uploaded parameters); and the single-precision product
for many columns; in both layouts and grains and both directions.  Tolerances are the project's: 1e-5 (FP32) and 1e-12 (FP64)."""
import numpy as np
import pytest
import torch

import oracle
from paper_2511_21535_amd import api
from paper_2511_21535_amd import workloads as W

pytestmark = pytest.mark.gpu

TOL = {"fp64": 1e-12, "fp32": 1e-5, "fp32_plain": 1e-5}
DEV = "cuda"


def _rel(a, b):
    a, b = np.asarray(a).ravel(), np.asarray(b).ravel()
    return float(np.linalg.norm(a - b) / np.linalg.norm(b))


CASES = [
    # sides, points per wavelength, nrhs
    ([4], [10], 2),
    ([8, 4], [10, 6], 15),
    ([8], [10], 16),
    ([12], [10], 17),
    ([12, 8, 4], [10, 6, 10], 31),
    ([16], [10], 33),                       # 2112 columns: one workgroup per tile
    ([8] * 5 + [4] * 5, [10, 6] * 5, 5),    # 10 instances: uploaded parameters
    # single precision: half tiles shared by four workgroups (up to 32 tiles), by
    # two (up to 64) and not, one right-hand side and several
    ([16], [10], 1),
    ([48], [10], 1),
    ([32], [10], 2),                        # FP64: 64 tiles, four workgroups each
    ([24], [10], 3),                        # FP64: 41 tiles, four; 36 and 37 tiles below: seven and four
    ([12, 24], [10, 6], 2),
    ([8, 20], [10, 10], 4),
    ([8], [10], 72),
    ([8], [10], 74),
    ([32], [10], 3),
    ([32], [10], 4),
    ([32], [10], 5),
]

# single precision with columns enough for the product that stages G in LDS: 16
# right-hand sides of one box per wavefront and not, a partial last tile per
# instance, two tables, uploaded parameters
MANY = [
    ([16, 12], [10, 6], 272),
    ([16, 12], [10, 10], 301),
    ([8] * 5 + [4] * 5, [10, 6] * 5, 560),
]


@pytest.mark.parametrize("sides,ppw,nrhs,prec", [(*c, p) for c in CASES for p in ("fp64", "fp32", "fp32_plain")] +
                         [(*c, p) for c in MANY for p in ("fp32", "fp32_plain")])
def test_columns_parity(sides, ppw, nrhs, prec):
    print(f"case columns sides={sides} nrhs={nrhs} prec={prec}", flush=True)
    h = np.array([1.0 / n for n in sides])
    kw = np.array([2 * np.pi / (p * hh) for p, hh in zip(ppw, h)])
    gt = api.Tree.build_grids([api.Grid(int(n), float(a), float(k)) for n, a, k in zip(sides, h, kw)], device=DEV)
    gn = gt.neighbors()
    cd = np.complex128 if prec == "fp64" else np.complex64
    q = W.grid_rhs(gt.n, nrhs, seed=81).astype(cd)
    gq = torch.as_tensor(q, device=DEV)
    ref = oracle.helmholtz(sides, q, h=h, kw=kw).reshape(q.shape)
    got = {"gather": api.helmholtz(gt, gn, gq, prec=prec)}
    for grain in (1, 2):
        red = api.restructure(gt, gn, [gq], prec=prec, nrhs=nrhs, grain=grain)
        got[f"redundant, grain {grain}"] = api.helmholtz(gt, gn, None, layout="redundant", prec=prec, red=red)
    for name, u in got.items():
        u = u.cpu().numpy().reshape(q.shape)
        err, col = _rel(u, ref), max(_rel(u[:, r], ref[:, r]) for r in range(nrhs))
        print(f"  {name}: {err:.2e} (worst column {col:.2e})", flush=True)
        assert err <= TOL[prec] and col <= TOL[prec]
    conj = api.helmholtz_adjoint(gt, gn, gq, prec=prec, conjugate=True).cpu().numpy()
    assert _rel(conj, np.conj(oracle.helmholtz(sides, np.conj(q), h=h, kw=kw))) <= TOL[prec]
