"""Helmholtz at the edges of the operands' range, each part of the result by
itself: real and imaginary part of very different size, magnitudes near both
ends of single precision, infinities.  The reference is the definition in numpy
(long double, or the stated set of non-finite targets).

Tolerances.  A part sums at most 2 x 1728 products in the working precision, in
any order, of operands rounded once: within (3456 + 4) u of the sum of the
products' magnitudes, u the unit roundoff."""
import numpy as np
import pytest
import torch

from paper_2511_21535_amd import api

pytestmark = pytest.mark.gpu

DEV = "cuda"
PI = np.longdouble("3.14159265358979323846264338327950288")
U = {"fp64": 2.0 ** -53, "fp32": 2.0 ** -24, "fp32_plain": 2.0 ** -24}


def _grid(side, kh):
    """A grid of spacing 1, so that u is not scaled."""
    t = api.Tree.build_grids([api.Grid(side, 1.0, kh)], device=DEV)
    return t, t.neighbors()


def _sum(side, kh, q, targets, conj=False):
    """(u, sum of |terms|), each as real and imaginary part, at the targets; q complex or real, [n, nrhs]."""
    ijk = np.stack([np.arange(side ** 3) % side, np.arange(side ** 3) // side % side, np.arange(side ** 3) // side ** 2], 1)
    qr, qi = q.real.astype(np.longdouble), q.imag.astype(np.longdouble)
    out = []
    for i in targets:
        near = np.all(np.abs(ijk // 4 - ijk[i] // 4) <= 1, axis=1)
        near[i] = False
        d = np.sqrt((((ijk[near] - ijk[i]) ** 2).sum(1)).astype(np.longdouble))
        a = 1 / (4 * PI * d)
        gr, gi = (a * np.cos(kh * d))[:, None], (a * np.sin(kh * d) * (-1 if conj else 1))[:, None]
        x, y = qr[near], qi[near]
        out.append(((gr * x - gi * y).sum(0), (gr * y + gi * x).sum(0),
                    (abs(gr * x) + abs(gi * y)).sum(0), (abs(gr * y) + abs(gi * x)).sum(0)))
    return [np.stack([o[k] for o in out]) for k in range(4)]


def _check(u, ref, prec, floor=0.0):
    tol = (2 * 1728 + 4) * U[prec]
    for got, want, size in ((u.real, ref[0], ref[2]), (u.imag, ref[1], ref[3])):
        err = np.abs(got.astype(np.longdouble) - want)
        assert np.all(err <= tol * size + floor), float((err / (size + 1e-4000)).max())


def _targets(side):
    return np.unique(np.concatenate([np.arange(0, side ** 3, 61), [side ** 3 - 1]]))


@pytest.mark.parametrize("nrhs", [2, 8, 17])
@pytest.mark.parametrize("kh", [0.6, 1e-4, 1e-8])
def test_fp64_parts_of_unequal_size(kh, nrhs):
    """Real q and a small kh: Im u is kh times smaller than Re u, and as accurate."""
    side = 12
    print(f"case fp64 parts kh={kh} nrhs={nrhs}", flush=True)
    t, nb = _grid(side, kh)
    rng = np.random.default_rng(nrhs)
    tg = _targets(side)
    for q in (rng.standard_normal((side ** 3, nrhs)) + 0j, 1j * rng.standard_normal((side ** 3, nrhs))):
        gq = torch.as_tensor(q, device=DEV)
        red = api.restructure(t, nb, [gq], prec="fp64", nrhs=nrhs)
        for u in (api.helmholtz(t, nb, gq, prec="fp64"),
                  api.helmholtz(t, nb, None, layout="redundant", prec="fp64", red=red)):
            _check(u.cpu().numpy()[tg], _sum(side, kh, q, tg), "fp64")
        _check(api.helmholtz_adjoint(t, nb, gq, prec="fp64", conjugate=True).cpu().numpy()[tg],
               _sum(side, kh, q, tg, conj=True), "fp64")


def _near(side, i):
    ijk = np.stack([np.arange(side ** 3) % side, np.arange(side ** 3) // side % side, np.arange(side ** 3) // side ** 2], 1)
    near = np.all(np.abs(ijk // 4 - ijk[i] // 4) <= 1, axis=1)
    return near


@pytest.mark.parametrize("nrhs", [2, 32])
def test_fp64_infinity_stays_an_infinity(nrhs):
    """An infinite real part of one source: Re and Im of every other target it reaches are infinite, none NaN (G of the
    point itself is zero), and targets of other boxes and columns are untouched."""
    side, i = 16, 77
    print(f"case fp64 infinity nrhs={nrhs}", flush=True)
    t, nb = _grid(side, 0.6)
    q = torch.randn(side ** 3, nrhs, dtype=torch.float64, device=DEV).to(torch.complex128)
    q[i, 0] = complex(float("inf"), 0.0)
    u = torch.view_as_real(api.helmholtz(t, nb, q, prec="fp64")).cpu().numpy()
    near = _near(side, i)
    other = near.copy()
    other[i] = False
    assert np.all(np.isinf(u[other, 0])) and np.all(np.isnan(u[i, 0]))
    assert np.all(np.isfinite(u[~near])) and np.all(np.isfinite(u[:, 1:]))


@pytest.mark.parametrize("prec,nrhs,kh,dk", [("fp64", 2, 40.0, 9e-13), ("fp32", 3, 3e7, 9e-13)])
def test_media_that_differ_little(prec, nrhs, kh, dk):
    """Two grids whose k h differ by less than 1e-12: each gets its own phases, as accurate as alone (the same bits)."""
    print(f"case two media {prec} kh={kh}", flush=True)
    side, khs = 8, (kh, kh * (1 + dk))
    q = torch.randn(2 * side ** 3, nrhs, dtype=torch.complex128 if prec == "fp64" else torch.complex64, device=DEV)
    both = api.Tree.build_grids([api.Grid(side, 1.0, k) for k in khs], device=DEV)
    u = api.helmholtz(both, both.neighbors(), q, prec=prec)
    for g, k in enumerate(khs):
        t, nb = _grid(side, k)
        part = slice(g * side ** 3, (g + 1) * side ** 3)
        assert torch.equal(u[part], api.helmholtz(t, nb, q[part].contiguous(), prec=prec))


@pytest.mark.parametrize("nrhs,tile", [(32, (4, 1, 32, 1)), (32, (2, 1, 32, 1)), (911, None)])
def test_single_precision_sums_of_many_columns(nrhs, tile):
    """prec "fp32_plain" keeps its sums in single precision: at most 24 roundings within an offset and 27 between them,
    1.7e-7 of a sum of random terms as independent roundings; half as much again is allowed."""
    side = 12
    print(f"case plain sums nrhs={nrhs} tile={tile}", flush=True)
    t, nb = _grid(side, 0.6)
    rng = np.random.default_rng(nrhs)
    q = (rng.standard_normal((side ** 3, nrhs)) + 1j * rng.standard_normal((side ** 3, nrhs))).astype(np.complex64)
    tg = _targets(side)
    ref = _sum(side, 0.6, q, tg)
    u = api.helmholtz(t, nb, torch.as_tensor(q, device=DEV), prec="fp32_plain", tile=tile).cpu().numpy()[tg]
    for got, want in ((u.real, ref[0]), (u.imag, ref[1])):
        assert float(np.linalg.norm((got - want).astype(np.float64)) / np.linalg.norm(want.astype(np.float64))) <= 2.6e-7


# single precision: few columns (one right-hand side, several, tiles shared and not), many columns by a launch shape
# (16 right-hand sides of one box to a wavefront) and by their number (3 right-hand sides do not divide by 16)
SINGLE = [(16, 1, None), (16, 3, None), (12, 33, None), (12, 32, (4, 1, 32, 1)), (12, 64, (2, 1, 64, 1)), (12, 911, None)]


def _close(u, ref, side):
    """Relative 2.6e-7 (see above) beside the roundings at the subnormal spacing, 2^-150 each, 2 x 1728 a part."""
    for got, want in ((u.real, ref[0]), (u.imag, ref[1])):
        err = np.linalg.norm((got.astype(np.longdouble) - want))
        assert err <= 2.6e-7 * np.linalg.norm(want) + (2 * 1728 * want.size) ** 0.5 * 2.0 ** -150, float(err / np.linalg.norm(want))


@pytest.mark.parametrize("side,nrhs,tile", SINGLE)
@pytest.mark.parametrize("prec", ["fp32", "fp32_plain"])
def test_small_and_large_magnitudes(side, nrhs, tile, prec):
    t, nb = _grid(side, 0.6)
    cols = np.unique(np.linspace(0, nrhs - 1, 24).astype(int))    # compared; nrhs // 2 among them
    cols = np.union1d(cols, [nrhs // 2])
    rng = np.random.default_rng(nrhs)
    base = rng.standard_normal((side ** 3, nrhs)) + 1j * rng.standard_normal((side ** 3, nrhs))
    tg = _targets(side)
    ramp = 2.0 ** -(np.arange(side ** 3) // side ** 2 * (150.0 / side))[:, None]      # 1 to 2^-150 across the grid
    huge = np.ones((side ** 3, nrhs))
    huge[side ** 3 // 2, nrhs // 2] = 3.4e38 / abs(base[side ** 3 // 2, nrhs // 2])   # rounds up in BF16
    for name, scale in [("2^-%d" % e, 2.0 ** -e) for e in (100, 108, 114, 120, 126, 136)] + [("ramp", ramp), ("huge", huge)]:
        print(f"case magnitudes side={side} nrhs={nrhs} tile={tile} {prec} {name}", flush=True)
        q = (base * scale).astype(np.complex64)
        gq = torch.as_tensor(q if nrhs > 1 else q[:, 0].copy(), device=DEV)
        ref = _sum(side, 0.6, q[:, cols], tg)
        red = api.restructure(t, nb, [gq], prec=prec, nrhs=nrhs)
        for u in (api.helmholtz(t, nb, gq, prec=prec, tile=tile),
                  api.helmholtz(t, nb, None, layout="redundant", prec=prec, red=red, tile=tile)):
            u = u.cpu().numpy().reshape(side ** 3, nrhs)[tg][:, cols]
            _close(u, ref, side)
            if name == "ramp":   # the targets far below the largest source, by themselves
                for z in range(0, side, 4):
                    low = (tg // side ** 2) // 4 == z // 4
                    _close(u[low], [r[low] for r in ref], side)
        if tile is None:
            u = api.helmholtz_adjoint(t, nb, gq, prec=prec, conjugate=True).cpu().numpy().reshape(side ** 3, nrhs)[tg]
            _close(u[:, cols], _sum(side, 0.6, q[:, cols], tg, conj=True), side)


@pytest.mark.parametrize("side,nrhs,tile", SINGLE)
def test_single_precision_infinity_stays_an_infinity(side, nrhs, tile):
    print(f"case fp32 infinity side={side} nrhs={nrhs} tile={tile}", flush=True)
    t, nb = _grid(side, 0.6)
    i = 77
    q = torch.view_as_complex(torch.randn(side ** 3, nrhs, 2, device=DEV))
    q[i, 0] = complex(float("inf"), 0.0)
    u = api.helmholtz(t, nb, q if nrhs > 1 else q[:, 0].contiguous(), prec="fp32", tile=tile)
    u = torch.view_as_real(u).reshape(side ** 3, nrhs, 2).cpu().numpy()
    near = _near(side, i)
    other = near.copy()
    other[i] = False
    assert np.all(np.isinf(u[other, 0])) and np.all(np.isnan(u[i, 0]))
    assert np.all(np.isfinite(u[~near])) and np.all(np.isfinite(u[:, 1:]))


@pytest.mark.parametrize("side,nrhs,tile", SINGLE)
def test_single_precision_tiny_kh(side, nrhs, tile):
    """Im G of about 1e-34: real q, each part of u as accurate as the other."""
    print(f"case fp32 tiny kh side={side} nrhs={nrhs} tile={tile}", flush=True)
    t, nb = _grid(side, 1e-33)
    q = np.random.default_rng(nrhs).standard_normal((side ** 3, nrhs)).astype(np.complex64)
    tg = _targets(side)
    u = api.helmholtz(t, nb, torch.as_tensor(q if nrhs > 1 else q[:, 0].copy(), device=DEV), prec="fp32", tile=tile)
    cols = np.unique(np.linspace(0, nrhs - 1, 24).astype(int))
    _close(u.cpu().numpy().reshape(side ** 3, nrhs)[tg][:, cols], _sum(side, 1e-33, q[:, cols], tg), side)
