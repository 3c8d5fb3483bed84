"""The FP64 gravity adjoint against its definition in long double.  The relative
error was 5.3e-16 to 5.6e-16 (positions) and 3.7e-16 (masses) of these inputs
with a pair's terms formed as the kernel's comment writes them and every G-th
source to a lane group; a tenth more is allowed.  The inputs are seeded and the
kernel's order of sums is fixed, so the figures are the same in every run."""
import numpy as np
import pytest
import torch

from paper_2511_21535_amd import api
from paper_2511_21535_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("seed", [3, 4])
def test_adjoint_rounding(seed):
    n, cap, eps = 5000, 64, 1e-3
    print(f"case adjoint rounding seed={seed}", flush=True)
    p = W.plummer_mixture(n, seed)
    rng = np.random.default_rng(seed)
    g = [rng.standard_normal(n) for _ in range(4)]
    gp, gg = ([torch.as_tensor(v, device="cuda") for v in a] for a in (p, g))
    t = api.Tree.build_particles(*gp[:3], depth=20, leaf_cap=cap)
    nb = t.neighbors()
    out = [v.cpu().numpy() for v in api.gravity_adjoint(t, nb, eps, *gp, *gg)]
    ls, perm = t.leaf_start.cpu().numpy(), t.perm.cpu().numpy()
    ns, ni = nb.nbr_start.cpu().numpy(), nb.nbr_idx.cpu().numpy()
    x, m = [v.astype(np.longdouble) for v in p[:3]], p[3].astype(np.longdouble)
    g = [v.astype(np.longdouble) for v in g]
    err, ref = [0.0, 0.0], [0.0, 0.0]
    for A in range(t.n_leaves):
        tg = perm[ls[A]:ls[A + 1]]
        src = np.concatenate([perm[ls[B]:ls[B + 1]] for B in ni[ns[A]:ns[A + 1]]])
        d = [v[tg][:, None] - v[src][None] for v in x]
        w = 1 / np.sqrt(d[0] ** 2 + d[1] ** 2 + d[2] ** 2 + np.longdouble(eps) ** 2)
        w[tg[:, None] == src[None]] = 0
        w3 = w ** 3
        gj, gk = [v[tg][:, None] for v in g], [v[src][None] for v in g]
        mj, mk = m[tg][:, None], m[src][None]
        gdj, gdk = (sum(a[1 + k] * d[k] for k in range(3)) for a in (gj, gk))
        cc = mk * (gj[0] * w3 + 3 * w3 * w * w * gdj) + mj * (gk[0] * w3 - 3 * w3 * w * w * gdk)
        want = [(cc * d[k] + w3 * (mj * gk[1 + k] - mk * gj[1 + k])).sum(1) for k in range(3)]
        want.append((w3 * gdk - gk[0] * w).sum(1))
        for k in range(4):
            err[k == 3] += float(((out[k][tg] - want[k]) ** 2).sum())
            ref[k == 3] += float((want[k] ** 2).sum())
    rel = [(err[i] / ref[i]) ** 0.5 for i in range(2)]
    print(f"  positions {rel[0]:.3e} masses {rel[1]:.3e}", flush=True)
    assert rel[0] <= 1.1 * 5.6e-16 and rel[1] <= 1.1 * 3.7e-16
