"""The sparse kernels' factorisation and solves at the edges of their parts:
rows in registers (two and four cells per wave); blocks of 16 pivots with one
state component per lane, the last one partly filled (n = 26, 57) and full
(64), and with two (n = 65, 112 and 128: a block of one pivot, full ones and
the largest).  The dense kernels' blocks of 16 rows likewise: N + 1 = 16 rows
(one full block), 17, 32 and 33 (one row into the next size), 56 (the last
block half), 57 and 64.  The solution of (I/hg - J) x = b is checked against the matrix
from the oracle's complex-step Jacobian by its normwise backward error.  An
unpivoted LU of a matrix whose diagonal dominates (small hg) has growth near
one, so the bound is the usual n eps with a margin of about ten for the
Jacobian's own rounding: 1e-12 holds up to n = 128."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

# species, reactions, pool fraction, seed, cells per wave: positions N + 2
MECHS = {
    "4 cells, n = 16": (14, 56, 0.15, 401, 4),
    "2 cells, n = 32": (30, 150, 0.3, 402, 2),
    "1 cell, n = 26": (24, 120, 0.5, 400, 1),
    "n = 57": (55, 330, 0.15, 400, 1),
    "n = 64": (62, 900, 0.6, 1, 1),
    "n = 65": (63, 400, 0.15, 400, 1),
    "n = 112": (110, 700, 0.15, 110, 1),
    "n = 128": (126, 2500, 0.5, 4, 1),
}


# the dense kernels: rows N + 1
DENSE = [(15, 60, 0.15, 400), (16, 60, 0.15, 400), (31, 150, 0.3, 400), (32, 170, 0.3, 400), (55, 330, 0.15, 400),
         (56, 340, 0.15, 400), (63, 400, 0.15, 400)]


def _backward_error(ns, nr, pf, seed, **kw):
    import torch

    import paper_2311_14941_amd as sc
    from oracle.oracle import Oracle
    from synth.mechgen import make_mechanism
    sc.ensure_built()
    mech = make_mechanism(ns, nr, nr // 10, nr // 20, ["C", "H", "O", "N"], seed=seed, pool_frac=pf)
    o = Oracle(mech.to_text())
    plan = sc.Plan(sc.Mechanism(mech.to_text()), **kw)
    rng = np.random.default_rng(ns)
    nc = 7
    T, p = rng.uniform(1000.0, 2000.0, nc), 101325.0 * rng.uniform(1.0, 5.0, nc)
    Y = rng.dirichlet(np.ones(ns), nc)
    b = rng.normal(size=(nc, ns + 1))
    J = [o.jac_cs(np.append(Y[c], T[c]), p[c]) for c in range(nc)]
    # every state's own scale: the diagonal exceeds its Jacobian's row sums
    hg = np.array([0.25 / np.abs(j).sum(1).max() for j in J])
    g = lambda a: torch.tensor(np.ascontiguousarray(a), device="cuda:0")
    x = plan.linsolve(g(T), g(p), g(Y.T), g(hg), g(b)).cpu().numpy()
    for c in range(nc):
        M = np.eye(ns + 1) / hg[c] - J[c]
        res = np.abs(M @ x[c] - b[c]).max() / (np.abs(M).max() * np.abs(x[c]).max() + np.abs(b[c]).max())
        assert res < 1e-12, (ns, c, res)


@pytest.mark.parametrize("key", list(MECHS))
def test_linsolve_backward_error(key):
    *mech, cpw = MECHS[key]
    _backward_error(*mech, linalg="sparse", cells_per_wave=cpw)


@pytest.mark.parametrize("mech", DENSE, ids=lambda m: str(m[0] + 1))
def test_dense_linsolve_backward_error(mech):
    _backward_error(*mech, linalg="dense")
