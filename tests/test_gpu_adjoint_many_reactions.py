"""The adjoint keeps one double per reaction in LDS beside the dense kernels'
layout: 15 species leave room for 18,592 reactions.  The mechanism is one of 56
reactions with 331 copies of each at a rate constant of 1e-290: the integration
and its gradients are those of the 56.  Steps are fixed; what differs is the
order of sums of rates, 1e-16 of the gross rates per sum, over 4 steps: 1e-9 of
each gradient's largest entry has a margin of more than a thousand."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

COPIES = 332


def test_gradient_of_18592_reactions():
    import copy

    import torch

    import paper_2311_14941_amd as sc
    from synth.mechgen import make_mechanism
    sc.ensure_built()
    base = make_mechanism(15, 56, 6, 3, ["C", "H", "O", "N"], seed=401, pool_frac=0.15)
    many = copy.deepcopy(base)
    many.reactions = []
    for r in base.reactions:
        none = copy.deepcopy(r)
        none.log10A = -290.0
        if none.kind == "troe":
            none.troe = (-290.0, *none.troe[1:])
        many.reactions += [r] + [none] * (COPIES - 1)
    rng = np.random.default_rng(15)
    nc, N = 3, base.n_species
    g = lambda a: torch.tensor(np.ascontiguousarray(a), device="cuda:0")
    T, p, Y = g(rng.uniform(1000.0, 2000.0, nc)), g(101325.0 * rng.uniform(1.0, 5.0, nc)), g(rng.dirichlet(np.ones(N), nc).T)
    dt = torch.full((nc,), 1e-10, dtype=torch.float64, device="cuda:0")
    gT, gY = g(rng.normal(size=nc)), g(rng.normal(size=(N, nc)))
    out = []
    for mech in (base, many):
        plan = sc.Plan(sc.Mechanism(mech.to_text()), linalg="dense", fixed_step=True)
        out.append(plan.adjoint(T, p, Y, dt, gT, gY, h=dt / 4, per_cell=True, forward_out=True))
    a, b = out
    # (a random mixture may run away: such a cell has its status and no gradient)
    ok = a["status"] == sc.CELL_OK
    assert torch.equal(a["status"], b["status"]) and int(ok.sum()) > 0, a["status"]
    b["g_dlnA_cell"] = b["g_dlnA_cell"].reshape(-1, COPIES, nc)[:, 0]
    for k in ("T", "Y", "gT0", "gY0", "g_dlnA_cell"):
        u, v = a[k][..., ok], b[k][..., ok]
        assert float((u - v).abs().max()) <= 1e-9 * float(u.abs().max()), k
