"""Workgroups of one, two and four waves of the sparse kernels, chosen by the
cells in flight: 57 species (one slot per lane) hold one workgroup of four waves
a CU, three of two or seven of one, 65 species (two slots) two crews of two or
four single waves.  Cells just within and beyond each choice on 256 CUs, queues
of one tile and of several and, of one-wave workgroups, a single one, integrate
bit for bit as the static launch; linear solves of a batch large enough for one
wave a cell as those of a small one."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", params=[57, 65])
def case(request):
    import torch

    import paper_2311_14941_amd as sc
    from synth.mechgen import make_mechanism
    sc.ensure_built()
    ns, nc = request.param, 2003
    mech = sc.Mechanism(make_mechanism(ns, 6 * ns, 6 * ns // 10, 6 * ns // 20, ["C", "H", "O", "N"], seed=400,
                                       pool_frac=0.15).to_text())
    rng = np.random.default_rng(ns)
    g = lambda a: torch.tensor(np.ascontiguousarray(a), device="cuda:0")
    T, p, Y = rng.uniform(1000.0, 2000.0, nc), 101325.0 * rng.uniform(1.0, 5.0, nc), rng.dirichlet(np.ones(ns), nc)
    dt = 10.0 ** rng.uniform(-9.0, -7.5, nc)
    dt[4], T[7] = 0.0, np.nan
    return mech, g(T), g(p), g(Y.T), g(dt)


def test_integration_is_the_static_launch(case):
    import torch

    import paper_2311_14941_amd as sc
    mech, T, p, Y, dt = case
    kw = dict(linalg="sparse", rtol=1e-4, atol=1e-10, max_steps=300)
    ref = sc.Plan(mech, mode="static", **kw).integrate(T, p, Y, dt)
    for n, cfg in ((1, dict(mode="persistent")), (300, dict(mode="persistent")), (1024, dict(mode="persistent")),
                   (1025, dict(mode="persistent")), (1200, dict(mode="plain")), (2003, dict(mode="plain")),
                   (2003, dict(mode="persistent")), (2003, dict(mode="persistent", tile=3, order="dt")),
                   (37, dict(mode="persistent", grid=1))):
        r = sc.Plan(mech, **cfg, **kw).integrate(T[:n].clone(), p[:n].clone(), Y[:, :n].contiguous(), dt[:n].clone())
        keep = torch.arange(n, device="cuda:0") != 7
        assert torch.equal(r["status"], ref["status"][:n]), (n, cfg)
        for k in ("T", "n_acc", "n_rej"):
            assert torch.equal(r[k][keep], ref[k][:n][keep]), (n, cfg, k)
        assert torch.equal(r["Y"][:, keep], ref["Y"][:, :n][:, keep]), (n, cfg)


def test_linear_solves_of_large_batches(case):
    import torch

    import paper_2311_14941_amd as sc
    mech, T, p, Y, dt = case
    plan = sc.Plan(mech, linalg="sparse")
    n = T.numel()
    hg = torch.full((n,), 1e-8, dtype=torch.float64, device="cuda:0")
    b = torch.rand((n, mech.N + 1), dtype=torch.float64, device="cuda:0")
    keep = torch.arange(n, device="cuda:0") != 7
    x = plan.linsolve(T, p, Y, hg, b)
    for a in range(0, n, 401):
        e = min(a + 401, n)
        part = plan.linsolve(T[a:e].clone(), p[a:e].clone(), Y[:, a:e].contiguous(), hg[a:e].clone(), b[a:e].clone())
        assert torch.equal(part[keep[a:e]], x[a:e][keep[a:e]])


def test_linear_solves_of_more_cells_than_a_launch_has_crews():
    """Crews of two (90 species) of 2^25 + 5 cells would be 2^32 threads and
    more: the parts' first and last cells solve as in a small call."""
    import torch

    import paper_2311_14941_amd as sc
    from synth.mechgen import make_mechanism
    sc.ensure_built()
    ns, n = 90, 2 ** 25 + 5
    mech = sc.Mechanism(make_mechanism(ns, 6 * ns, 54, 27, ["C", "H", "O", "N"], seed=400, pool_frac=0.15).to_text())
    d = dict(dtype=torch.float64, device="cuda:0")
    k = torch.arange(n, device="cuda:0")
    T = 1000.0 + (k % 997).to(torch.float64)
    p, hg = torch.full((n,), 2e5, **d), torch.full((n,), 1e-8, **d)
    Y = torch.full((ns, n), 1.0 / ns, **d)
    b = torch.ones((n, ns + 1), **d)
    b[:, 0] = 1.0 + (k % 991).to(torch.float64)
    plan = sc.Plan(mech, linalg="sparse")
    x = plan.linsolve(T, p, Y, hg, b)
    for c in (0, 2 ** 24, 2 ** 25, n):
        i = torch.arange(max(c - 4, 0), min(c + 4, n), device="cuda:0")
        part = plan.linsolve(T[i], p[i], Y[:, i].contiguous(), hg[i], b[i])
        assert torch.equal(part, x[i]), c


@pytest.mark.parametrize("ns,copies", [(57, 13), (65, 11)])
def test_more_reaction_passes_than_a_crew_keeps_in_a_word(ns, copies):
    """More than 64 passes of 64 reactions: a crew's waves find their passes by
    the rule instead of the word they keep.  Copies of every reaction, the
    added ones at a rate constant of 1e-290; bit for bit the static launch."""
    import copy

    import torch

    import paper_2311_14941_amd as sc
    from synth.mechgen import make_mechanism
    sc.ensure_built()
    mech = make_mechanism(ns, 6 * ns, 6 * ns // 10, 6 * ns // 20, ["C", "H", "O", "N"], seed=400, pool_frac=0.15)
    base, mech.reactions = mech.reactions, []
    for r in base:
        none = copy.deepcopy(r)
        none.log10A = -290.0
        if none.kind == "troe":
            none.troe = (-290.0, *none.troe[1:])
        mech.reactions += [r] + [none] * (copies - 1)
    assert len(mech.reactions) > 4096
    rng = np.random.default_rng(ns)
    g = lambda a: torch.tensor(np.ascontiguousarray(a), device="cuda:0")
    n = 9
    a = (g(rng.uniform(1000.0, 2000.0, n)), g(101325.0 * rng.uniform(1.0, 5.0, n)), g(rng.dirichlet(np.ones(ns), n).T),
         g(10.0 ** rng.uniform(-10.0, -9.0, n)))
    m = sc.Mechanism(mech.to_text())
    kw = dict(linalg="sparse", rtol=1e-4, atol=1e-10, max_steps=300)
    ref = sc.Plan(m, mode="static", **kw).integrate(*a)
    for cfg in (dict(mode="plain"), dict(mode="persistent"), dict(mode="persistent", grid=1)):
        r = sc.Plan(m, **cfg, **kw).integrate(*a)
        for k in ("status", "T", "Y", "n_acc", "n_rej"):
            assert torch.equal(r[k], ref[k]), (cfg, k)
