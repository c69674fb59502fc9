"""Several waves on one cell of the sparse kernels: a crew adds the reaction
passes in the order one wave takes them in, so its results are those of the
static launch (always one wave per cell), bit for bit.  Fewer cells than the
workgroup has waves, one more, several rounds of the queue and tiles whose rest
a crew takes over; one block of pivots, two, four and eight; both reactors; a
bad cell and one with nothing to do among them."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

# species, reactions, pool fraction, seed: positions N + 2 in blocks of 16
MECHS = {"n = 16": (14, 56, 0.15, 401), "n = 32": (30, 150, 0.3, 402), "n = 57": (55, 330, 0.15, 400),
         "n = 128": (126, 2500, 0.5, 4)}


@pytest.mark.parametrize("reactor", ["const_p", "const_v"])
@pytest.mark.parametrize("key", list(MECHS))
def test_crew_is_one_wave_bit_for_bit(key, reactor):
    import torch

    import paper_2311_14941_amd as sc
    from synth.mechgen import make_mechanism
    sc.ensure_built()
    ns, nr, pf, seed = MECHS[key]
    mech = sc.Mechanism(make_mechanism(ns, nr, nr // 10, nr // 20, ["C", "H", "O", "N"], seed=seed,
                                       pool_frac=pf).to_text())
    rng = np.random.default_rng(ns)
    nc = 23
    g = lambda a: torch.tensor(np.ascontiguousarray(a), device="cuda:0")
    T, p, Y = rng.uniform(1000.0, 2000.0, nc), 101325.0 * rng.uniform(1.0, 5.0, nc), rng.dirichlet(np.ones(ns), nc)
    dt = 10.0 ** rng.uniform(-9.0, -6.0, nc)
    if reactor == "const_v":
        p = p / 4e5  # densities
    dt[4], T[7] = 0.0, np.nan
    T, p, Y, dt = g(T), g(p), g(Y.T), g(dt)
    kw = dict(linalg="sparse", cells_per_wave=1, reactor=reactor, max_steps=300)
    for n in (1, 3, 5, nc):
        a = (T[:n].clone(), p[:n].clone(), Y[:, :n].contiguous(), dt[:n].clone())
        ref = sc.Plan(mech, mode="static", **kw).integrate(*a)
        keep = torch.arange(n, device="cuda:0") != 7
        for cfg in (dict(mode="plain"), dict(mode="persistent", grid=1), dict(mode="persistent", grid=2, tile=3),
                    dict(mode="persistent", order="dt")):
            r = sc.Plan(mech, **cfg, **kw).integrate(*a)
            assert torch.equal(r["status"], ref["status"]), (n, cfg)
            for k in ("T", "n_acc", "n_rej"):
                assert torch.equal(r[k][keep], ref[k][keep]), (n, cfg, k)
            assert torch.equal(r["Y"][:, keep], ref["Y"][:, keep]), (n, cfg)
