"""Calls of more cells than a launch's 2^32 threads hold a wave each (2^26):
9 species, 2^26 + 5 cells, every entry point that takes a workgroup per cell,
dense and sparse (one cell per wave).  The first and last cells and those
around the parts' ends are as in small calls, bit for bit.  The transport step,
a thread per cell, with 2^32 and more."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

N_CELLS = 2 ** 26 + 5


@pytest.fixture(scope="module")
def case():
    import torch

    import paper_2311_14941_amd as sc
    from synth.mechgen import standard_mechanism
    sc.ensure_built()
    mech = sc.Mechanism(standard_mechanism("h2_9").to_text())
    k = torch.arange(N_CELLS, device="cuda:0")
    d = dict(dtype=torch.float64, device="cuda:0")
    T = 1000.0 + (k % 997).to(torch.float64)
    p, Y = torch.full((N_CELLS,), 2e5, **d), torch.full((mech.N, N_CELLS), 1.0 / mech.N, **d)
    near = [i for c in (0, 2 ** 24, 2 ** 25, 2 ** 26, N_CELLS) for i in range(max(c - 3, 0), min(c + 3, N_CELLS))]
    return mech, T, p, Y, torch.tensor(sorted(set(near)), device="cuda:0")


@pytest.mark.parametrize("linalg", ["dense", "sparse"])
def test_single_passes(case, linalg):
    import torch

    import paper_2311_14941_amd as sc
    mech, T, p, Y, i = case
    plan = sc.Plan(mech, linalg=linalg, cells_per_wave=0 if linalg == "dense" else 1)
    small = (T[i], p[i], Y[:, i].contiguous())
    fT, fY = plan.rhs(T, p, Y)
    sT, sY = plan.rhs(*small)
    assert torch.equal(fT[i], sT) and torch.equal(fY[:, i], sY)
    del fT, fY
    J = plan.jacobian(T, p, Y)
    assert torch.equal(J[i], plan.jacobian(*small))
    del J
    hg, b = torch.full_like(T, 1e-8), torch.ones((N_CELLS, mech.N + 1), dtype=torch.float64, device="cuda:0")
    b[:, 0] = T
    x = plan.linsolve(T, p, Y, hg, b)
    assert torch.equal(x[i], plan.linsolve(*small, hg[i], b[i]))
    del x, b
    if linalg == "dense":
        g = plan.vjp(T, p, Y, T, Y, per_cell=True)
        s = plan.vjp(*small, T[i], Y[:, i].contiguous(), per_cell=True)
        assert all(torch.equal(u[..., i], v) for u, v in zip(g, s))


@pytest.mark.parametrize("mode", ["plain", "static", "persistent"])
@pytest.mark.parametrize("linalg", ["dense", "sparse"])
def test_integration(case, linalg, mode):
    """Every cell has nothing to do but those compared; workgroups as many as
    cells where the option says so."""
    import torch

    import paper_2311_14941_amd as sc
    mech, T, p, Y, i = case
    dt = torch.zeros_like(T)
    dt[i] = 1e-8
    kw = dict(linalg=linalg, cells_per_wave=0 if linalg == "dense" else 1, rtol=1e-4, atol=1e-10)
    out = sc.Plan(mech, mode=mode, grid=0 if mode == "plain" else 2 ** 31 - 1, **kw).integrate(T, p, Y, dt)
    ref = sc.Plan(mech, mode="static", **kw).integrate(T[i], p[i], Y[:, i].contiguous(), dt[i])
    assert int(ref["n_acc"].min()) > 0
    for k in ("status", "T", "Y", "n_acc", "n_rej"):
        assert torch.equal(out[k][..., i], ref[k]), k
    assert int((out["n_acc"] > 0).sum()) == i.numel()
    assert torch.equal(out["T"][dt == 0.0], T[dt == 0.0]) and int(out["status"].max()) == 0


def test_transport():
    """The last rows of a grid of 65,536 x 65,537 cells are those of the same
    rows by themselves (their south row is not compared: it is a boundary
    there)."""
    import torch

    import paper_2311_14941_amd as sc
    sc.ensure_built()
    nx, ny, part = 65536, 65537, 5
    d = dict(dtype=torch.float64, device="cuda:0")
    q, u, dt = torch.full((1, nx * ny), 0.25, **d), torch.full((nx * ny,), 3.0, **d), torch.full((nx * ny,), 1e-4, **d)
    tail = slice(nx * (ny - part), None)
    q[0, tail] = torch.rand(nx * part, **d)
    inflow = torch.rand((1, ny), **d)
    out = sc.transport2d(nx, ny, q, u, dt, 1e-3, 2e-4, inflow)
    ref = sc.transport2d(nx, part, q[:, tail].contiguous(), u[tail].clone(), dt[tail].clone(), 1e-3, 2e-4,
                         inflow[:, ny - part:].contiguous())
    assert torch.equal(out[0, nx * (ny - part + 1):], ref[0, nx:])
    first = slice(0, nx)  # a row of 0.25 within rows of 0.25, its inflow apart
    assert torch.equal(out[0, first][2:], q[0, first][2:])
