"""The largest mechanism that loads, 127 species: its 128 state components
fill both slots of every lane.  Right-hand side against the oracle within
rounding of its largest terms (as for the smaller mechanisms) and Jacobian
against the oracle's complex steps, both reactors.  The bordered system has
one position more than the lanes hold rows: every solve is refused."""
import numpy as np
import pytest

from test_gpu_parity import gross_scale

pytestmark = pytest.mark.gpu

NS, NC = 127, 5


@pytest.fixture(scope="module")
def case():
    import torch  # noqa: F401  (its HIP runtime first)

    import paper_2311_14941_amd as sc
    from oracle.oracle import Oracle
    from synth.mechgen import make_mechanism
    sc.ensure_built()
    mech = make_mechanism(NS, 6 * NS, 76, 38, ["C", "H", "O", "N"], seed=400, pool_frac=0.15)
    rng = np.random.default_rng(NS)
    T, p = rng.uniform(1000.0, 2000.0, NC), 101325.0 * rng.uniform(1.0, 5.0, NC)
    return mech, Oracle(mech.to_text()), sc.Mechanism(mech.to_text()), T, p, rng.dirichlet(np.ones(NS), NC)


def gpu(*a):
    import torch
    return [torch.tensor(np.ascontiguousarray(x), device="cuda:0") for x in a]


def test_rhs(case):
    import paper_2311_14941_amd as sc
    mech, o, cm, T, p, Y = case
    fT, fY = sc.Plan(cm).rhs(*gpu(T, p, Y.T))
    fT, fY = fT.cpu().numpy(), fY.cpu().numpy().T
    for c in range(NC):
        f = o.rhs(np.append(Y[c], T[c]), p[c])
        sY, sT = gross_scale(o, mech, T[c], p[c], Y[c])
        assert (np.abs(fY[c] - f[:-1]) / (sY + 1e-300)).max() < 1e-12
        assert abs(fT[c] - f[-1]) / (sT + 1e-300) < 1e-12


@pytest.mark.parametrize("reactor", ["const_p", "const_v"])
def test_jacobian(case, reactor):
    import paper_2311_14941_amd as sc
    mech, o, cm, T, p, Y = case
    if reactor == "const_v":
        p = p / (8.314462618 * T * (Y / mech.molar_masses()).sum(1))  # densities
    J = sc.Plan(cm, reactor=reactor).jacobian(*gpu(T, p, Y.T)).cpu().numpy()
    for c in range(NC):
        ref = o.jac_cs(np.append(Y[c], T[c]), p[c], constv=reactor == "const_v")
        row = np.abs(ref).max(1, keepdims=True) + 1e-300
        assert (np.abs(J[c] - ref) / (1e-8 * np.abs(ref) + 1e-12 * row + 1e-20 * np.abs(ref).max())).max() <= 1.0


@pytest.mark.parametrize("mode", ["plain", "persistent", "static"])
def test_solves_are_refused(case, mode):
    import paper_2311_14941_amd as sc
    mech, o, cm, T, p, Y = case
    T, p, Y = gpu(T, p, Y.T)
    dt, b = gpu(np.full(NC, 1e-7), np.ones((NC, NS + 1)))
    plan = sc.Plan(cm, mode=mode)
    fuel, ox = np.zeros(NS), np.zeros(NS)
    fuel[0], ox[1] = 1.0, 1.0
    plan.set_mapping(fuel, ox, z_tol=0.1, dT=10.0)
    for call in (lambda: plan.linsolve(T, p, Y, dt, b), lambda: plan.integrate(T, p, Y, dt),
                 lambda: plan.integrate_noalloc(T, p, Y, dt), lambda: plan.integrate_mapped(T, p, Y, dt)):
        with pytest.raises(sc.StiffchemError) as e:
            call()
        assert e.value.code == sc.SC_EUNSUPPORTED and "126" in str(e.value)
    empty = plan.integrate(T[:0], p[:0], Y[:, :0], dt[:0])  # nothing to solve
    assert empty["T"].numel() == 0
