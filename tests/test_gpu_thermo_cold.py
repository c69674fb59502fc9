"""Interpolated thermodynamics where 1/K_c is at the largest double: A = B + C
with dG/RT = 712 at 200 K, so exp(712) overflows and the reaction's
exp(dG/RT - ln(p0/RT)) does not.  The lanes behind the last reaction of a pass
have no reaction and no share in the result: the Jacobian is finite and the
exact plan's (its K_c differs by the tables' error, 1e-9 relative, so 1e-7 of
each row's largest entry has a margin of a hundred)."""
import pytest

pytestmark = pytest.mark.gpu

MECH = """STIFFCHEM-MECH 1
NAME cold
GAS_CONSTANT 8.314462618
REF_PRESSURE 101325.0
ELEMENTS 1 X
SPECIES 3
SP A 0.028 2
SP B 0.014 1
SP C 0.014 1
NASA7 A 5.0 0 0 0 0 0 0
NASA7 B 2.5 0 0 0 0 142400.0 0
NASA7 C 2.5 0 0 0 0 0 0
REACTIONS 1
RX plain 3.0 0.0 1164024.7 1 A 1 2 B 1 C 1
END
"""


@pytest.mark.parametrize("cells", [1, 2, 4])
def test_lanes_without_a_reaction_add_nothing(cells):
    import torch

    import paper_2311_14941_amd as sc
    sc.ensure_built()
    g = lambda *a: torch.tensor(a, dtype=torch.float64, device="cuda:0")
    T, p, Y = g(200.0, 220.0, 400.0), g(1e5, 1e5, 1e5), g([0.4] * 3, [0.3] * 3, [0.3] * 3)
    mech = sc.Mechanism(MECH)
    kw = dict(linalg="sparse", cells_per_wave=cells)
    J = sc.Plan(mech, **kw).jacobian(T, p, Y)
    Jt = sc.Plan(mech, thermo_tol=1e-9, thermo_Tmin=150.0, thermo_Tmax=1000.0, **kw).jacobian(T, p, Y)
    assert torch.isfinite(J).all() and float(J[0].abs().max()) > 0.0
    assert torch.isfinite(Jt).all()
    assert ((Jt - J).abs() <= 1e-7 * J.abs().amax(2, keepdim=True)).all()
