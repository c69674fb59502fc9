"""Performance cases of the chemistry library.

Each case is one call (or one split step, or one forward and backward pass)
that a program using the package makes, on the seeded mechanisms and cell
states of ``synth/``:

* ``integrate``: every cell over its own dt with error control, the work
  the library exists for.  A reactor or two, an ordinary batch and a large
  one; the 9-, 53- and 110-species mechanisms; the launches the autotuner
  picks (persistent queue, longest first by predicted cost) and the plain
  default plan;
* ``chain``: operator-split substeps captured in one HIP graph;
* ``split``: one split step of the 2-D flame grid (chemistry over local time
  steps, then transport);
* ``adjoint``: forward and gradients through ``torch.autograd``;
* ``rhs``, ``jacobian``, ``linsolve``: the single-pass entry points a solver
  of its own (a flow code's integrator, a Newton or Krylov method) calls on a
  whole field;
* ``transport``: the transport update alone, on a large grid.

An adaptive integration returns the states and the per-cell status.  The
counters n_acc and n_rej and the carried step h are decisions of the step
controller: where an error estimate lies within rounding of its bound
they differ by a step between two roundings of the same arithmetic (about one
cell in 3,000 at rtol 1e-6 when the reactions are merely listed in
another order), while the states agree to far below the tolerance.
"""
import math

import numpy as np
import torch

import paper_2311_14941_amd as sc
from synth.cells import make_cells
from synth.field import flame_field
from synth.mechgen import P_REF, R_GAS, standard_mechanism

# mechanism -> workload of synth.cells whose states it takes
WORKLOAD = {"h2_9": "C1", "chon_53": "C2", "chon_110": "C3"}


def listed():
    return [
        # one reactor in a script, or the handful a user tries a mechanism on:
        # the default plan, every microsecond a serial chain of small steps
        dict(name="integrate 8 x 53, default plan", kind="integrate", mech="chon_53", n=8, dt=1e-4, rtol=1e-6,
             linalg="auto", mode="plain", order="none", reactor="const_p"),
        # the headline batch (a quarter of its cells): igniting, cold and burnt
        # cells in thirds, queue in predicted-cost order
        dict(name="integrate 16384 x 53", kind="integrate", mech="chon_53", n=16384, dt=1e-4, rtol=1e-6,
             linalg="sparse", mode="persistent", order="cost", reactor="const_p"),
        # one rank's share of a flow solver's step at the time step of the
        # paper's speed-up experiment (1e-6 s), rigid-vessel reactors
        dict(name="integrate 1999 x 53, const. volume", kind="integrate", mech="chon_53", n=1999, dt=1e-6,
             rtol=1e-6, linalg="sparse", mode="persistent", order="none", reactor="const_v"),
        # the small mechanism (four cells per wave), at the loosest decade of
        # rtol that keeps nearly every cell within the parity bar
        dict(name="integrate 16384 x 9", kind="integrate", mech="h2_9", n=16384, dt=1e-5, rtol=1e-7,
             linalg="sparse", mode="persistent", order="cost", reactor="const_p"),
        # the largest mechanism, per-cell dt over four decades (local time steps)
        dict(name="integrate 4096 x 110", kind="integrate", mech="chon_110", n=4096, dt=0.0, rtol=1e-6,
             linalg="sparse", mode="persistent", order="cost", reactor="const_p"),
        # chained substeps of a small domain in one HIP graph
        dict(name="chain 300 x 53, 8 substeps", kind="chain", mech="chon_53", n=300, dt=5e-6, substeps=8, rtol=1e-6,
             linalg="sparse", mode="persistent"),
        # the flame grid of the split-step workload (28,900 cells)
        dict(name="split step 170 x 170", kind="split", nx=170, ny=170, steps=1, mapped=False),
        # training through the integrator: T1, Y1 and the gradients of T0, Y0, dlnA
        dict(name="adjoint 1024 x 53", kind="adjoint", mech="chon_53", n=1024, dt=1e-6, rtol=1e-6),
        # source terms of a field, for a flow solver's own integrator
        dict(name="rhs 65536 x 53", kind="rhs", mech="chon_53", n=65536, linalg="sparse", reactor="const_p"),
        # analytical Jacobians of a batch
        dict(name="jacobian 4096 x 53", kind="jacobian", mech="chon_53", n=4096, linalg="sparse", reactor="const_p"),
        # one linearly implicit solve per cell, largest mechanism
        dict(name="linsolve 3001 x 110", kind="linsolve", mech="chon_110", n=3001, linalg="sparse",
             reactor="const_p"),
        # the transport update of a larger grid (species rows and temperature)
        dict(name="transport 601 x 512 x 54", kind="transport", nx=601, ny=512, ncomp=54),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case of the same ranges (sizes log-uniform, any residue)."""
    kind = rng.choice(["integrate"] * 5 + ["chain", "split", "adjoint", "adjoint", "rhs", "jacobian", "linsolve",
                                           "transport"])
    mech = rng.choice(["h2_9", "chon_53", "chon_53", "chon_110"])
    small = mech == "chon_110"
    linalg = "sparse" if small else rng.choice(["sparse", "sparse", "auto"])
    reactor = rng.choice(["const_p", "const_p", "const_p", "const_v"])
    if kind == "integrate":
        mode = rng.choice(["persistent", "persistent", "plain", "static"])
        order = rng.choice(["none", "dt", "cost"]) if mode == "persistent" else "none"
        if mech == "h2_9":
            n, dt, rtol = _log(rng, 1, 16384), 10.0 ** rng.uniform(-6, -5), 1e-7
        elif mech == "chon_53":
            n, dt, rtol = _log(rng, 1, 8192), 10.0 ** rng.uniform(-6, -4), 1e-6
        else:
            n, dt, rtol = _log(rng, 1, 3000), 0.0, 1e-6
        if mode == "static":
            n = min(n, 2048)
        return dict(kind=kind, mech=mech, n=n, dt=dt, rtol=rtol, linalg=linalg, mode=mode, order=order,
                    reactor=reactor)
    if kind == "chain":
        return dict(kind=kind, mech="chon_53", n=_log(rng, 1, 1024), dt=10.0 ** rng.uniform(-6, -5),
                    substeps=rng.randint(2, 12), rtol=1e-6, linalg=rng.choice(["sparse", "auto"]),
                    mode=rng.choice(["persistent", "plain"]))
    if kind == "split":
        return dict(kind=kind, nx=rng.randint(20, 170), ny=rng.randint(40, 170), steps=1, mapped=rng.random() < 0.4)
    if kind == "adjoint":
        return dict(kind=kind, mech=rng.choice(["chon_53", "chon_53", "h2_9"]), n=_log(rng, 1, 1024),
                    dt=10.0 ** rng.uniform(-7, -6), rtol=1e-6)
    if kind == "rhs":
        return dict(kind=kind, mech=mech, n=_log(rng, 64, 65536), linalg=linalg, reactor=reactor)
    if kind == "jacobian":
        return dict(kind=kind, mech=mech, n=_log(rng, 16, 1500 if small else 4096), linalg=linalg, reactor=reactor)
    if kind == "linsolve":
        return dict(kind=kind, mech=mech, n=_log(rng, 16, 3000), linalg=linalg, reactor=reactor)
    return dict(kind=kind, nx=rng.randint(40, 600), ny=rng.randint(40, 500), ncomp=rng.randint(5, 54))


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------
def _gpu(a):
    return torch.tensor(np.ascontiguousarray(a), dtype=torch.float64, device="cuda:0")


def _cells(case, seed):
    """Seeded cells of the mechanism's workload; with reactor const_v the
    second input is each cell's initial density."""
    c = make_cells(WORKLOAD[case["mech"]], n=case["n"], seed=seed)
    p = c["p"]
    if case.get("reactor") == "const_v":
        W = c["mech"].molar_masses()
        p = p * (1.0 / (c["Y"] / W).sum(1)) / (R_GAS * c["T"])
    dt = np.full(case["n"], case["dt"]) if case.get("dt") else c["dt"]
    return c["mech"], _gpu(c["T"]), _gpu(p), _gpu(c["Y"].T), _gpu(dt)


def _mixed_field(nx, ny, seed):
    """The flame field with its streams mixed downstream: every column is the
    inflow profile smoothed over the width a passive scalar has diffused to
    (T and Y alike), so jet, pilot and coflow meet in layers a few cells wide."""
    f = flame_field(nx=nx, ny=ny, seed=seed)
    y = np.arange(ny) * f["dx"]
    prof = np.concatenate([f["inflow_Y"], f["inflow_T"][None]])  # [N + 1, ny]
    q = np.empty((prof.shape[0], ny, nx))
    for ix in range(nx):
        sig = math.sqrt(2.0 * f["D"] * (ix + 0.5) * f["dx"] / 10.0) + 0.2 * f["dx"]
        K = np.exp(-0.5 * ((y[:, None] - y[None, :]) / sig) ** 2)
        q[:, :, ix] = prof @ (K / K.sum(1, keepdims=True)).T
    q = q.reshape(prof.shape[0], -1)
    f["Y"], f["T"] = q[:-1], q[-1]
    return f


def prepare(case, seed):
    kind = case["kind"]
    rng = np.random.default_rng(seed + 1000003)
    if kind == "transport":
        nx, ny, k = case["nx"], case["ny"], case["ncomp"]
        g = torch.Generator(device="cuda:0").manual_seed(seed)
        q = torch.rand(k, nx * ny, dtype=torch.float64, device="cuda:0", generator=g)
        u = 50.0 * torch.rand(nx * ny, dtype=torch.float64, device="cuda:0", generator=g)
        dx, D = 1e-3, 2e-4
        dt = 0.5 * torch.minimum(dx / u, torch.full_like(u, dx * dx / (4.0 * D)))
        inflow = torch.rand(k, ny, dtype=torch.float64, device="cuda:0", generator=g)
        return dict(kind=kind, a=(nx, ny, q, u, dt, dx, D, inflow), out=torch.empty_like(q))
    if kind == "split":
        f = _mixed_field(case["nx"], case["ny"], seed)
        plan = sc.Plan(sc.Mechanism(f["mech"].to_text()), rtol=1e-6, atol=1e-12, linalg="sparse", mode="persistent",
                       order="cost")
        from paper_2311_14941_amd.driver import SplitDriver
        mapping = dict(Y_fuel=f["Y_fuel"], Y_ox=f["Y_ox"], z_tol=1e-3, dT=2.0) if case["mapped"] else None
        d = SplitDriver(plan, case["nx"], case["ny"], f["p"], f["u"], f["dt"], f["dx"], f["D"], f["inflow_T"],
                        f["inflow_Y"], mapping=mapping)
        return dict(kind=kind, d=d, T=_gpu(f["T"]), Y=_gpu(f["Y"]), steps=case["steps"])
    mech, T, p, Y, dt = _cells(case, seed)
    m = sc.Mechanism(mech.to_text())
    rtol = case.get("rtol", 1e-6)
    kw = dict(rtol=rtol, atol=1e-6 * rtol, linalg=case.get("linalg", "auto"), reactor=case.get("reactor", "const_p"))
    n, N, R = case["n"], m.N, m.R
    if kind == "integrate":
        plan = sc.Plan(m, mode=case["mode"], order=case["order"], **kw)
        s = dict(kind=kind, plan=plan, a=(T, p, Y, dt), out=None)
        if case["order"] == "cost":
            # the counts a program carries from its previous split step: those
            # of a nearby state
            w = 1.0 + _gpu(rng.uniform(-0.01, 0.01, (2, n)))
            pre = sc.Plan(m, mode="persistent", **kw).integrate(T * w[0], p * w[1], Y, dt)
            s["pred"] = (pre["n_acc"].clone(), pre["n_rej"].clone())
            s["out"] = dict(pre)
        return s
    if kind == "chain":
        plan = sc.Plan(m, mode=case["mode"], **kw)
        return dict(kind=kind, c=sc.Chain(plan, T, p, Y, dt, case["substeps"]), T=T, Y=Y)
    if kind == "adjoint":
        d = _gpu(rng.normal(0.0, 0.05, R)).requires_grad_()
        return dict(kind=kind, plan=sc.Plan(m, **kw), p=p, dt=dt, x=(T.requires_grad_(), Y.requires_grad_(), d),
                    g=(_gpu(1e-3 * rng.normal(size=n)), _gpu(rng.normal(size=(N, n)))))
    plan = sc.Plan(m, **kw)
    s = dict(kind=kind, plan=plan, a=(T, p, Y))
    if kind == "linsolve":
        # h gamma over the steps an integration takes, right-hand sides of the
        # size of a stage's
        s["a"] += (_gpu(10.0 ** rng.uniform(-9, -6, n)), _gpu(rng.normal(size=(n, N + 1))))
    return s


def run(s):
    kind = s["kind"]
    if kind == "integrate":
        if "pred" in s:
            s["out"]["n_acc"].copy_(s["pred"][0])
            s["out"]["n_rej"].copy_(s["pred"][1])
        r = s["plan"].integrate(*s["a"], out=s["out"])
        return r["T"], r["Y"], r["status"]
    if kind == "chain":
        return s["c"].run(s["T"], s["Y"])[:2]
    if kind == "split":
        s["d"].load(s["T"], s["Y"])
        s["d"].step(s["steps"])
        return s["d"].T, s["d"].Y, s["d"].failed
    if kind == "adjoint":
        T, Y, d = s["x"]
        T1, Y1, _ = sc.chem_integrate(T, Y, d, s["p"], s["dt"], s["plan"])
        return (T1.detach(), Y1.detach()) + torch.autograd.grad([T1, Y1], [T, Y, d], list(s["g"]))
    if kind == "transport":
        return sc.transport2d(*s["a"], out=s["out"])
    return getattr(s["plan"], kind)(*s["a"])


# ---------------------------------------------------------------------------
# work: algorithmic bytes and flops
# ---------------------------------------------------------------------------
# attempted steps per cell (means measured once over each workload's cells)
_STEPS = {"h2_9": 458.0, "chon_53": 67.0, "chon_110": 31.0}


def _counts(mech):
    return sc.Mechanism(standard_mechanism(mech).to_text()).info


def work(case):
    kind = case["kind"]
    if kind == "transport":
        n, k = case["nx"] * case["ny"], case["ncomp"]
        return dict(bytes=8.0 * (2 * k * n + 2 * n + k * case["ny"]), flops=14.0 * k * n)
    if kind == "split":
        i, n = _counts("chon_53"), case["nx"] * case["ny"] * case["steps"]
        N = i["n_species"]
        return dict(bytes=8.0 * n * (4 * (N + 1) + 6), flops=n * (4.0 * i["flops_step_sparse"] + 14 * (N + 1)))
    i, n = _counts(case["mech"]), case["n"]
    N, R = i["n_species"], i["n_reactions"]
    state = 8.0 * n * (N + 2)
    step = i["flops_step_sparse"]
    # fewer steps over a shorter dt (a transient's steps shrink with it)
    steps = _STEPS[case["mech"]] * ((case.get("dt") or 1e-4) / (1e-5 if case["mech"] == "h2_9" else 1e-4)) ** 0.15
    if kind == "integrate":
        return dict(bytes=2 * state + 8.0 * n, flops=n * steps * step)
    if kind == "chain":
        return dict(bytes=(2 * state + 8.0 * n) * case["substeps"], flops=n * case["substeps"] * 0.4 * steps * step)
    if kind == "adjoint":
        return dict(bytes=5 * state + 16.0 * R, flops=n * 5.0 * steps * step)
    if kind == "rhs":
        return dict(bytes=2 * state, flops=float(n) * i["flops_rhs"])
    if kind == "jacobian":
        return dict(bytes=state + 8.0 * n * (N + 1) ** 2, flops=float(n) * i["flops_jac"])
    return dict(bytes=3 * state, flops=float(n) * (i["flops_jac"] + i["flops_lu_sparse"] + i["flops_solve_sparse"]))


# ---------------------------------------------------------------------------
# the same results in plain torch, 64 bits
# ---------------------------------------------------------------------------
class _Reactor:
    """f(T, Y) of the reactor from its textbook definition (CHEMKIN rate laws,
    NASA-7), batched over cells: T [n], Y [n, N]."""

    def __init__(self, mech, p, constv):
        dev = p.device
        t = lambda a, dt=torch.float64: torch.tensor(np.array(a), dtype=dt, device=dev)
        N, rx = mech.n_species, mech.reactions
        self.N, self.p, self.cv = N, p, constv
        self.W, self.nasa = t(mech.molar_masses()), t(mech.nasa_array())
        self.nu = t(mech.stoich())  # [N, R]

        def side(s):
            idx, two = np.full((3, len(rx)), N), np.zeros((3, len(rx)), bool)
            for j, r in enumerate(rx):
                for i, (k, v) in enumerate(getattr(r, s)):
                    idx[i, j], two[i, j] = k, v == 2
            return t(idx, torch.int64), t(two, torch.bool)

        self.reac, self.prod = side("reac"), side("prod")
        ln10 = math.log(10.0)
        order = np.array([sum(v for _, v in r.reac) for r in rx])
        third = np.array([r.kind == "third" for r in rx])
        troe = np.array([r.kind == "troe" for r in rx])
        self.third, self.troe = t(third, torch.bool), t(np.nonzero(troe)[0], torch.int64)
        self.lnA = t([ln10 * (r.log10A - 6.0 * (o + th - 1)) for r, o, th in zip(rx, order, third)])
        self.b, self.EaR = t([r.b for r in rx]), t([r.Ea / R_GAS for r in rx])
        al = np.ones((N, len(rx)))
        for j, r in enumerate(rx):
            for k, a in r.eff.items():
                al[k, j] = a
        self.alpha = t(al)
        self.tr = t([r.troe for r in rx if r.kind == "troe"] or np.zeros((0, 7)))
        self.lnA0 = t([ln10 * (r.troe[0] - 6.0 * o) for r, o in zip(rx, order) if r.kind == "troe"])

    def __call__(self, T, Y):
        a, Tc = self.nasa.T, T[:, None]
        lnT = torch.log(Tc)
        cp = a[0] + Tc * (a[1] + Tc * (a[2] + Tc * (a[3] + Tc * a[4])))
        h = a[0] + Tc * (a[1] / 2 + Tc * (a[2] / 3 + Tc * (a[3] / 4 + Tc * a[4] / 5))) + a[5] / Tc
        s = a[0] * lnT + Tc * (a[1] + Tc * (a[2] / 2 + Tc * (a[3] / 3 + Tc * a[4] / 4))) + a[6]
        yw = Y / self.W
        Wbar = 1.0 / yw.sum(1)
        rho = self.p if self.cv else self.p * Wbar / (R_GAS * T)
        C = rho[:, None] * yw
        c = R_GAS * (cp * yw).sum(1) - (R_GAS / Wbar if self.cv else 0.0)
        lnk = self.lnA + self.b * lnT - self.EaR / Tc
        M = C @ self.alpha
        if self.troe.numel():
            j, x = self.troe, self.tr
            lnPr = self.lnA0 + x[:, 1] * lnT - x[:, 2] / (R_GAS * Tc) - lnk[:, j] + torch.log(M[:, j])
            Fc = (1 - x[:, 3]) * torch.exp(-Tc / x[:, 4]) + x[:, 3] * torch.exp(-Tc / x[:, 5]) + torch.exp(-x[:, 6] / Tc)
            L, ln10 = torch.log10(Fc), math.log(10.0)
            X = lnPr / ln10 - 0.4 - 0.67 * L
            f = X / (0.75 - 1.27 * L - 0.14 * X)
            lnF = ln10 * L / (1 + f * f)
            lnk = lnk.index_copy(1, j, lnk[:, j] + lnPr - torch.nn.functional.softplus(lnPr, threshold=700.0) + lnF)
        lnKc = -(h - s) @ self.nu + self.nu.sum(0) * (math.log(P_REF / R_GAS) - lnT)
        C1 = torch.cat([C, torch.ones_like(Tc)], 1)

        def prod(side):
            idx, two = side
            r = 1.0
            for i in range(3):
                x = C1[:, idx[i]]
                r = r * torch.where(two[i], x * x, x)
            return r

        kf = torch.exp(lnk)
        q = kf * prod(self.reac) - torch.exp(lnk - lnKc) * prod(self.prod)
        q = torch.where(self.third, q * M, q)
        wdot = q @ self.nu.T
        e = (h - 1.0) if self.cv else h
        return -R_GAS * T * (e * wdot).sum(1) / (rho * c), self.W * wdot / rho[:, None]


def _jacobian(f, T, Y):
    """[n, N+1, N+1] over (Y, T), row by row by reverse differentiation."""
    T, Y = T.detach().requires_grad_(), Y.detach().requires_grad_()
    fT, fY = f(T, Y)
    rows = []
    for c in list(fY.sum(0)) + [fT.sum()]:
        gT, gY = torch.autograd.grad(c, [T, Y], retain_graph=True)
        rows.append(torch.cat([gY, gT[:, None]], 1))
    return torch.stack(rows, 1)


def exact(case, seed):
    """Single passes and the transport update.  An integration's result is the
    outcome of its own adaptive steps, which 64-bit arithmetic does not define
    apart from the method that takes them: None."""
    kind = case["kind"]
    if kind in ("integrate", "chain", "split", "adjoint"):
        return None
    s = prepare(case, seed)
    if kind == "transport":
        nx, ny, q, u, dt, dx, D, inflow = s["a"]
        q3 = q.view(-1, ny, nx)
        w = torch.cat([inflow[:, :, None], q3[:, :, :-1]], 2)
        e = torch.cat([q3[:, :, 1:], q3[:, :, -1:]], 2)
        sth = torch.cat([q3[:, :1], q3[:, :-1]], 1)
        nth = torch.cat([q3[:, 1:], q3[:, -1:]], 1)
        co, fo = (u * dt / dx).view(ny, nx), (D * dt / dx**2).view(ny, nx)
        return (q3 - co * (q3 - w) + fo * (e + w + nth + sth - 4 * q3)).reshape(q.shape)
    mech = standard_mechanism(case["mech"])
    T, p, Y = s["a"][0], s["a"][1], s["a"][2].T.contiguous()
    part = max(1, 2 ** 21 // mech.n_reactions // 4)
    if kind == "linsolve" and case["n"] * mech.n_species**3 > 2e10:
        return None
    outs = []
    for i in range(0, case["n"], part):
        c = slice(i, i + part)
        f = _Reactor(mech, p[c], case.get("reactor") == "const_v")
        if kind == "rhs":
            fT, fY = f(T[c], Y[c])
            outs.append((fT, fY))
        else:
            J = _jacobian(f, T[c], Y[c])
            if kind == "linsolve":
                hg, b = s["a"][3][c], s["a"][4][c]
                A = torch.eye(J.shape[1], dtype=J.dtype, device=J.device) / hg[:, None, None] - J
                J = torch.linalg.solve(A.cpu(), b.cpu()[:, :, None])[:, :, 0]
            outs.append((J,))
    outs = [torch.cat(x) for x in zip(*outs)]
    if kind == "rhs":
        return outs[0], outs[1].T.contiguous()
    return outs[0]
