"""The work a user of this framework has it do, as timed cases.

Kinds of pass (``case["kind"]``), each through the public binding ``paper_1910_02858_amd.dgsem``:

* ``step``     one step of the five-stage Runge-Kutta scheme (``DGSolver.rk_stage`` with ping-pong
               buffers, as every time loop does);
* ``loop``     one pass of an adaptive time loop: ``timestep``, the step, ``integrals`` and
               ``check_finite``;
* ``vjp``      one vector-Jacobian product of the operator (``DGSolver.rhs_vjp``);
* ``rollout``  a differentiated rollout: ``dgsem.rollout`` and the gradient of the kinetic energy;
* ``ensemble`` one step of a batch of uneven meshes (``dgsem.Batch.step`` replayed as a graph);
* ``fv``       the shock-capturing step: ``fv_switch``, then the five stages of the hybrid operator.

Meshes (``case["mesh"]``): ``lattice`` (periodic, optionally curved), ``octant`` (the Taylor-Green
vortex's octant: six symmetry planes and every element's axes rotated, so faces meet in all
orientations), ``refined`` (half the cells split 2x2x2: non-conforming faces).

``exact`` evaluates the same operator in 64 bits with plain torch, written from the discretisation's
equations alone (its gradients come from torch's own differentiation).
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_1910_02858_amd import dgsem, inputs

TWO_PI = 2.0 * math.pi
GAMMA, R_GAS, PRANDTL, REYNOLDS = 1.4, 1.0, 0.72, 1600.0


def _case(name, kind, N, kx, ky=None, kz=None, nodes="lgl", eqn="ns", form="split", vf="kep", rs="roe", curved=False,
          mesh="lattice", **more):
    c = dict(kind=kind, N=N, kx=kx, ky=kx if ky is None else ky, kz=kx if kz is None else kz, nodes=nodes, eqn=eqn,
             form=form, vf=vf, rs=rs, curved=curved, mesh=mesh, **more)
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # the first thing a new user runs, and every unit test of a coupled code: the Euler density
        # wave on 4^3 elements (5 launches of 64 small workgroups: latency)
        _case("euler_dwave_lg3_k4", "step", 3, 4, nodes="lg", eqn="euler", form="weak", vf="central", rs="llf"),
        # the same scheme where it fills the GPU: low degree, many elements (48^3, 7.1 M nodes)
        _case("euler_dwave_lg3_k48", "step", 3, 48, nodes="lg", eqn="euler", form="weak", vf="central", rs="llf"),
        # a time loop as a production run has it, at a middle size (curved TGV, 16^3, N=5): step size
        # from the state, the step, the integrals that are logged, the blow-up guard
        _case("loop_ns_kep_lgl5_k16_curved", "loop", 5, 16, curved=True),
        # the headline scheme (entropy-conserving split form, N=7) at 32^3, the largest size here
        _case("ns_ec_lgl7_k32", "step", 7, 32, vf="ec"),
        # an odd degree and a ragged mesh on LGL nodes, strong form
        _case("ns_strong_lgl4_ragged_curved", "step", 4, 21, 18, 17, form="strong", vf="central", curved=True),
        # Gauss nodes, weak form, Navier-Stokes (traces and gradients interpolated to the faces)
        _case("ns_weak_lg7_k16", "step", 7, 16, form="weak", vf="central", nodes="lg"),
        # a general mesh: boundaries, faces in every orientation
        _case("octant_ns_ec_lgl7_k16", "step", 7, 16, vf="ec", mesh="octant"),
        # a locally refined mesh: 256 cells whole, 256 split into 8 (N=7, 64 non-conforming faces a plane)
        _case("refined_ns_ec_lgl7_k8", "step", 7, 8, vf="ec", mesh="refined"),
        # shock capturing: periodic shock tube, indicator and switch before the step
        _case("fv_euler_ec_lgl7_k16", "fv", 7, 16, eqn="euler", vf="ec"),
        # one reverse evaluation of the operator where the data do not fit the caches
        _case("vjp_ns_kep_lgl5_k24_curved", "vjp", 5, 24, curved=True),
        # gradient of an objective through a rollout, checkpointed (the size of the adjoint workload)
        _case("rollout_ns_kep_lgl5_k12_curved", "rollout", 5, 12, curved=True, steps=4, ckpt=2),
        # a batch of small uneven meshes, N = 3..7, 4^3..12^3 elements each
        dict(name="ensemble_ns_kep_32", kind="ensemble", members=32, draw=0, eqn="ns", form="split", vf="kep", rs="roe"),
    ]


def _ragged(rng, N, lo, hi):
    """Lattice sizes kx, ky, kz >= 2 with about 10^U(log lo, log hi) nodes, ragged."""
    n3 = (N + 1) ** 3
    k = max(2.0, (math.exp(rng.uniform(math.log(lo), math.log(hi))) / n3) ** (1.0 / 3.0))
    ks = [max(2, round(k * rng.uniform(0.75, 1.3))) for _ in range(3)]
    while ks[0] * ks[1] * ks[2] * n3 > hi and max(ks) > 2:
        ks[ks.index(max(ks))] -= 1
    return ks


def draw(rng):
    kind = rng.choices(("step", "loop", "octant", "refined", "fv", "vjp", "rollout", "ensemble"),
                       (8, 2, 2, 1, 2, 3, 2, 1))[0]
    vf, rs = rng.choice(("kep", "ec", "central")), rng.choice(("llf", "roe", "roe", "volflux_roe"))
    if kind in ("step", "loop"):
        N = rng.randint(1, 8)
        ks = _ragged(rng, N, 4e3, 8e6)
        form = rng.choice(("weak", "strong", "split", "split"))
        nodes = "lgl" if form == "split" else rng.choice(("lg", "lgl"))
        return _case(None, kind, N, *ks, nodes=nodes, eqn=rng.choice(("euler", "ns", "ns")), form=form, vf=vf, rs=rs,
                     curved=rng.random() < 0.5)
    if kind == "octant":
        N = rng.randint(2, 8)
        form = rng.choice(("weak", "split", "split"))
        nodes = "lgl" if form == "split" else rng.choice(("lg", "lgl"))
        return _case(None, "step", N, *_ragged(rng, N, 2e4, 2e6), nodes=nodes, eqn=rng.choice(("euler", "ns")), form=form,
                     vf=vf, rs=rs, mesh="octant")
    if kind == "refined":
        N = rng.randint(2, 7)
        return _case(None, "step", N, rng.choice((4, 6, 8)), rng.randint(2, 7), rng.randint(2, 7), vf=vf, rs="roe",
                     mesh="refined")
    if kind == "fv":
        N = rng.randint(3, 7)
        return _case(None, "fv", N, *_ragged(rng, N, 2e4, 2e6), eqn="euler", vf=vf, rs=rs)
    if kind == "vjp":
        N = rng.randint(2, 7)
        ks = _ragged(rng, N, 2e4, 2e6)
        if rng.random() < 0.3:
            return _case(None, "vjp", N, *ks, nodes=rng.choice(("lg", "lgl")), eqn="euler", form="weak", vf="central",
                         rs=rng.choice(("llf", "roe")), curved=rng.random() < 0.5)
        return _case(None, "vjp", N, *ks, eqn=rng.choice(("euler", "ns", "ns")), vf=vf, rs=rs, curved=rng.random() < 0.5)
    if kind == "rollout":
        N = rng.randint(3, 7)
        return _case(None, "rollout", N, *_ragged(rng, N, 2e4, 4e5), vf=rng.choice(("kep", "kep", "ec")), curved=True,
                     steps=rng.randint(2, 5), ckpt=rng.randint(1, 5))
    return dict(kind="ensemble", members=rng.randint(8, 32), draw=rng.randint(1, 10 ** 6), eqn="ns", form="split",
                vf=rng.choice(("kep", "ec")), rs="roe")


# ------------------------------------------------------------------------------------ inputs
def _mesh(case, lgl):
    """Element coordinates, connectivity and the node map of rotated elements (None elsewhere)."""
    N, ks = case["N"], (case["kx"], case["ky"], case["kz"])
    if case["mesh"] == "refined":
        X = inputs.refined_lattice(lgl, ks, (2, 2, 2))
        nbr, side, flip, mort = inputs.connect_boxes(X, N + 1)
        return dict(X=X, nbr=nbr, side=side, flip=flip, mortar=mort, node_map=None)
    if case["mesh"] == "octant":
        X = inputs.lattice_points(lgl, *ks, box=(math.pi,) * 3)
        nbr, side, flip = inputs.box_lattice(*ks)
        rot = np.random.default_rng(0).integers(0, 24, len(X))
        X, nbr, side, flip, nm = inputs.rotate_elements(X, nbr, side, flip, N, rot)
        return dict(X=X, nbr=nbr, side=side, flip=flip, mortar=None, node_map=nm)
    X = inputs.lattice_points(lgl, *ks)
    nbr, side, _ = inputs.periodic_lattice(*ks)
    return dict(X=inputs.warp_sine(X) if case["curved"] else X, nbr=nbr, side=side, flip=None, mortar=None, node_map=None)


def _viscosity(case, amp=1.0):
    return amp / REYNOLDS if case["eqn"] == "ns" else 0.0


def _state(case, x, seed, amp=1.0, mach=0.1):
    """The flow at the nodes x[K,3,n3], with phases, strength and under-resolved content from the seed."""
    g = torch.Generator(device=x.device).manual_seed(int(seed))
    u4 = torch.rand(4, generator=g, device=x.device, dtype=torch.float64)
    sh = TWO_PI * u4[:3].view(1, 3, 1)
    one = torch.ones_like(x[:, 0])
    if case["kind"] == "fv":
        # a dense slab in x: two shocks, two contacts, two rarefactions
        s = torch.remainder(x[:, 0] + sh[0, 0, 0], TWO_PI)
        inside = (s > 2.0) & (s < 4.0)
        rho, p = torch.where(inside, one, 0.3 * one), torch.where(inside, one, 0.2 * one)
        u, v, w = (0.1 + 0.1 * u4[3]) * one, 0.0 * one, 0.0 * one
    elif case["eqn"] == "euler" and case["mesh"] == "lattice":
        # density wave carried by a uniform flow
        rho = 1.0 + (0.1 + 0.1 * u4[3]) * torch.sin(x[:, 0] + x[:, 1] + x[:, 2] + sh.sum())
        u, v, w, p = one, one, one, one
    else:
        # Taylor-Green vortex with some flow along z; shifted on periodic meshes
        a = amp * (0.8 + 0.4 * u4[3])
        X, Y, Z = (x + (sh if case.get("mesh", "lattice") != "octant" else 0.0)).unbind(1)
        u, v, w = a * X.sin() * Y.cos() * Z.cos(), -a * X.cos() * Y.sin() * Z.cos(), 0.1 * a * Z.sin()
        p = amp * amp / (GAMMA * mach * mach) + a * a / 16.0 * ((2 * X).cos() + (2 * Y).cos()) * ((2 * Z).cos() + 2.0)
        rho = one
    U = torch.stack((rho, rho * u, rho * v, rho * w, p / (GAMMA - 1.0) + 0.5 * rho * (u * u + v * v + w * w)), 1)
    if case["kind"] != "fv":
        U = U * (1.0 + 1e-4 * torch.randn(U.shape, generator=g, device=x.device, dtype=torch.float64))
    return U


def _adjoint(U, seed):
    g = torch.Generator(device=U.device).manual_seed(int(seed) + 1)
    return torch.randn(U.shape, generator=g, device=U.device, dtype=torch.float64)


def _members(case, seed):
    """One case per member of the ensemble, with its amplitude, Mach number and seed."""
    out = []
    for i, w in enumerate(inputs.ensemble_draw(case["members"], case["draw"])):
        c = _case(None, "step", w.N, w.K1, vf=case["vf"], rs=case["rs"])
        out.append((c, w.amp, w.mach, 1000 * int(seed) + i))
    return out


def _solver(case, amp=1.0):
    lgl, _ = dgsem.nodes(case["N"], "lgl")
    M = _mesh(case, lgl)
    S = dgsem.DGSolver(M["X"], M["nbr"], M["side"], case["N"], case["nodes"], case["eqn"], case["form"], case["vf"],
                       case["rs"], GAMMA, R_GAS, _viscosity(case, amp), PRANDTL, flip=M["flip"], mortar=M["mortar"])
    return S, torch.from_numpy(S.node_coords()).cuda()


def prepare(case, seed):
    if case["kind"] == "ensemble":
        sols, cur = [], []
        for c, amp, mach, sd in _members(case, seed):
            S, x = _solver(c, amp)
            sols.append(S)
            cur.append(_state(c, x, sd, amp, mach))
        B = dgsem.Batch(sols)
        B.tune(cur, 2)
        return dict(kind="ensemble", B=B, cur=cur, nxt=[S.empty() for S in sols], R=[torch.zeros_like(u) for u in cur],
                    dt=[S.timestep(u, 0.5, 0.5) for S, u in zip(sols, cur)])
    S, x = _solver(case)
    U = _state(case, x, seed)
    st = dict(kind=case["kind"], S=S, U=U)
    if case["kind"] == "vjp":
        return dict(st, W=_adjoint(U, seed), out=S.empty())
    if case["kind"] == "fv":
        S.fv_enable(1, -5.0, -2.5)
    st["dt"] = S.timestep(U, 0.5, 0.5) if case["kind"] == "fv" else S.timestep(U, 0.9, 0.9)
    if case["kind"] == "rollout":
        return dict(st, steps=case["steps"], ckpt=case["ckpt"], wJ=S.mass_weights())
    return dict(st, A=S.empty(), B=S.empty(), R=torch.zeros_like(U), ab=dgsem.rk_coefficients())


def _step(st, dt):
    """One Runge-Kutta step from st["U"] (kept); returns the new state."""
    S, R, (a, b, _) = st["S"], st["R"], st["ab"]
    cur, nxt, free = st["U"], st["A"], st["B"]
    for s in range(5):
        S.rk_stage(cur, nxt, R, a[s], b[s], dt)
        cur, nxt, free = nxt, free, nxt
    return cur


def run(state):
    kind = state["kind"]
    if kind == "ensemble":
        # the batch advances: the new states are the next pass's input
        state["B"].step(state["cur"], state["nxt"], state["R"], state["dt"])
        state["cur"], state["nxt"] = state["nxt"], state["cur"]
        return state["cur"]
    S, U = state["S"], state["U"]
    if kind == "step":
        return _step(state, state["dt"]), state["R"]
    if kind == "loop":
        dt = S.timestep(U, 0.9, 0.9)
        V = _step(state, dt)
        return V, S.integrals(V), dt, S.check_finite(V)
    if kind == "fv":
        S.fv_switch(U)  # U then holds the mixed nodal values and subcell means; a repeated switch keeps them
        return _step(state, state["dt"]), U
    if kind == "vjp":
        return S.rhs_vjp(U, state["W"], state["out"])
    u = U.detach().requires_grad_(True)
    UT = dgsem.rollout(S, u, state["steps"], state["dt"], state["ckpt"])
    (g,) = torch.autograd.grad(dgsem.kinetic_energy(UT, state["wJ"]), u)
    return UT.detach(), g


# ------------------------------------------------------------------------------------ work
def _count(case):
    K = case["kx"] * case["ky"] * case["kz"]
    if case["mesh"] == "refined":  # half of the cells are split into 8
        K += 7 * (case["kx"] // 2) * case["ky"] * case["kz"]
    return K


def work(case):
    """A stage cannot do without reading the state, the metric terms (10 doubles a node) and, after the
    first, the register, and writing state and register; the reverse of an evaluation reads state, metric
    terms and the adjoint and writes one. Operations: the volume terms (the pair fluxes or the contraction of
    each direction's fluxes, for Navier-Stokes the gradients and the viscous contraction too)."""
    if case["kind"] == "ensemble":
        ws = [work(c) for c, _, _, _ in _members(case, 0)]
        return {"bytes": sum(w["bytes"] for w in ws), "flops": sum(w["flops"] for w in ws)}
    n = case["N"] + 1
    nodes = _count(case) * n ** 3
    if case["form"] == "split":
        flops = 3 * (n / 2) * {"kep": 45, "ec": 75, "central": 50}[case["vf"]] + 3 * n * 10
    else:
        flops = 3 * (35 + 10 * n)
    if case["eqn"] == "ns":
        flops += 3 * n * 24 + 3 * n * 8 + 120
    if case["kind"] == "vjp":
        return {"bytes": 25 * 8.0 * nodes, "flops": 2.5 * flops * nodes}
    step = {"bytes": (5 * 30 - 5) * 8.0 * nodes, "flops": 5.0 * flops * nodes}
    if case["kind"] == "rollout":
        # forward, and in reverse each stage's evaluation at its kept state (35 doubles a node, 2.5 times the operations)
        return {"bytes": case["steps"] * (step["bytes"] + 5 * 35 * 8.0 * nodes), "flops": case["steps"] * 3.5 * step["flops"]}
    if case["kind"] == "loop":
        return {"bytes": step["bytes"] + (15 + 6 + 5) * 8.0 * nodes, "flops": step["flops"] + 100.0 * nodes}
    return step


# ------------------------------------------------------------------------------------ exact
# The discretisation in plain torch, 64 bits. Fields are [K, comp, k, j, i]; direction d runs along axis
# -1-d; a side's face points are the remaining two axes.

_A = (0.0, -567301805773 / 1357537059087, -2404267990393 / 2016746695238, -3550918686646 / 2091501179385,
      -1275806237668 / 842570457699)
_B = (1432997174477 / 9575080441755, 5161836677717 / 13612068292357, 1720146321549 / 2090206949498,
      3134564353537 / 4481467310338, 2277821191437 / 14882151754819)


def _legendre(N, x):
    """P_N and P_N' at x (recurrence; the derivative from P_N and P_{N-1} off the end points)."""
    a, b = np.ones_like(x), x
    for k in range(2, N + 1):
        a, b = b, ((2 * k - 1) * x * b - (k - 1) * a) / k
    d = np.where(np.abs(x) < 1, N * (a - x * b) / np.where(np.abs(x) < 1, 1 - x * x, 1), 0)
    return b, d


def _quadrature(N, kind):
    """Nodes and weights in extended precision: Newton's method from numpy's roots."""
    leg = np.polynomial.legendre
    if kind == "lg":
        x = leg.leggauss(N + 1)[0].astype(np.longdouble)
        for _ in range(3):
            P, dP = _legendre(N + 1, x)
            x = x - P / dP
        x = (x - x[::-1]) / 2
        return x, 2 / ((1 - x * x) * _legendre(N + 1, x)[1] ** 2)
    c = np.zeros(N + 1)
    c[N] = 1.0
    x = np.concatenate(([-1.0], np.sort(leg.legroots(leg.legder(c)).real) if N > 1 else [], [1.0])).astype(np.longdouble)
    for _ in range(4):
        P, dP = _legendre(N, x[1:-1])
        x[1:-1] -= dP * (1 - x[1:-1] ** 2) / (2 * x[1:-1] * dP - N * (N + 1) * P)
    x = (x - x[::-1]) / 2
    return x, 2 / (N * (N + 1) * _legendre(N, x)[0] ** 2)


def _lagrange(x, at):
    """[len(at), len(x)]: the Lagrange polynomials of the nodes x at the points at."""
    x = np.asarray(x, np.longdouble)
    return np.array([[np.prod([(t - xk) / (xj - xk) for k, xk in enumerate(x) if k != j]) for j, xj in enumerate(x)]
                     for t in np.asarray(at, np.longdouble)])


def _derivative(x):
    n = len(x)
    bw = np.array([1 / np.prod([x[j] - x[k] for k in range(n) if k != j]) for j in range(n)])
    D = np.array([[0 * x[0] if r == s else bw[s] / bw[r] / (x[r] - x[s]) for s in range(n)] for r in range(n)])
    return D - np.diag(D.sum(1))


def _rows(f, B):
    """f @ B for a small matrix B, some millions of rows at a time (a product of 16 M rows and more came back wrong)."""
    if B.dim() == 1:
        return _rows(f, B.unsqueeze(1)).squeeze(-1)
    x = f.reshape(-1, f.shape[-1])
    return torch.cat([c @ B for c in x.split(1 << 22)]).view(f.shape[:-1] + (B.shape[-1],))


def _along(A, f, d):
    """The matrix A applied along direction d."""
    return torch.movedim(_rows(torch.movedim(f, -1 - d, -1), A.T), -1, -1 - d)


def _col(t, d):
    return t.view((-1,) + (1,) * d)


class _Exact:
    def __init__(self, case, amp=1.0, device=None):
        self.case, N, n = case, case["N"], case["N"] + 1
        dev = device or ("cuda" if torch.cuda.is_available() else "cpu")
        t = lambda a: torch.as_tensor(np.ascontiguousarray(a, np.float64), device=dev)  # noqa: E731
        xl, _ = _quadrature(N, "lgl")
        x, w = _quadrature(N, case["nodes"])
        self.n, self.dev, self.w = n, dev, t(w)
        D = _derivative(x)
        self.D, self.Dh = t(D), t(-(w[None, :] / w[:, None]) * D.T)
        ends = _lagrange(x, (-1.0, 1.0))
        self.l, self.lh = t(ends), t(ends / w[None, :])
        self.mu = _viscosity(case, amp)
        self.kappa = self.mu * GAMMA * R_GAS / (GAMMA - 1.0) / PRANDTL
        M = _mesh(case, xl.astype(np.float64))
        self.node_map = None
        if M["node_map"] is not None:
            # the same operator on the elements before their axes were rotated
            self.node_map = torch.from_numpy(M["node_map"]).to(dev)
            ks = (case["kx"], case["ky"], case["kz"])
            X = inputs.lattice_points(xl.astype(np.float64), *ks, box=(math.pi,) * 3)
            nbr, mort = inputs.box_lattice(*ks)[0], None
        else:
            X, nbr, mort = M["X"], M["nbr"], M["mortar"]
        K = len(X)
        self.K = K
        self.nbr = torch.from_numpy(nbr.astype(np.int64)).to(dev)
        self.mort = None if mort is None else torch.from_numpy(mort.astype(np.int64)).to(dev)
        if mort is not None:
            lo, up = _lagrange(x, (x - 1) / 2), _lagrange(x, (x + 1) / 2)
            self.I = (t(lo), t(up))
            self.P = tuple(t(a.T * w[None, :] / w[:, None]) for a in (lo, up))
        # metric terms in curl form at the LGL nodes, J at the solution nodes
        X = t(X).view(K, 3, n, n, n)
        mid = X.mean((2, 3, 4), keepdim=True)
        X = X - mid
        Dl = t(_derivative(xl))
        Ja = torch.empty((K, 3, 3, n, n, n), dtype=torch.float64, device=dev)  # [K, direction, component]
        for c in range(3):
            m, l = (c + 1) % 3, (c + 2) % 3
            g = [X[:, l] * _along(Dl, X[:, m], d) for d in range(3)]
            for d in range(3):
                a, b = (d + 1) % 3, (d + 2) % 3
                Ja[:, d, c] = _along(Dl, g[a], b) - _along(Dl, g[b], a)
        V = t(_lagrange(xl, x)) if case["nodes"] == "lg" else None
        if V is not None:
            for d in range(3):
                Ja, X = _along(V, Ja, d), _along(V, X, d)
        self.Ja = Ja
        jac = torch.stack([_along(self.D, X, d) for d in range(3)], -1).permute(0, 2, 3, 4, 1, 5)
        a, b, c = jac[..., 0], jac[..., 1], jac[..., 2]
        self.J = (a * torch.linalg.cross(b, c)).sum(-1).unsqueeze(1)
        self.points = (X + mid).reshape(K, 3, n ** 3)
        # outward normal times surface element of every side, the master's (the + side's) on both
        self.nt = {}
        for d in range(3):
            plus, minus = self.trace(Ja[:, d], 2 * d + 1), self.trace(Ja[:, d], 2 * d)
            nb = self.nbr[:, 2 * d]
            other = plus[nb.clamp(min=0)]
            own = _col(nb < 0, 3) if self.mort is None else _col((nb < 0) | (self.mort[:, 2 * d] > 0), 3)
            self.nt[2 * d + 1], self.nt[2 * d] = plus, -torch.where(own, minus, other)

    def trace(self, f, s):
        return _rows(torch.movedim(f, -1 - s // 2, -1), self.l[s % 2])

    # ---- rotated elements
    def to_lattice(self, U):
        if self.node_map is None:
            return U
        return torch.zeros_like(U).scatter(2, self.node_map[:, None, :].expand_as(U), U)

    def from_lattice(self, U):
        return U if self.node_map is None else torch.gather(U, 2, self.node_map[:, None, :].expand_as(U))

    # ---- pointwise physics; states are [K, 5, ...]
    @staticmethod
    def prim(U):
        u = U[:, 1:4] / U[:, :1]
        return U[:, 0], u, (GAMMA - 1.0) * (U[:, 4] - 0.5 * (U[:, 1:4] * u).sum(1))

    def lifted(self, U):
        rho, u, p = self.prim(U)
        return torch.cat((u, (p / (rho * R_GAS)).unsqueeze(1)), 1)

    def flux(self, U, nv):
        _, u, p = self.prim(U)
        un = (u * nv).sum(1)
        return torch.cat(((U[:, :1] * un.unsqueeze(1)), U[:, 1:4] * un.unsqueeze(1) + p.unsqueeze(1) * nv,
                          ((U[:, 4] + p) * un).unsqueeze(1)), 1)

    def viscous(self, U, G, nv):
        """G[K, 3 (derivative), 4 (u, v, w, T), ...] along nv."""
        _, u, _ = self.prim(U)
        gu = G[:, :, :3]
        div = gu[:, 0, 0] + gu[:, 1, 1] + gu[:, 2, 2]
        tau = [[self.mu * (gu[:, b, a] + gu[:, a, b]) - ((2.0 / 3.0) * self.mu * div if a == b else 0.0) for b in range(3)]
               for a in range(3)]
        m = [sum(tau[a][b] * nv[:, b] for b in range(3)) for a in range(3)]
        e = sum(m[a] * u[:, a] for a in range(3)) + self.kappa * (G[:, :, 3] * nv).sum(1)
        return torch.stack((torch.zeros_like(e), *m, e), 1)

    @staticmethod
    def logmean(a, b):
        f = (a - b) / (a + b)
        u = f * f
        small = u < 1e-4
        series = (a + b) / (2.0 + u * (2.0 / 3.0 + u * (2.0 / 5.0 + u * (2.0 / 7.0 + u * (2.0 / 9.0)))))
        bb = torch.where(small, 0.5 * a, b)  # a value whose logarithm differs, where it is not used
        return torch.where(small, series, (a - bb) / (a.log() - bb.log()))

    def two_point(self, UA, UB, nv):
        ra, ua, pa = self.prim(UA)
        rb, ub, pb = self.prim(UB)
        um = 0.5 * (ua + ub)
        un = (um * nv).sum(1)
        if self.case["vf"] == "central":
            return 0.5 * (self.flux(UA, nv) + self.flux(UB, nv))
        if self.case["vf"] == "kep":
            f0 = 0.5 * (ra + rb) * un
            pm = 0.5 * (pa + pb)
            h = 0.5 * ((UA[:, 4] + pa) / ra + (UB[:, 4] + pb) / rb)
            return torch.cat((f0.unsqueeze(1), f0.unsqueeze(1) * um + pm.unsqueeze(1) * nv, (f0 * h).unsqueeze(1)), 1)
        ba, bb = 0.5 * ra / pa, 0.5 * rb / pb
        f0 = self.logmean(ra, rb) * un
        ph = 0.5 * (ra + rb) / (ba + bb)
        fm = f0.unsqueeze(1) * um + ph.unsqueeze(1) * nv
        q = 0.5 * ((ua * ua).sum(1) + (ub * ub).sum(1))
        fe = f0 * (0.5 / ((GAMMA - 1.0) * self.logmean(ba, bb)) - 0.5 * q) + (um * fm).sum(1)
        return torch.cat((f0.unsqueeze(1), fm, fe.unsqueeze(1)), 1)

    def roe(self, L, R, nh):
        """Sum over the waves of |lambda| times strength times eigenvector at the Roe average."""
        rl, ul, pl = self.prim(L)
        rr, ur, pr = self.prim(R)
        sl, sr = rl.sqrt(), rr.sqrt()
        mean = lambda a, b: (sl * a + sr * b) / (sl + sr)  # noqa: E731
        u = torch.stack([mean(ul[:, c], ur[:, c]) for c in range(3)], 1)
        H = mean((L[:, 4] + pl) / rl, (R[:, 4] + pr) / rr)
        q = (u * u).sum(1)
        c = ((GAMMA - 1.0) * (H - 0.5 * q)).sqrt()
        un, r = (u * nh).sum(1), sl * sr
        du, dp, dr = ur - ul, pr - pl, rr - rl
        dun = (du * nh).sum(1)
        a1, a5 = 0.5 * (dp - r * c * dun) / c ** 2, 0.5 * (dp + r * c * dun) / c ** 2
        s1, s2, s5 = (un - c).abs() * a1, un.abs() * (dr - dp / c ** 2), (un + c).abs() * a5
        sh = (un.abs() * r).unsqueeze(1) * (du - dun.unsqueeze(1) * nh)  # shear waves
        e = lambda v: v.unsqueeze(1)  # noqa: E731
        mom = e(s1) * (u - e(c) * nh) + e(s2) * u + e(s5) * (u + e(c) * nh) + sh
        en = s1 * (H - un * c) + 0.5 * s2 * q + s5 * (H + un * c) + (u * sh).sum(1)
        return torch.cat((e(s1 + s2 + s5), mom, e(en)), 1)

    def riemann(self, L, R, nv):
        """Numerical flux times the surface element along nv (not normalised)."""
        sh = (nv * nv).sum(1, keepdim=True).sqrt()
        nh, rs = nv / sh, self.case["rs"]
        if rs == "llf":
            (rl, ul, pl), (rr, ur, pr) = self.prim(L), self.prim(R)
            lam = torch.maximum((ul * nh).sum(1).abs() + (GAMMA * pl / rl).sqrt(),
                                (ur * nh).sum(1).abs() + (GAMMA * pr / rr).sqrt())
            return sh * (0.5 * (self.flux(L, nh) + self.flux(R, nh)) - 0.5 * lam.unsqueeze(1) * (R - L))
        f = self.two_point(L, R, nh) if rs.startswith("volflux") else 0.5 * (self.flux(L, nh) + self.flux(R, nh))
        return sh * (f if rs == "volflux" else f - 0.5 * self.roe(L, R, nh))

    # ---- faces
    @staticmethod
    def mirror(v, nh):
        """A field of vectors [K, 3, ...] reflected across the plane with unit normal nh."""
        return v - 2.0 * (v * nh).sum(1, keepdim=True) * nh

    def outer(self, tr, s, kind):
        """The other side's trace at side s: the neighbour's, the mirrored own one at a symmetry plane, the big
        side's restricted to this small side."""
        nb = self.nbr[:, s]
        out = tr[s ^ 1][nb.clamp(min=0)]
        if bool((nb < 0).any()):
            own, nh = tr[s], self.nt[s] / (self.nt[s] ** 2).sum(1, keepdim=True).sqrt()
            if kind == "U":
                m = torch.cat((own[:, :1], self.mirror(own[:, 1:4], nh), own[:, 4:]), 1)
            elif kind == "W":
                m = torch.cat((self.mirror(own[:, :3], nh), own[:, 3:]), 1)
            else:
                g = torch.stack([self.mirror(own[:, :, c], nh) for c in range(4)], 2)
                m = torch.stack([torch.cat((self.mirror(g[:, d, :3], nh), g[:, d, 3:]), 1) for d in range(3)], 1)
            out = torch.where(_col(nb < 0, out.dim() - 1), m, out)
        if self.mort is not None:
            for p in range(4):
                e = (self.mort[:, s] == 4 + p).nonzero().squeeze(1)
                if len(e):
                    out = out.index_copy(0, e, _along(self.I[p >> 1], _along(self.I[p & 1], tr[s ^ 1][nb[e]], 0), 1))
        return out

    def project(self, f):
        """The big sides' outward terms from the small sides' (f: side -> outward term)."""
        if self.mort is None:
            return f
        out = dict(f)
        for s in range(6):
            big = _col(self.mort[:, s] == 3, f[s].dim() - 1)
            acc = torch.zeros_like(f[s])
            for p in range(4):
                e = (self.mort[:, s ^ 1] == 4 + p).nonzero().squeeze(1)
                if len(e):
                    acc = acc.index_add(0, self.nbr[e, s ^ 1], -_along(self.P[p >> 1], _along(self.P[p & 1], f[s ^ 1][e], 0), 1))
            out[s] = torch.where(big, acc, f[s])
        return out

    def own_first(self, s):
        """Whether this element's state is the flux's first argument (the + side's, a boundary's, a small side's)."""
        m = torch.full((self.K,), bool(s & 1), device=self.dev)
        m = m | (self.nbr[:, s] < 0)
        return m if self.mort is None else torch.where(self.mort[:, s] > 0, torch.ones_like(m), m)

    def spread(self, f, s):
        """A face term lifted onto the element: lhat(+-1) along the side's direction."""
        return torch.movedim(f.unsqueeze(-1) * self.lh[s % 2], -1, -1 - s // 2)

    # ---- the operator; U [K, 5, n, n, n]
    def gradients(self, U):
        W = self.lifted(U)
        Wt = {s: self.trace(W, s) for s in range(6)}
        f = {s: self.nt[s].unsqueeze(2) * (0.5 * (Wt[s] + self.outer(Wt, s, "W"))).unsqueeze(1) for s in range(6)}
        f = self.project(f)
        G = sum(_along(self.Dh, self.Ja[:, d].unsqueeze(2) * W.unsqueeze(1), d) for d in range(3))
        return (G + sum(self.spread(f[s], s) for s in range(6))) / self.J.unsqueeze(1)

    def surface(self, U):
        """Outward numerical flux times the surface element of every side, and the gradients."""
        ns = self.case["eqn"] == "ns"
        Ut = {s: self.trace(U, s) for s in range(6)}
        G = self.gradients(U) if ns else None
        Gt = {s: self.trace(G, s) for s in range(6)} if ns else None
        f = {}
        for s in range(6):
            own, oth = Ut[s], self.outer(Ut, s, "U")
            first = _col(self.own_first(s), 3)
            sg = torch.where(first, 1.0, -1.0).to(own)
            nv = sg * self.nt[s]
            f[s] = sg * self.riemann(torch.where(first, own, oth), torch.where(first, oth, own), nv)
            if ns:
                f[s] = f[s] - 0.5 * (self.viscous(own, Gt[s], self.nt[s]) +
                                     self.viscous(oth, self.outer(Gt, s, "G"), self.nt[s]))
        return self.project(f), G

    def volume(self, U, G):
        form, n = self.case["form"], self.n
        acc = 0.0
        for d in range(3):
            Fv = self.viscous(U, G, self.Ja[:, d]) if G is not None else 0.0
            Fc = self.flux(U, self.Ja[:, d])
            if form == "weak":
                acc = acc + _along(self.Dh, Fc - Fv, d)
                continue
            F = Fc - Fv
            inner = self.spread(self.trace(F, 2 * d + 1), 2 * d + 1) - self.spread(self.trace(F, 2 * d), 2 * d)
            if form == "strong":
                acc = acc + _along(self.D, F, d) - inner
                continue
            # every pair of nodes of a line once
            i, j = torch.triu_indices(n, n, 1, device=self.dev)
            u, nv = torch.movedim(U, -1 - d, -1), torch.movedim(self.Ja[:, d], -1 - d, -1)
            P = self.two_point(u[..., i], u[..., j], 0.5 * (nv[..., i] + nv[..., j]))
            at = torch.arange(len(i), device=self.dev)
            M = torch.zeros((len(i), n), dtype=torch.float64, device=self.dev)
            M[at, i] = 2.0 * self.D[i, j]
            M[at, j] = 2.0 * self.D[j, i]
            acc = acc + torch.movedim(_rows(P, M), -1, -1 - d) + _along(torch.diag(2.0 * torch.diagonal(self.D)), Fc, d) - inner
            if G is not None:
                acc = acc - _along(self.D, Fv, d)
        return acc

    def rhs(self, U):
        f, G = self.surface(U)
        return -(self.volume(U, G) + sum(self.spread(f[s], s) for s in range(6))) / self.J

    def stages(self, U, dt, steps=1, rhs=None):
        rhs = rhs or self.rhs
        for _ in range(steps):
            R = torch.zeros_like(U)
            for a, b in zip(_A, _B):
                R = a * R + dt * rhs(U)
                U = U + b * R
        return U, R

    def timestep(self, U, cfl):
        rho, u, p = self.prim(U)
        nn = (self.Ja ** 2).sum(2)
        J, c = self.J[:, 0], (GAMMA * p / rho).sqrt()
        sc = sum(((u * self.Ja[:, d]).sum(1).abs() + c * nn[:, d].sqrt()) / J for d in range(3))
        dt = cfl * 2.0 / ((2 * self.case["N"] + 1) * float(sc.max()))
        if self.mu > 0.0:
            sv = sum(max(4.0 / 3.0, GAMMA / PRANDTL) * (self.mu / rho) * nn[:, d] / J ** 2 for d in range(3))
            dt = min(dt, cfl * 4.0 / ((2 * self.case["N"] + 1) * float(sv.max())))
        return dt

    def weights(self):
        return self.J * (self.w.view(-1, 1, 1) * self.w.view(1, -1, 1) * self.w.view(1, 1, -1))

    def integrals(self, U):
        q = self.weights()
        rho, u, p = self.prim(U)
        fields = [U[:, v] for v in range(5)] + [0.5 * rho * (u * u).sum(1), -rho * (p.log() - GAMMA * rho.log()) / (GAMMA - 1.0)]
        return np.array([float((q[:, 0] * f).sum()) for f in fields] + [float(self.J.min())])

    # ---- finite-volume subcells (periodic lattices, reference axes aligned)
    def subcells(self):
        n = self.n
        x, w = _quadrature(n - 1, self.case["nodes"])
        V = np.array([w @ _lagrange(x, -1 + (2 * k + x + 1) / n) / 2 for k in range(n)]).astype(np.float64)
        L = np.array([math.sqrt(k + 0.5) * (_legendre(k, x)[0] if k else 1 + 0 * x) for k in range(n)]).T.astype(np.float64)
        t = lambda a: torch.as_tensor(a, dtype=torch.float64, device=self.dev)  # noqa: E731
        self.V, self.Vi, self.Li = t(V), t(np.linalg.inv(V)), t(np.linalg.inv(L))

    def all3(self, A, f):
        return _along(A, _along(A, _along(A, f, 0), 1), 2)

    def troubled(self, U, hi):
        rho, _, p = self.prim(U)
        e = self.all3(self.Li, rho * p) ** 2
        i = torch.arange(self.n, device=self.dev)
        m = torch.maximum(torch.maximum(i.view(-1, 1, 1), i.view(1, -1, 1)), i.view(1, 1, -1))
        tot, eN, eM = e.sum((1, 2, 3)), (e * (m == self.n - 1)).sum((1, 2, 3)), (e * (m == self.n - 2)).sum((1, 2, 3))
        return torch.maximum(eN / tot.clamp(min=1e-300), eM / (tot - eN).clamp(min=1e-300)).clamp(min=1e-300).log10() > hi

    def as_prim(self, U):
        rho, u, p = self.prim(U)
        return torch.cat((rho.unsqueeze(1), u, p.unsqueeze(1)), 1)

    @staticmethod
    def as_cons(W):
        return torch.cat((W[:, :1], W[:, :1] * W[:, 1:4],
                          (W[:, 4] / (GAMMA - 1.0) + 0.5 * W[:, 0] * (W[:, 1:4] ** 2).sum(1)).unsqueeze(1)), 1)

    @staticmethod
    def minmod(a, b):
        return torch.where(a * b <= 0.0, torch.zeros_like(a), torch.where(a.abs() < b.abs(), a, b))

    def hybrid(self, U, fv):
        """The operator with the elements fv holding subcell means."""
        n = self.n
        sel = lambda f, s: f.select(-1 - s // 2, n - 1 if s & 1 else 0)  # noqa: E731
        is_fv = lambda k: _col(fv, k)  # noqa: E731
        face = {s: torch.where(is_fv(3), sel(U, s), _along(self.V, _along(self.V, self.trace(U, s), 0), 1)) for s in range(6)}
        outer = {s: face[s ^ 1][self.nbr[:, s]] for s in range(6)}
        W = self.as_prim(U)
        lo = torch.zeros_like(W)
        slopes = []
        for d in range(3):
            ax = -1 - d
            ext = torch.cat((self.as_prim(outer[2 * d]).unsqueeze(ax), W, self.as_prim(outer[2 * d + 1]).unsqueeze(ax)), ax)
            df = ext.diff(dim=ax)
            slopes.append(self.minmod(df.narrow(ax, 0, n), df.narrow(ax, 1, n)))
        rec = lambda d, sg: self.as_cons(W + 0.5 * sg * slopes[d])  # noqa: E731
        side = {s: torch.where(is_fv(3), sel(rec(s // 2, 1.0 if s & 1 else -1.0), s), face[s]) for s in range(6)}
        area = lambda d, shape: self.Ja[:, d, :, :1, :1, :1].expand(shape)  # noqa: E731  constant on these meshes
        f, _ = self.surface(U)
        acc = 0.0
        for d in range(3):
            ax = -1 - d
            for s in (2 * d, 2 * d + 1):
                own, oth = side[s], side[s ^ 1][self.nbr[:, s]]
                sg = 1.0 if s & 1 else -1.0
                nv = self.Ja[:, d, :, 0, 0, :1].unsqueeze(-1).expand(self.K, 3, n, n)
                sub = sg * (self.riemann(own, oth, nv) if s & 1 else self.riemann(oth, own, nv))
                near = _col(fv[self.nbr[:, s]] & ~fv, 3)
                f[s] = torch.where(near, _along(self.Vi, _along(self.Vi, sub, 0), 1), f[s])
                if s & 1:
                    fp = sub
                else:
                    fm = -sub
            L, R = rec(d, 1.0).narrow(ax, 0, n - 1), rec(d, -1.0).narrow(ax, 1, n - 1)
            inner = self.riemann(L, R, area(d, (self.K, 3) + L.shape[2:]))
            acc = acc + torch.cat((fm.unsqueeze(ax), inner, fp.unsqueeze(ax)), ax).diff(dim=ax)
        sub = -acc / (2.0 / n * self.J)
        dg = -(self.volume(U, None) + sum(self.spread(f[s], s) for s in range(6))) / self.J
        return torch.where(is_fv(4), sub, dg)


def exact(case, seed):
    if case["kind"] == "ensemble":
        out = []
        for c, amp, mach, sd in _members(case, seed):
            E = _Exact(c, amp)
            U = _state(c, E.points, sd, amp, mach).view(E.K, 5, E.n, E.n, E.n)
            out.append(E.stages(U, E.timestep(U, 0.5))[0].reshape(E.K, 5, -1))
        return out
    E = _Exact(case)
    U = _state(case, E.from_lattice(E.points), seed)
    W = _adjoint(U, seed) if case["kind"] == "vjp" else None
    shape, field = U.shape, (E.K, 5, E.n, E.n, E.n)
    U = E.to_lattice(U).view(field)
    back = lambda x: E.from_lattice(x.reshape(shape))  # noqa: E731
    if case["kind"] == "vjp":
        U = U.requires_grad_(True)
        (g,) = torch.autograd.grad(E.rhs(U), U, W.view(field))
        return back(g)
    if case["kind"] == "rollout":
        dt = E.timestep(U, 0.9)
        U = U.requires_grad_(True)
        UT = E.stages(U, dt, case["steps"])[0]
        ke = (E.weights()[:, 0] * 0.5 * (UT[:, 1:4] ** 2).sum(1) / UT[:, 0]).sum()
        (g,) = torch.autograd.grad(ke, U)
        return back(UT.detach()), back(g)
    if case["kind"] == "fv":
        dt = E.timestep(U, 0.5)
        E.subcells()
        fv = E.troubled(U, -2.5)
        U = torch.where(_col(fv, 4), E.all3(E.V, U), U)
        return back(E.stages(U, dt, rhs=lambda u: E.hybrid(u, fv))[0]), back(U)
    dt = E.timestep(U, 0.9)
    V, R = E.stages(U, dt)
    if case["kind"] == "loop":
        return back(V), E.integrals(V), dt, True
    return back(V), back(R)
