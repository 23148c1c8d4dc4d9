"""Meshes whose workgroups fit the GPU in one round take kernels with a lane per end of every line, larger ones with a
lane per line.  A mesh, and more than 512 disjoint elements made of copies of it: the split form gives the same bits
(members of a batch always take the larger meshes' kernels), the weak and strong forms the same to the bar of the
operator (1e-12 of the whole vector: their sums are split).  Every degree, on lattices (affine and curved), boxes
with boundary sides and turned axes, refined lattices, and with finite-volume elements; the small mesh itself is
compared with the oracle elsewhere."""
import numpy as np
import pytest

from paper_1910_02858_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dg():
    import torch
    from paper_1910_02858_amd import dgsem
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    dgsem.lib()
    return dgsem


def _base(kind, x, N):
    """Coordinates, neighbours, sides, orientation codes and mortar kinds of a small mesh."""
    if kind == "refined":
        X = inputs.refined_lattice(x, (2, 2, 1), (2, 2, 2))
        return (X, *inputs.connect_boxes(X, N + 1))
    if kind.startswith("box"):
        X = inputs.lattice_points(x, 2, 2, 3, box=(np.pi,) * 3)
        X = inputs.warp_sine(X) if kind == "box_curved" else X
        nbr, side, flip = inputs.box_lattice(2, 2, 3)
        rot = np.random.default_rng(N).integers(0, 24, len(X))
        X, nbr, side, flip, _ = inputs.rotate_elements(X, nbr, side, flip, N, rot)
        out = np.asarray(nbr) < 0  # every boundary kind in turn
        side = np.where(out, (np.arange(out.size).reshape(out.shape) // 2) % 5, side).astype(np.int8)
        return X, nbr, side, flip, None
    X = inputs.lattice_points(x, 2, 2, 3)
    nbr, side, flip = inputs.periodic_lattice(2, 2, 3)
    return (inputs.warp_sine(X) if kind in ("curved", "fv") else X), nbr, side, flip, None


def _copies(base, m):
    X, nbr, side, flip, mort = base
    K = len(X)
    off = np.repeat(np.arange(m) * K, K)[:, None]
    nb = np.tile(nbr, (m, 1))
    nb = np.where(nb >= 0, nb + off, nb).astype(np.int32)
    return np.tile(X, (m, 1, 1)), nb, np.tile(side, (m, 1)), np.tile(flip, (m, 1)), None if mort is None else np.tile(mort, (m, 1))


FORMS = [("split", "kep", "lgl", "ns", "roe"), ("split", "ec", "lgl", "ns", "volflux_roe"), ("split", "central", "lgl", "euler", "llf"),
         ("weak", "central", "lg", "euler", "llf"), ("weak", "central", "lg", "ns", "roe"), ("weak", "ec", "lgl", "euler", "volflux"),
         ("strong", "central", "lgl", "ns", "llf"), ("strong", "kep", "lg", "euler", "volflux_roe"), ("strong", "central", "lg", "ns", "roe")]


@pytest.mark.parametrize("kind", ["affine", "curved", "box", "box_curved", "refined", "fv"])
@pytest.mark.parametrize("form,vf,nodes,eqn,rs", FORMS, ids=["_".join(f) for f in FORMS])
def test_copies_of_a_mesh(dg, form, vf, nodes, eqn, rs, kind):
    import torch
    if kind == "fv" and eqn != "euler":
        pytest.skip("finite-volume elements: Euler only")
    for N in range(1, 9):
        print(f"case {form} {vf} {nodes} {eqn} {rs} {kind} N={N}", flush=True)
        x, _ = dg.nodes(N, "lgl")
        base = _base(kind, x, N)
        m = 512 // len(base[0]) + 1
        mu = 1e-2 if eqn == "ns" else 0.0
        sols = []
        for X, nbr, side, flip, mort in (base, _copies(base, m)):
            S = dg.DGSolver(np.ascontiguousarray(X), nbr, side, N, nodes, eqn, form, vf, rs, 1.4, 1.0, mu, 0.72, flip=flip, mortar=mort)
            if kind.startswith("box"):
                S.set_boundary_state(np.array([1.1, 0.2, -0.1, 0.1, 2.6]))
                S.set_wall_temperature(0.9)
                S.set_outflow_pressure(0.95)
            sols.append(S)
        K, n3 = len(base[0]), (N + 1) ** 3
        rng = np.random.default_rng(N)
        U = inputs.constant_state(K, n3)
        U = U * (1 + 0.02 * rng.standard_normal(U.shape))
        if kind == "fv":
            fv = (rng.random(K) < 0.4).astype(np.uint8)
            for S, t in zip(sols, (fv, np.tile(fv, m))):
                S.fv_enable(1, -5.0, -2.5)
                S.fv_set_types(t)
        u1 = torch.from_numpy(U).cuda()
        u2 = u1.repeat(m, 1, 1)
        got = []
        for S, u in zip(sols, (u1, u2)):
            R, o = torch.full_like(u, 0.5), S.empty()
            S.rk_stage(u, o, R, -0.4, 0.3, 1e-3)
            got.append((S.rhs(u), R, o))
        assert torch.isfinite(got[0][0]).all()
        for a, b in zip(*got):
            b = b.view(m, K, 5, n3)
            if form == "split":
                assert torch.equal(b, a.expand_as(b)), N
            else:
                assert float((b - a).abs().max() / a.abs().max()) <= 1e-12, N
