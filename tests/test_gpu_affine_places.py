"""Affine meshes away from the origin, turned and sheared, and meshes that are nearly affine.  A uniform flow
stays uniform and every state is conserved to the bars of the lattice at the origin (1e-12 of the flux scale,
1e-13 of the quadrature of |U_t|), whether the metric terms are constants of the element or, where the coordinates'
rounding is too coarse for that, per node; and the operator is the oracle's on the same coordinates (1e-12 of the
whole vector)."""
import numpy as np
import pytest

from paper_1910_02858_amd import inputs
from gpu_common import gpu_solver, norm_err, to_gpu

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dg():
    import torch
    from paper_1910_02858_amd import dgsem
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    dgsem.lib()
    return dgsem


SHEAR = np.array([[1.0, 0.2, -0.1], [0.15, 0.9, 0.25], [-0.2, 0.1, 1.1]])


def _turn(X, t=0.3):
    c, s = np.cos(t), np.sin(t)
    return np.stack((c * X[:, 0] - s * X[:, 1], s * X[:, 0] + c * X[:, 1], X[:, 2]), 1)


def _shear(X):
    return np.einsum("cd,kdq->kcq", SHEAR, X)


PLACES = {"centred": lambda X: X - np.pi, "turned": _turn, "sheared": _shear, "sheared_1e3": lambda X: _shear(X) + 1e3,
          "sheared_1e6": lambda X: _shear(X) + 1e6}
def _lattice(x, k, place):
    """A periodic lattice whose nodes are placed once each: two elements have the same coordinates on the face they
    share, and the same up to one translation on a periodic face."""
    n = x.size
    pos = [np.append((np.arange(m)[:, None] + 0.5 * (x[:-1] + 1)).ravel(), m) * (2 * np.pi / m) for m in k]
    shape = tuple(p.size for p in pos[::-1])
    P = np.stack(np.broadcast_arrays(pos[0][None, None, :], pos[1][None, :, None], pos[2][:, None, None]))
    P = PLACES[place](P.reshape(1, 3, -1)).reshape((3,) + shape)
    for ax in (3, 2, 1):
        first, last = (np.take(P, [i], ax) for i in (0, -1))
        shift = (last - first)[:, :1, :1, :1]
        P = np.concatenate((np.delete(P, -1, ax), first + shift), ax)
    X = np.empty((k[0] * k[1] * k[2], 3, n, n, n))
    for e in range(len(X)):
        i, j, l = e % k[0] * (n - 1), e // k[0] % k[1] * (n - 1), e // (k[0] * k[1]) * (n - 1)
        X[e] = P[:, l:l + n, j:j + n, i:i + n]
    return np.ascontiguousarray(X.reshape(len(X), 3, -1))


FORMS = [("split", "ec", "lgl", "ns", 7), ("split", "kep", "lgl", "euler", 3), ("weak", "central", "lg", "euler", 3),
         ("weak", "central", "lg", "ns", 5), ("weak", "central", "lgl", "ns", 4), ("strong", "central", "lgl", "ns", 4),
         ("strong", "central", "lg", "euler", 6)]


@pytest.mark.parametrize("place", list(PLACES))
@pytest.mark.parametrize("form,vf,nodes,eqn,N", FORMS, ids=["_".join(map(str, f)) for f in FORMS])
def test_freestream_conservation_and_parity(dg, orc, form, vf, nodes, eqn, N, place):
    print(f"case {form} {vf} {nodes} {eqn} {N} {place}", flush=True)
    k = (12, 3, 2)
    wl = inputs.workload(2, eqn=eqn, form=form, volflux=vf, riemann="roe", nodes=nodes, N=N)
    X = _lattice(orc.basis(N, "lgl")["x"], k, place)
    nbr, side, _ = inputs.periodic_lattice(*k)
    M = orc.OracleMesh(X, nbr, side, N, nodes)
    S = gpu_solver(dg, wl, X, nbr, side)
    Uc = inputs.constant_state(M.K, M.n3)
    Ut = S.rhs(to_gpu(Uc)).cpu().numpy()
    fscale = np.abs(Uc).max() * 2 * (N + 1) ** 2 / (2 * np.pi / 12)
    print("free stream", np.abs(Ut).max() / fscale, flush=True)
    assert np.abs(Ut).max() < 1e-12 * fscale
    # a state without a large mean pressure: its cancellation is not what is looked at here
    rng = np.random.default_rng(5)
    U = inputs.constant_state(M.K, M.n3)
    U = U * (1 + 0.1 * rng.standard_normal(U.shape))
    Utg = S.rhs(to_gpu(U))
    tot = S.integrals(Utg)[:5]
    w = orc.basis(N, nodes)["w"]
    wq = np.einsum("k,j,i->kji", w, w, w).ravel()[None] * M.geometry()["J"]
    scale = np.einsum("eq,evq->v", wq, np.abs(Utg.cpu().numpy()))
    print("conservation", np.abs(tot / scale).max(), flush=True)
    assert np.all(np.abs(tot) < 1e-13 * scale), (tot, scale)
    err = norm_err(Utg.cpu().numpy(), M.rhs(orc.Scheme.of(wl), U))
    print("parity", err, flush=True)
    assert err <= 1e-12


@pytest.mark.parametrize("N", [2, 4, 7])
@pytest.mark.parametrize("move", [1e-13, 1e-11, 1e-9])
def test_nearly_affine_against_the_moved_mesh(dg, orc, N, move):
    """One inner node moved by ``move`` of an element: the per-node path, on the moved mesh's metric terms.  The
    constants of the unmoved one would miss the bar by the derivative's share of it from 1e-11 on."""
    k = (2, 3, 2)
    wl = inputs.workload(2, N=N)
    x = orc.basis(N, "lgl")["x"]
    X = _shear(inputs.lattice_points(x, *k))
    n = N + 1
    X[1, 0, 1 + n * (1 + n)] += move * np.pi
    X = np.ascontiguousarray(X)
    nbr, side, _ = inputs.periodic_lattice(*k)
    M = orc.OracleMesh(X, nbr, side, N, "lgl")
    U = inputs.random_perturbation(inputs.initial_state(wl, M.points()), 3, 1e-2)
    S = gpu_solver(dg, wl, X, nbr, side)
    assert norm_err(S.rhs(to_gpu(U)).cpu().numpy(), M.rhs(orc.Scheme.of(wl), U)) <= 1e-12


@pytest.mark.parametrize("vf,eqn", [("kep", "ns"), ("ec", "euler")])
def test_degree_1_curved(dg, orc, vf, eqn):
    """Degree 1 has no inner node to move: a warped lattice takes the per-node path."""
    wl = inputs.workload(2, N=1, volflux=vf, eqn=eqn)
    X = inputs.warp_sine(inputs.lattice_points(orc.basis(1, "lgl")["x"], 4, 3, 4))
    nbr, side, _ = inputs.periodic_lattice(4, 3, 4)
    M = orc.OracleMesh(X, nbr, side, 1, "lgl")
    U = inputs.random_perturbation(inputs.initial_state(wl, M.points()), 3, 1e-2)
    S = gpu_solver(dg, wl, X, nbr, side)
    assert norm_err(S.rhs(to_gpu(U)).cpu().numpy(), M.rhs(orc.Scheme.of(wl), U)) <= 1e-12


@pytest.mark.parametrize("place", ["centred", "sheared_1e3"])
@pytest.mark.parametrize("form,vf,nodes,eqn", [("split", "kep", "lgl", "ns"), ("weak", "central", "lg", "euler"),
                                               ("weak", "central", "lg", "ns")])
def test_refined_lattice_freestream_and_conservation(dg, orc, form, vf, nodes, eqn, place):
    """Non-conforming faces: their fluxes take the small sides' normals.  Bars as for the refined mesh at the origin."""
    print(f"case {form} {vf} {nodes} {eqn} {place}", flush=True)
    N = 4
    wl = inputs.workload(2, eqn=eqn, form=form, volflux=vf, riemann="roe", nodes=nodes, N=N)
    x = orc.basis(N, "lgl")["x"]
    X0 = inputs.refined_lattice(x, (4, 2, 2), (2, 2, 2))
    nbr, side, flip, mort = inputs.connect_boxes(X0, N + 1)
    X = np.ascontiguousarray(PLACES[place](X0))
    M = orc.OracleMesh(X, nbr, side, N, nodes, flip=flip, mortar=mort)
    S = dg.DGSolver.from_workload(wl, X, nbr, side, flip=flip, mortar=mort)
    Uc = inputs.constant_state(M.K, M.n3)
    Ut = S.rhs(to_gpu(Uc)).cpu().numpy()
    fscale = np.abs(Uc).max() * 2 * (N + 1) ** 2 / (np.pi / 4)
    print("free stream", np.abs(Ut).max() / fscale, flush=True)
    U = Uc * (1 + 0.1 * np.random.default_rng(5).standard_normal(Uc.shape))
    Utg = S.rhs(to_gpu(U))
    tot = S.integrals(Utg)[:5]
    w = orc.basis(N, nodes)["w"]
    wq = np.einsum("k,j,i->kji", w, w, w).ravel()[None] * M.geometry()["J"]
    scale = np.einsum("eq,evq->v", wq, np.abs(Utg.cpu().numpy()))
    print("conservation", np.abs(tot / scale).max(), flush=True)
    assert np.abs(Ut).max() < 1e-12 * fscale
    assert np.all(np.abs(tot) < 1e-13 * scale), (tot, scale)


@pytest.mark.parametrize("N", [3, 7])
def test_which_metric_terms_are_read(dg, orc, N):
    """dg_affine: a lattice, shifted or turned, reads one set per element; a curved mesh and a lattice with one node
    moved by more than rounding read them at every node."""
    k = (12, 3, 2)
    wl = inputs.workload(2, N=N)
    nbr, side, _ = inputs.periodic_lattice(*k)
    X = _lattice(orc.basis(N, "lgl")["x"], k, "turned")
    moved, P = X.copy(), inputs.lattice_points(orc.basis(N, "lgl")["x"], *k)
    moved[1, 0, 1 + (N + 1) * (N + 2)] += 1e-9  # an inner node
    curved = P + 0.02 * np.sin(P[:, [1, 2, 0]])  # periodic like the lattice
    assert [gpu_solver(dg, wl, np.ascontiguousarray(x), nbr, side).affine for x in (X, moved, curved)] == [True, False, False]
