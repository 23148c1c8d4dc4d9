"""Reverse of the split form with the kinetic-energy preserving flux at every degree, on affine meshes (constant
metric terms) and curved ones, with each surface flux, and with every boundary kind: <J^T w, v> = <w, J v>
with J v from the oracle's tangent.  Bar: 1e-12 of the sum of the terms' magnitudes (both sides are sums of
rounded terms of that size)."""
import numpy as np
import pytest

from paper_1910_02858_amd import inputs
from gpu_common import gpu_solver, problem, to_gpu
from test_gpu_general_mesh import box_problem, box_solver

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dg():
    import torch
    from paper_1910_02858_amd import dgsem
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    dgsem.lib()
    return dgsem


def check(orc, wl, M, S, U0, seed):
    sc = orc.Scheme.of(wl)
    w = np.random.default_rng(seed).standard_normal(U0.shape)
    v = inputs.random_directions(U0, seed + 1, 1)[0]
    _, Jv = M.rhs_jvp(sc, U0, v)
    Ug, wg = to_gpu(U0), to_gpu(w)
    JTw = S.rhs_vjp(Ug, wg).cpu().numpy()
    lhs, rhs = float(np.sum(JTw * v)), float(np.sum(w * Jv))
    assert abs(lhs - rhs) <= 1e-12 * float(np.sum(np.abs(JTw * v)))
    assert np.array_equal(S.rhs_vjp(Ug, wg).cpu().numpy(), JTw)  # a fixed order of sums


@pytest.mark.parametrize("curved", [False, True], ids=["straight", "curved"])
@pytest.mark.parametrize("eqn,rs", [("ns", "roe"), ("ns", "llf"), ("euler", "volflux_roe"), ("euler", "volflux")])
def test_every_degree(dg, orc, eqn, rs, curved):
    for N in range(1, 9):
        print(f"case {eqn} {rs} N={N} curved={curved}", flush=True)
        wl = inputs.workload(5, eqn=eqn, riemann=rs, N=N, K1=2)
        M, xgeo, nbr, side, U0 = problem(orc, wl, kxyz=(3, 2, 2), curved=curved, perturb=1e-2, seed=N)
        check(orc, wl, M, gpu_solver(dg, wl, xgeo, nbr, side), U0, N)


BOXES = [("symmetry_rotated", 0, 8), ("given_state", 1, None), ("wall", 2, 5), ("isothermal_wall", 3, 7), ("outflow", 4, 6)]


@pytest.mark.parametrize("curved", [False, True], ids=["straight", "curved"])
@pytest.mark.parametrize("N", [1, 4, 5, 7])
@pytest.mark.parametrize("name,kind,seed", BOXES, ids=[b[0] for b in BOXES])
def test_boundaries(dg, orc, name, kind, seed, N, curved):
    print(f"case {name} N={N} curved={curved}", flush=True)
    wl = inputs.workload(5, N=N, mach=0.3)
    M, (X, nbr, side, flip), U0 = box_problem(orc, wl, 2, seed=seed, curved=curved, perturb=1e-2, kind=kind)
    check(orc, wl, M, box_solver(dg, wl, X, nbr, side, flip, kind=kind), U0, 10 + N)
