"""Non-conforming faces at the ends of the degrees' range (one lane per small-side point: 16 lanes of 64 at
N = 1, 324 of 384 at N = 8) for the three mortar types, against the oracle; bar 1e-12 as for every operator
evaluation."""
import pytest

from paper_1910_02858_amd import inputs
from gpu_common import check_rhs, to_gpu
from test_gpu_mortar import dg, mortar_problem, mortar_solver  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("split", [(2, 2, 2), (1, 2, 1), (1, 1, 2)], ids=["type3", "type1", "type2"])
@pytest.mark.parametrize("N,form,nodes", [(1, "split", "lgl"), (2, "weak", "lg"), (8, "split", "lgl"), (8, "weak", "lg")])
def test_mortar_degrees(dg, orc, N, form, nodes, split):  # noqa: F811
    wl = inputs.workload(2, N=N, form=form, nodes=nodes, volflux="kep" if form == "split" else "central")
    M, mesh, U0 = mortar_problem(orc, wl, 2, split, rot_seed=N)
    S = mortar_solver(dg, wl, 2, mesh)
    check_rhs(S.rhs(to_gpu(U0)).cpu().numpy(), M.rhs(orc.Scheme.of(wl), U0))
