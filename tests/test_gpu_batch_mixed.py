"""Batches that mix members on affine and on curved meshes within a degree, in orders that leave ragged last
workgroups in both groups: the bits of the one-mesh stages and steps for every tile that the degree offers, for the
single pair of launches, and replayed from graphs; dg_batch_info counts a degree once."""
import numpy as np
import pytest

from paper_1910_02858_amd import inputs
from gpu_common import gpu_solver, to_gpu

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dg():
    import torch
    from paper_1910_02858_amd import dgsem
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    dgsem.lib()
    return dgsem


SIZES = ((2, 3, 2), (1, 1, 1), (3, 1, 1), (1, 5, 1), (1, 2, 3))


def _members(dg, orc, degrees, curved):
    sols, Us = [], []
    for N in degrees:
        wl = inputs.workload(2, N=N)
        for i, (k, cv) in enumerate(zip(SIZES, curved)):
            X = inputs.lattice_points(orc.basis(N, "lgl")["x"], *k) - 1.0
            nbr, side, _ = inputs.periodic_lattice(*k)
            S = gpu_solver(dg, wl, inputs.warp_sine(X) if cv else X, nbr, side)
            sols.append(S)
            Us.append(to_gpu(inputs.random_perturbation(inputs.initial_state(wl, S.node_coords()), 7 * N + i, 1e-2)))
    return sols, Us


@pytest.mark.parametrize("curved", [(0, 1, 0, 1, 1), (1, 0, 1, 1, 0), (0, 0, 0, 0, 1)], ids=["acacc", "cacca", "aaaac"])
@pytest.mark.parametrize("degrees", [(1, 2, 3), (4, 5), (3, 7), (6, 8)], ids=["1-3", "4-5", "3-7", "6-8"])
def test_mixed_members_keep_their_bits(dg, orc, degrees, curved):
    import torch
    print(f"case {degrees} {curved}", flush=True)
    sols, Us = _members(dg, orc, degrees, curved)
    ref = []
    for S, U in zip(sols, Us):
        o, R = S.empty(), torch.full_like(U, 0.5)
        S.rk_stage(U, o, R, -0.4, 0.3, 1e-3)
        ref.append((o, R))
    B = dg.Batch(sols)
    modes = [(False, 1), (False, 2), (False, 4)] + ([(True, 0)] if max(degrees) <= 7 else [])
    for fused, epb in modes:
        B.fused = fused
        if not fused:
            for N in degrees:
                e = min(epb, 4 if N <= 3 else (2 if N <= 5 else 1))
                B.set_tile(N, e, e)
            assert [t[:3] for t in B.info()] == [(N, 5, sum(int(np.prod(k)) for k in SIZES)) for N in degrees]
        outs, Rs = [S.empty() for S in sols], [torch.full_like(U, 0.5) for U in Us]
        B.rk_stage(Us, outs, Rs, -0.4, 0.3, 1e-3)
        torch.cuda.synchronize()
        for i, ((o, R), o2, R2) in enumerate(zip(ref, outs, Rs)):
            assert torch.equal(o, o2) and torch.equal(R, R2), (i, fused, epb)
        cur, nxt, Rs = [U.clone() for U in Us], [S.empty() for S in sols], [torch.zeros_like(U) for U in Us]
        for _ in range(4):  # two argument sets, each replayed
            B.step(cur, nxt, Rs, 1e-3)
            cur, nxt = nxt, cur
        torch.cuda.synchronize()
        for i, (S, U, got) in enumerate(zip(sols, Us, cur)):
            assert torch.equal(S.steps(U.clone(), 4, 1e-3), got), (i, fused, epb)
