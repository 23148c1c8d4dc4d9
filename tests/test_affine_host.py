"""Which meshes count as affine, and their constants, on the CPU: lattices wherever they lie and however they are
turned, as long as what they deviate by is rounding; never a mesh that is curved by more, nor one so far from the
origin that its coordinates no longer resolve the elements' shape.  The constants: Ja^dir is bit for bit the same
vector on both sides of every conforming face, and within the rounding of the coordinates of the exact one."""
import ctypes
import os
import subprocess

import numpy as np
import pytest

from paper_1910_02858_amd import inputs

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SHEAR = np.array([[1.0, 0.2, -0.1], [0.15, 0.9, 0.25], [-0.2, 0.1, 1.1]])


@pytest.fixture(scope="module")
def affine(tmp_path_factory):
    so = str(tmp_path_factory.mktemp("affine") / "affine.so")
    subprocess.run(["g++", "-O2", "-std=c++17", "-pthread", "-shared", "-fPIC",
                    os.path.join(ROOT, "tests", "affine_selftest.cpp"), "-o", so], check=True)
    f = ctypes.CDLL(so).affine

    def call(x, X, nbr, side, mort=None):
        X, x = np.ascontiguousarray(X), np.ascontiguousarray(x)
        C = np.zeros((X.shape[0], 28))
        p = [a if a is None else a.ctypes.data_as(ctypes.c_void_p) for a in (x, X, nbr, side, mort, C)]
        return C if f(X.shape[0], x.size, *p) else None

    return call


def _turn(X, t):
    c, s = np.cos(t), np.sin(t)
    return np.stack((c * X[:, 0] - s * X[:, 1], s * X[:, 0] + c * X[:, 1], X[:, 2]), 1)


PLACES = {
    "corner_at_0": lambda X: X, "centred": lambda X: X - np.pi, "unit_box": lambda X: X / (2 * np.pi) - 0.5,
    "turned": lambda X: _turn(X, 0.3), "centred_turned": lambda X: _turn(X - np.pi, 0.3),
    "sheared": lambda X: np.einsum("cd,kdq->kcq", SHEAR, X),
    "stretched": lambda X: X * np.array([1.0, 1e-3, 40.0])[:, None],
}


@pytest.mark.parametrize("place", list(PLACES))
def test_lattices_are_affine(orc, affine, place):
    for N, k in ((7, (32, 4, 32)), (7, (16, 5, 16)), (5, (16, 16, 4)), (5, (12, 12, 12)), (4, (18, 5, 18)), (3, (48, 4, 48)),
                 (2, (60, 3, 60)), (1, (96, 3, 96)), (8, (4, 4, 4)), (7, (1, 2, 1))):
        x = orc.basis(N, "lgl")["x"]
        nbr, side, _ = inputs.periodic_lattice(*k)
        C = affine(x, PLACES[place](inputs.lattice_points(x, *k)), nbr, side)
        assert C is not None, (place, N, k)


def _box(orc, N, k, seed=None):
    """A box with boundary sides, its elements' axes turned if a seed is given."""
    x = orc.basis(N, "lgl")["x"]
    X = inputs.lattice_points(x, k, k, k, box=(np.pi,) * 3)
    nbr, side, flip = inputs.box_lattice(k, k, k)
    if seed is not None:
        rot = np.random.default_rng(seed).integers(0, 24, k ** 3)
        X, nbr, side, flip, _ = inputs.rotate_elements(X, nbr, side, flip, N, rot)
    return x, X, nbr, side


@pytest.mark.parametrize("name", ["lattice", "centred_turned", "sheared", "axes_turned", "stretched"])
def test_constants_continuous_and_exact(orc, affine, name):
    N, k = 4, 6
    if name == "axes_turned":
        x, X, nbr, side = _box(orc, N, k, 3)
    else:
        x = orc.basis(N, "lgl")["x"]
        X = PLACES.get(name, PLACES["corner_at_0"])(inputs.lattice_points(x, k, k, k))
        nbr, side, _ = inputs.periodic_lattice(k, k, k)
    C = affine(x, X, nbr, side)
    assert C is not None
    nt = C[:, 10:].reshape(-1, 6, 3)
    Ja = C[:, :9].reshape(-1, 3, 3)
    e, s = np.nonzero(nbr >= 0)
    assert np.array_equal(nt[nbr[e, s], side[e, s]], -nt[e, s])
    assert np.array_equal(nt[:, 1::2], Ja) and np.array_equal(nt[:, ::2], -Ja)
    # from the corners: a_d = dx/dxi_d in extended precision; both differ by the rounding of the coordinates, eight
    # of which enter each edge: 8 ulp of the largest coordinate over the smallest edge, twice
    n = N + 1
    Y = X.reshape(-1, 3, n, n, n).astype(np.longdouble)
    o = Y[:, :, 0, 0, 0]
    A = [(v - o) / 2 for v in (Y[:, :, 0, 0, -1], Y[:, :, 0, -1, 0], Y[:, :, -1, 0, 0])]
    ln = np.array([np.sqrt((a * a).sum(1)) for a in A])
    rel = 16 * 2.3e-16 * float((np.abs(X).max((0, 2)) / ln.min(1).astype(float)).max())
    for d in range(3):
        p, q = A[(d + 1) % 3], A[(d + 2) % 3]
        ref = np.stack([p[:, (m + 1) % 3] * q[:, (m + 2) % 3] - p[:, (m + 2) % 3] * q[:, (m + 1) % 3] for m in range(3)], 1)
        scale = ln[(d + 1) % 3] * ln[(d + 2) % 3]
        assert float((np.abs(Ja[:, d] - ref) / scale[:, None]).max()) <= rel
        if d == 0:
            J = (A[0] * ref).sum(1)
            assert float(np.abs(C[:, 9] * J - 1).max()) <= 2 * rel * float((ln[0] * ln[1] * ln[2] / J).max())
    # an element's constants do not depend on the numbering
    rnd = np.random.default_rng(1).permutation(len(X))
    inv = np.argsort(rnd)
    nb2 = np.where(nbr[rnd] >= 0, inv[nbr[rnd]], -1).astype(nbr.dtype)
    assert np.array_equal(affine(x, X[rnd], np.ascontiguousarray(nb2), np.ascontiguousarray(side[rnd])), C[rnd])


@pytest.mark.parametrize("N", [2, 4, 7])
def test_what_is_not_affine(orc, affine, N):
    x = orc.basis(N, "lgl")["x"]
    n, k = N + 1, 4
    nbr, side, _ = inputs.periodic_lattice(k, k, k)
    X = inputs.lattice_points(x, k, k, k)
    h = 2 * np.pi / k
    mid = 1 + n * (1 + n)
    for move, is_affine in ((4e-16, True), (1e-12 * h, False), (1e-9 * h, False), (1.1e-13 * h, False)):
        Y = X.copy()
        Y[5, 0, mid] += move
        assert (affine(x, Y, nbr, side) is not None) == is_affine, move
    Y = X.copy()
    Y[5, 1, mid] = np.nan
    assert affine(x, Y, nbr, side) is None
    assert affine(x, inputs.warp_sine(X), nbr, side) is None
    for shift in (1e3, 1e6):  # the coordinates' rounding is 1e-13 and 1e-10 of an element
        k2 = (24, 4, 4)
        X2 = inputs.lattice_points(x, *k2) + shift
        nb2, sd2, _ = inputs.periodic_lattice(*k2)
        assert affine(x, X2, nb2, sd2) is None


def test_slow_taper_is_not_affine(orc, affine):
    """A wedge whose cells grow by 7e-15 of their height each (an element's rounding, and affine over a few cells),
    over 400 cells: the ends of the chain differ by 3e-12."""
    def wedge(k, taper, first=0):
        X = np.zeros((k, 3, 8))
        for e in range(k):
            for q in range(8):
                i, j, l = q & 1, (q >> 1) & 1, q >> 2
                X[e, :, q] = (first + e + i) / 4096.0, j * (1 + taper * (first + e + i)) / 64.0, l / 64.0
        nbr, side = np.full((k, 6), -1, np.int32), np.zeros((k, 6), np.int8)
        nbr[:-1, 1], side[:-1, 1] = np.arange(1, k), 0
        nbr[1:, 0], side[1:, 0] = np.arange(k - 1), 1
        return X, nbr, side

    x = orc.basis(1, "lgl")["x"]
    assert affine(x, *wedge(400, 0.0)) is not None
    assert affine(x, *wedge(4, 2.0 ** -47, 396)) is not None
    assert affine(x, *wedge(400, 2.0 ** -47)) is None


def test_mortar_sides_are_not_tied(orc, affine):
    """A locally refined lattice: the big element's Ja is four times the small ones', not one chain."""
    N = 3
    x = orc.basis(N, "lgl")["x"]
    X = inputs.refined_lattice(x, (2, 2, 2), (2, 2, 2))
    nbr, side, flip, mort = inputs.connect_boxes(X, N + 1)
    C = affine(x, X, nbr, side, mort)
    assert C is not None
    area = np.abs(C[:, 0])
    assert np.isclose(area.max() / area.min(), 4.0)


@pytest.mark.parametrize("N", [2, 3, 7])
def test_every_node_decides_near_the_limit(orc, affine, N):
    """Single sheared elements far enough from the origin that the rounding of their coordinates is about the share
    of the element that counts as rounding: accepted exactly where every node's own deviation is within it, also
    where the largest deviations of the three coordinates, taken together, are not."""
    x = orc.basis(N, "lgl")["x"]
    n, rng = N + 1, np.random.default_rng(N)
    nbr, side = np.full((1, 6), -1, np.int32), np.zeros((1, 6), np.int8)
    xl = x.astype(np.longdouble)
    ref = np.stack((np.tile(xl, n * n), np.tile(np.repeat(xl, n), n), np.repeat(xl, n * n)))
    accepted = rejected = together_only = 0
    for _ in range(400):
        A0 = np.eye(3) + 0.4 * rng.standard_normal((3, 3))
        if np.linalg.det(A0) < 0.2:
            continue
        X = (A0.T @ ref.astype(float) + rng.uniform(200, 3200, (3, 1)) / n)[None]
        Y = X[0].astype(np.longdouble).reshape(3, n, n, n)
        Y = Y - Y[:, :1, :1, :1]
        cs = Y[:, ::N, ::N, ::N]
        c = cs.mean((1, 2, 3))
        A = np.stack([(np.take(cs, 1, a) - np.take(cs, 0, a)).mean((1, 2)) / 2 for a in (3, 2, 1)])
        v = Y.reshape(3, -1) - c[:, None] - A.T @ ref
        Ja = np.stack([np.cross(A[(i + 1) % 3], A[(i + 2) % 3]) for i in range(3)])
        J, limit = A[0] @ Ja[0], 2 * np.longdouble(1.6e-13) / n
        moved, together = np.abs(Ja @ v).max() / J, (np.abs(Ja) @ np.abs(v).max(1)).max() / J
        if abs(moved / limit - 1) < 1e-6:  # the two sums' own rounding
            continue
        ok = bool(moved <= limit)
        assert np.abs(v).max() <= 4 * 2.0 ** -52 * np.abs(X).max()
        assert (affine(x, X, nbr, side) is not None) == ok, (moved, limit)
        accepted, rejected, together_only = accepted + ok, rejected + (not ok), together_only + (ok and together > limit)
    print(accepted, rejected, together_only)
    assert min(accepted, rejected, together_only) >= 10
