"""The ways out of a solve other than convergence, in every form of the iteration.

Non-finite: a field whose sums overflow at the start (w.r), in the first product
(p.Ap; a checkerboard, for which p.Ap is nearly 2 w.r) or in the first update (a long
wave, whose residual the first step amplifies).  The step returns
LF_ENONFINITE, counts the iterations before, leaves T as it was, and the next
step from a good field is that of a fresh problem.  Singular: a zero field and
minIter = 1 break at p.Ap = 0 with no iteration counted, as the oracle does; and the
iteration limits end the loop at the oracle's iterates.
"""
import numpy as np
import pytest

import synth
from tests.gpu_common import lapfoam, max_rel

pytestmark = pytest.mark.gpu

# shape, numbering seed, amul_walk, form
FP64 = {"two_launches": ((20, 18, 16), 0, 0, 0), "two_launches_rows": ((20, 18, 16), 3, 0, 0),
        "two_launches_more_rows": ((82, 81, 80), 0, 0, 0), "five_launches": ((139, 138, 137), 0, 2, 0),
        "row_walk": ((21, 18, 16), 0, 1, 1), "block_walk": ((20, 18, 16), 0, 1, 2),
        "scaled": ((104, 104, 104), 0, 1, 4)}
MIXED = {"two_launches": ((20, 18, 16), 0, 0, 0), "two_launches_rows": ((20, 18, 16), 3, 0, 0),
         "two_launches_more_rows": ((66, 64, 64), 0, 0, 0), "one_workgroup_start": ((130, 128, 128), 0, 0, 0),
         "five_launches_rows": ((129, 128, 96), 3, 0, 0), "row_walk": ((21, 18, 16), 0, 1, 1),
         "block_walk": ((20, 18, 16), 0, 1, 2), "block_and_row_walk": ((22, 18, 16), 0, 1, 2)}


def _mesh(shape, seed):
    mesh = synth.box_mesh(*shape)
    return synth.renumber(mesh, synth.random_permutation(mesh.n_cells, seed)) if seed else mesh


def _first_residual(mesh, T, DT, dt):
    """b - A T and the diagonal of one step with zeroGradient walls."""
    d = mesh.cell_centre[mesh.neighbour] - mesh.cell_centre[mesh.owner]
    mag = np.linalg.norm(mesh.face_area, axis=1)
    up = DT * mag / ((mesh.face_area * d).sum(1) / mag)
    n = mesh.n_cells
    diag = mesh.cell_volume / dt + np.bincount(mesh.owner, up, n) + np.bincount(mesh.neighbour, up, n)
    flux = up * (T[mesh.neighbour] - T[mesh.owner])
    return np.bincount(mesh.owner, flux, n) - np.bincount(mesh.neighbour, flux, n), diag


def _field(mesh, where, single):
    """A field at which the given sum is the first to overflow (single: an FP32 vector)."""
    x = mesh.cell_centre
    if where == "update":
        T = np.cos(np.pi * x[:, 0])
    else:
        T = (-1.0) ** np.floor(x * np.array(mesh.shape)).sum(1)
    r, diag = _first_residual(mesh, T, 1.0, 1.0)
    if single:
        top = {"start": 1e39, "product": 2.5e38, "update": 2.5e38}[where]
        return T * (top / np.max(np.abs(r) / np.sqrt(diag)))
    if where == "start":
        return T * 1e200
    return T * (np.sqrt(1.2e308) / np.sqrt(np.sum(r * r / diag)))


def _check(L, shape, seed, walk, form, where, **opts):
    mesh = _mesh(shape, seed)
    bcs = synth.all_zero_gradient()
    single = bool(opts)
    m = L.Mesh(mesh)
    P = L.Problem(m, bcs, 1.0, 1.0, L.make_opts(amul_walk=walk, **opts))
    assert P.amul_form() == form
    T0 = _field(mesh, where, single)
    P.set_T(T0)
    st, status = P.step(1, check=False)
    assert status == L.LF_ENONFINITE and st[0]["nonfinite"] == 1 and st[0]["converged"] == 0, st
    assert st[0]["n_iter"] == (1 if where == "update" else 0), st
    if form == 4:       # x sqrt(d) / sqrt(d): two roundings
        assert np.allclose(P.get_T(), T0, rtol=4e-16, atol=0.0)
    else:
        assert np.array_equal(P.get_T(), T0)
    good = synth.initial_field(mesh.n_cells, 8)
    out = []
    Q = L.Problem(m, bcs, 1.0, 1.0, L.make_opts(amul_walk=walk, **opts))
    for X in (P, Q):
        X.set_T(good)
        st, _ = X.step(1)
        out.append((X.get_T(), st[0]["n_iter"], st[0]["initial_residual"]))
        X.close()
    assert np.array_equal(out[0][0], out[1][0]) and out[0][1:] == out[1][1:]
    m.close()


@pytest.mark.parametrize("where", ["start", "product", "update"])
@pytest.mark.parametrize("name", list(FP64))
def test_nonfinite_fp64(name, where):
    _check(lapfoam(), *FP64[name], where)


@pytest.mark.parametrize("where", ["start", "product", "update"])
@pytest.mark.parametrize("name", list(MIXED))
def test_nonfinite_mixed(name, where):
    L = lapfoam()
    _check(L, *MIXED[name], where, precision=L.LF_PREC_MIXED)


@pytest.mark.parametrize("name", ["two_launches_more_rows", "five_launches", "row_walk", "block_walk", "scaled"])
def test_singular(oracle, name):
    L = lapfoam()
    shape, seed, walk, form = FP64[name]
    mesh = _mesh(shape, seed)
    m = L.Mesh(mesh)
    P = L.Problem(m, synth.all_zero_gradient(), 1e-3, 1e-3, L.make_opts(amul_walk=walk, min_iter=1))
    assert P.amul_form() == form
    P.set_T(np.zeros(mesh.n_cells))
    st, _ = P.step(2)
    _, so, _ = oracle.run(mesh, synth.all_zero_gradient(), 1e-3, 1e-3, 1, np.zeros(mesh.n_cells), min_iter=1)
    for s in st:
        assert s["singular"] == so[0]["singular"] == 1 and s["n_iter"] == so[0]["n_iter"] == 0
        assert s["nonfinite"] == 0
    assert np.array_equal(P.get_T(), np.zeros(mesh.n_cells))
    P.close()
    m.close()


@pytest.mark.parametrize("name", ["five_launches", "row_walk", "block_walk", "scaled"])
@pytest.mark.parametrize("max_iter,min_iter,tol", [(0, 0, 1e-9), (1, 0, 1e-9), (2, 0, 1e-9), (1000, 3, 1.0),
                                                   (1000, 0, 1.0)])
def test_limits(oracle, name, max_iter, min_iter, tol):
    L = lapfoam()
    shape, seed, walk, form = FP64[name]
    mesh = _mesh(shape, seed)
    T0 = synth.initial_field(mesh.n_cells, 12)
    m = L.Mesh(mesh)
    P = L.Problem(m, synth.fixed_x_bcs(), 1e-3, 1e-3,
                  L.make_opts(tol=tol, max_iter=max_iter, min_iter=min_iter, amul_walk=walk))
    assert P.amul_form() == form
    P.set_T(T0)
    st, _ = P.step(1)
    T, so, _ = oracle.run(mesh, synth.fixed_x_bcs(), 1e-3, 1e-3, 1, T0, tol=tol, max_iter=max_iter, min_iter=min_iter)
    assert st[0]["n_iter"] == so[0]["n_iter"] and st[0]["converged"] == so[0]["converged"]
    # the same iterates to rounding: a few iterations from the same start
    assert max_rel(P.get_T(), T) <= 1e-12, max_rel(P.get_T(), T)
    P.close()
    m.close()
