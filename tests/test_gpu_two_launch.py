"""FP64 diagonal solves with two launches per iteration, at the edges of their rules.

Up to 2^19 rows the kernels take one row per thread, up to 5 * 2^19 two or four,
above that (without a walk: an odd x side) the five-launch form runs; workgroups
take contiguous shares per die up to 3 * 2^19.  A box of 2.5 M rows takes the
block walk.  Steps against the oracle within the
FP64 parity bar (1e-8 relative, iterations within one) on every layout the form
accepts: one to four bands and the row layout.
"""
import numpy as np
import pytest

import synth
from tests.gpu_common import lapfoam, max_rel

pytestmark = pytest.mark.gpu


def _box(name):
    shape, numbering = {
        "one_cell": ((1, 1, 1), None), "line_513": ((513, 1, 1), None), "plane_2_bands": ((33, 31, 1), None),
        "rows_below_one_row": ((80, 80, 81), "random"), "bands_at_one_row": ((128, 64, 64), None),
        "bands_above_one_row": ((81, 81, 81), None), "rows_above_one_row": ((81, 81, 81), "random"),
        "above_die_shares": ((117, 117, 117), None), "at_most_rows": ((137, 138, 138), None),
        "above_most_rows": ((139, 138, 137), None), "block_walk": ((136, 136, 134), None)}[name]
    mesh = synth.box_mesh(*shape, z_ratio=1.0 if min(shape) == 1 else 3.0)
    if numbering:
        mesh = synth.renumber(mesh, synth.random_permutation(mesh.n_cells, 5))
    return mesh


@pytest.mark.parametrize("name", ["one_cell", "line_513", "plane_2_bands", "rows_below_one_row", "bands_at_one_row",
                                  "bands_above_one_row", "rows_above_one_row", "above_die_shares", "at_most_rows",
                                  "above_most_rows", "block_walk"])
def test_steps(oracle, name):
    L = lapfoam()
    mesh = _box(name)
    T0 = synth.initial_field(mesh.n_cells, 11)
    m = L.Mesh(mesh)
    P = L.Problem(m, synth.fixed_x_bcs(), 1e-3, 1e-3)
    assert P.amul_form() == (4 if name == "block_walk" else 0)
    P.set_T(T0)
    stats, _ = P.step(2)
    T, so, _ = oracle.run(mesh, synth.fixed_x_bcs(), 1e-3, 1e-3, 2, T0)
    assert max_rel(P.get_T(), T) <= 1e-8, max_rel(P.get_T(), T)
    for a, b in zip(stats, so):
        assert a["converged"] == 1 and abs(a["n_iter"] - b["n_iter"]) <= 1
        assert abs(a["initial_residual"] - b["initial_residual"]) <= 1e-9 * b["initial_residual"]
    P.close()
    m.close()


@pytest.mark.parametrize("shape", [(20, 21, 22), (81, 81, 81)], ids=["one_row", "two_rows"])
@pytest.mark.parametrize("max_iter,min_iter,tol", [(0, 0, 1e-9), (1, 0, 1e-9), (2, 0, 1e-9), (1000, 3, 1.0),
                                                   (1000, 0, 1.0)])
def test_iteration_limits(oracle, shape, max_iter, min_iter, tol):
    """The checks' semantics: every exit of the loop applies the same updates."""
    L = lapfoam()
    mesh = synth.box_mesh(*shape)
    T0 = synth.initial_field(mesh.n_cells, 12)
    m = L.Mesh(mesh)
    P = L.Problem(m, synth.fixed_x_bcs(), 1e-3, 1e-3, L.make_opts(tol=tol, max_iter=max_iter, min_iter=min_iter))
    P.set_T(T0)
    st, _ = P.step(1)
    T, so, _ = oracle.run(mesh, synth.fixed_x_bcs(), 1e-3, 1e-3, 1, T0, tol=tol, max_iter=max_iter, min_iter=min_iter)
    assert st[0]["n_iter"] == so[0]["n_iter"] and st[0]["converged"] == so[0]["converged"]
    # the same iterates to rounding: a few iterations from the same start
    assert np.allclose(P.get_T(), T, rtol=1e-12, atol=0.0)
    P.close()
    m.close()
