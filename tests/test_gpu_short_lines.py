"""FP64 boxes with x-lines of less than 32 cells keep one row per thread up to 4.2 M cells.

At the rule's edge the line's length decides: both forms against the oracle's steps
(1e-8, iterations within one).
"""
import pytest

import synth
from tests.gpu_common import lapfoam, max_rel

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape,form", [((30, 300, 300), 0), ((32, 300, 300), 4), ((8, 580, 580), 0)])
def test_form_and_steps(oracle, shape, form):
    L = lapfoam()
    mesh = synth.box_mesh(*shape, z_ratio=2.0)
    T0 = synth.initial_field(mesh.n_cells, 31)
    m = L.Mesh(mesh)
    P = L.Problem(m, synth.fixed_x_bcs(), 1e-3, 1e-3)
    assert P.amul_form() == form
    P.set_T(T0)
    stats, _ = P.step(1)
    T, so, _ = oracle.run(mesh, synth.fixed_x_bcs(), 1e-3, 1e-3, 1, T0)
    assert max_rel(P.get_T(), T) <= 1e-8, max_rel(P.get_T(), T)
    assert stats[0]["converged"] == 1 and abs(stats[0]["n_iter"] - so[0]["n_iter"]) <= 1
    P.close()
    m.close()
