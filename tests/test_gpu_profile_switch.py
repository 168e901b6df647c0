"""The kernel timers switched while an lf_step_begin run is in flight: every solve is committed exactly once.

With max_iter = 1 the block in flight when the switch is thrown is the one that
ends the solve.  T and the residuals are bitwise those of lf_step, over two steps
(the second one's normalisation takes the first commit's sums of T).
"""
import numpy as np
import pytest

import synth
from tests.gpu_common import lapfoam

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("on", [True, False], ids=["switched_on", "switched_off"])
@pytest.mark.parametrize("form", ["two_launches", "walk"])
def test_commit_once(form, on):
    L = lapfoam()
    mesh = synth.box_mesh(20, 18, 16)
    T0 = synth.initial_field(mesh.n_cells, 5)
    m = L.Mesh(mesh)
    P = L.Problem(m, synth.fixed_x_bcs(), 1e-3, 1e-3,
                  L.make_opts(max_iter=1, amul_walk=L.LF_WALK_ON if form == "walk" else L.LF_WALK_AUTO))
    P.set_T(T0)
    ref, _ = P.step(2)
    T = P.get_T()
    P.set_T(T0)
    L.lf_profile_enable(P.h, not on)
    P.step_begin(2)
    L.lf_profile_enable(P.h, on)
    finished = False
    while not finished:
        _, finished, stats, status = P.step_poll()
    L.lf_profile_enable(P.h, False)
    assert status == L.LF_OK
    assert np.array_equal(P.get_T(), T)
    for a, b in zip(stats, ref):
        assert all(a[k] == b[k] for k in ("n_iter", "initial_residual", "final_residual"))
    P.close()
    m.close()
