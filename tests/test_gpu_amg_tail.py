"""The multigrid cycle's last levels in one workgroup against the oracle.

From the first level on whose rows, with those of the levels below it, fit into
the LDS (2852 rows), the cycle is one launch; the levels above keep their
launches.  Either way the cycle sums in the order of the sequential definition,
so one application is compared bit for bit: at boxes whose second level is the
first that fits and the first that does not, with odd sides, with one level
only, and at thin boxes whose coarsest level is large.
"""
import numpy as np
import pytest

import synth
from tests.gpu_common import lapfoam
from tests.test_gpu_amg import DT, dt, _run_hook

pytestmark = pytest.mark.gpu

BOXES = [(26, 26, 26), (25, 26, 27), (28, 28, 28), (27, 25, 40), (10, 9, 200), (11, 10, 226), (9, 8, 8), (5, 4, 300),
         (3, 2, 400), (64, 52, 7)]


@pytest.fixture(scope="module")
def L():
    return lapfoam()


@pytest.mark.parametrize("walk", [0, 2], ids=["auto", "nowalk"])
@pytest.mark.parametrize("box", BOXES, ids=["x".join(map(str, b)) for b in BOXES])
def test_amg_cycle_tail_bitwise(L, oracle, box, walk):
    mesh = synth.box_mesh(*box, z_ratio=3.0)
    T0 = synth.initial_field(mesh.n_cells, 31)
    r, w = _run_hook(L, mesh, T0, L.LF_PC_AMG, amul_walk=walk)
    A = oracle.assemble(mesh, synth.fixed_x_bcs(), DT, dt, T0)
    lc, ag = synth.box_aggregation(box)
    want = oracle.amg_apply(mesh, A["diag_b"], A["upper"], r, lc, ag)
    assert np.array_equal(w, want), (box, len(lc), float(np.max(np.abs(w - want))))
