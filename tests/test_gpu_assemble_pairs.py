"""The assembly fused with a solve's start, two adjacent rows per thread (walked boxes).

The same step with the walk (rows in pairs) and without it (one row per thread):
the start's residual is a sum of the same terms in another order, so with at most
1e5 rows it agrees within 1e5 rounding errors (1e-11); T within the bar of the
other parity cases, also against the oracle.  Boxes: one pair, x-lines shorter and
longer than a wavefront's rows, a mesh that ends inside a wavefront, single lines
per plane, in the precision form (x-lines of a multiple of four).  The scaled solve
takes the pairs from 1 M rows on; its own tests compare it with one row per thread
and the oracle.
"""
import numpy as np
import pytest

import synth
from tests.gpu_common import lapfoam, max_rel

pytestmark = pytest.mark.gpu

BOXES = [(4, 2, 2), (8, 5, 7), (132, 4, 3), (1028, 3, 2), (64, 33, 31)]


@pytest.mark.parametrize("box", BOXES, ids=["x".join(map(str, b)) for b in BOXES])
def test_pairs_match_rows_and_oracle(oracle, box):
    L = lapfoam()
    mesh = synth.box_mesh(*box, z_ratio=2.0)
    T0 = synth.initial_field(mesh.n_cells, 51)
    got = {}
    for walk in (L.LF_WALK_ON, L.LF_WALK_OFF):
        m = L.Mesh(mesh)
        P = L.Problem(m, synth.fixed_x_bcs(), 1e-3, 1e-3, L.make_opts(precision=L.LF_PREC_MIXED, amul_walk=walk))
        P.set_T(T0)
        out = []
        for _ in range(2):
            stats, _ = P.step(1)
            out.append((P.get_T(), stats[0]))
        got[walk] = (P.amul_form(), out)
        P.close()
        m.close()
    assert got[L.LF_WALK_ON][0] >= 2 and got[L.LF_WALK_OFF][0] == 0
    a, b = got[L.LF_WALK_ON][1], got[L.LF_WALK_OFF][1]
    ra, rb = a[0][1]["initial_residual"], b[0][1]["initial_residual"]
    assert abs(ra - rb) <= 1e-11 * rb, (ra, rb)
    ref, _, _ = oracle.run(mesh, synth.fixed_x_bcs(), 1e-3, 1e-3, 1, T0)
    for s in range(2):
        assert a[s][1]["converged"] == 1 and max_rel(a[s][0], b[s][0]) <= 1e-8
    assert max_rel(a[0][0], ref) <= 1e-8
