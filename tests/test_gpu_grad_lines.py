"""The band gradient's rows stored by whole lines through the LDS, at the edges of its rule.

Above 655360 cells a wavefront that holds 64 consecutive cells writes their rows
together; one whose cells wrap to the next layer, or that the mesh ends, writes
each by itself.  Boxes at the rule's last size and just above it, with layers that
are and are not multiples of a wavefront, an odd number of layers (the last walk
holds one cell), and two bands only: bitwise the oracle's face loop.
"""
import numpy as np
import pytest

import synth
from tests.gpu_common import lapfoam
from tests.test_gpu_grad import _gpu_grad, _inputs

pytestmark = pytest.mark.gpu

BOXES = [(128, 80, 64), (128, 80, 65), (89, 87, 86), (97, 83, 83), (1021, 651, 1), (64, 2, 5200)]


@pytest.mark.parametrize("box", BOXES, ids=["x".join(map(str, b)) for b in BOXES])
def test_rows_by_lines_bitwise(oracle, box):
    L = lapfoam()
    mesh = synth.affine(synth.box_mesh(*box, z_ratio=2.0 if box[2] > 1 else 1.0), synth.SKEW)
    T, Tb, snb = _inputs(mesh, 71)
    m = L.Mesh(mesh, gradient=True, non_orthogonal=True)
    g, bg = _gpu_grad(L, m, T, Tb, snb)
    m.close()
    og, obg = oracle.gauss_grad(mesh, T, Tb, snb)
    assert np.array_equal(g, og) and np.array_equal(bg, obg)
