"""The band gradient on meshes whose widest band has a short offset, where its rows are stored one by one.

Up to 3 * 2^20 cells an offset of 512 and more takes the stores by lines, above one
of 4 and more: both sides of both edges, bitwise the oracle's face loop.
"""
import numpy as np
import pytest

import synth
from tests.gpu_common import lapfoam
from tests.test_gpu_grad import _gpu_grad, _inputs

pytestmark = pytest.mark.gpu

BOXES = [(700001, 1, 1), (511, 1300, 1), (512, 1300, 1), (3, 1048577, 1), (4, 786433, 1)]


@pytest.mark.parametrize("box", BOXES, ids=["x".join(map(str, b)) for b in BOXES])
def test_short_runs_bitwise(oracle, box):
    L = lapfoam()
    mesh = synth.affine(synth.box_mesh(*box), synth.SKEW)
    T, Tb, snb = _inputs(mesh, 72)
    m = L.Mesh(mesh, gradient=True, non_orthogonal=True)
    g, bg = _gpu_grad(L, m, T, Tb, snb)
    m.close()
    og, obg = oracle.gauss_grad(mesh, T, Tb, snb)
    assert np.array_equal(g, og) and np.array_equal(bg, obg)
