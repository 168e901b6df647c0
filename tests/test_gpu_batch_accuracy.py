"""The batched form's distance to the exactly solved steps is no larger than lf_step's precision form's.

Both stop at the same residual and solve the corrections in FP32; the batched form
scales r and the correction with 1/sqrt(diagB) in FP64 where the other takes
sqrt(diagB) rounded to FP32, so rounding adds less to its error.  Five steps of cubes of
16^3 to 24^3, root mean square of the relative differences to FP64 steps solved far
below the tolerance, for three random fields each.
"""
import numpy as np
import pytest

import synth
from tests.gpu_common import lapfoam

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("seed", [0, 1, 2])
def test_no_further_than_the_step(seed):
    import torch
    L = lapfoam()
    sides = (16, 18, 20, 22, 24)
    step = batch = 0.0
    for i, n in enumerate(sides):
        mesh = synth.box_mesh(n, n, n)
        T0 = synth.initial_field(mesh.n_cells, 100 * seed + i)
        DT = 1e-4 * 100.0 ** ((i + 0.5) / len(sides))
        m = L.Mesh(mesh)
        X = L.Problem(m, synth.fixed_x_bcs(), DT, 1e-3, L.make_opts(tol=1e-15, max_iter=200))
        X.set_T(T0)
        X.step(5)
        exact = X.get_T()
        P = L.Problem(m, synth.fixed_x_bcs(), DT, 1e-3, L.make_opts(precision=L.LF_PREC_MIXED))
        P.set_T(T0)
        P.step(5)
        step += np.mean(((P.get_T() - exact) / exact) ** 2)
        P.set_T(T0)
        torch.cuda.synchronize()
        b = L.Batch(1, 5)
        b.launch([P], 5)
        b.wait()
        batch += np.mean(((P.get_T() - exact) / exact) ** 2)
        b.close()
        for x in (X, P, m):
            x.close()
    assert batch <= step, np.sqrt([batch, step])
