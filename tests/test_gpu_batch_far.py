"""The batched kernel past 2^28 rows, where a row's byte offset no longer fits an access's 32 bits.

A line of 2^28 + 1001 cells in the row layout: one step by the batch against the
same step by lf_step (other kernels, the same refinement to 1e-9; the precision
form's bar of 1e-8), the last rows among them.
"""
import types

import numpy as np
import pytest

from tests.gpu_common import lapfoam

pytestmark = pytest.mark.gpu


def test_line_past_2_to_28():
    import torch
    L = lapfoam()
    n = (1 << 28) + 1001
    x = np.zeros((n, 3))
    x[:, 0] = np.arange(n) + 0.5
    owner = np.arange(n - 1, dtype=np.int32)
    face_area = np.zeros((n - 1, 3))
    face_area[:, 0] = 1.0
    m = L.Mesh(types.SimpleNamespace(
        n_cells=n, n_faces=n - 1, owner=owner, neighbour=owner + 1, cell_volume=np.ones(n), cell_centre=x,
        face_area=face_area, patch_start=np.array([0, 1, 2]), bface_cell=np.array([0, n - 1]),
        bface_area=np.array([[-1.0, 0.0, 0.0], [1.0, 0.0, 0.0]]),
        bface_centre=np.array([[0.0, 0.0, 0.0], [float(n), 0.0, 0.0]])))
    del x, owner, face_area
    P = L.Problem(m, [(L.LF_BC_FIXED_VALUE, 273.0), (L.LF_BC_FIXED_VALUE, 573.0)], 0.05, 1.0,
                  L.make_opts(precision=L.LF_PREC_MIXED, layout=L.LF_LAYOUT_ROWS))
    g = torch.Generator(device="cuda")
    g.manual_seed(3)
    T0 = 273.0 + 300.0 * torch.rand(n, generator=g, device="cuda", dtype=torch.float64)
    P.set_T(T0)
    P.step(1)
    ref = P.get_T(torch.empty_like(T0))
    P.set_T(T0)
    torch.cuda.synchronize()
    b = L.Batch(1, 1)
    b.launch([P], 1, block_threads=1024)
    b.wait()
    assert b.stats()[0][0][0]["converged"] == 1
    T = P.get_T(T0)
    torch.cuda.synchronize()
    assert ((T - ref).abs() / ref).max().item() <= 1e-8
    b.close()
    P.close()
    m.close()
