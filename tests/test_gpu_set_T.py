"""lf_set_T of a device field: the copy moves 16 bytes per thread where both ends allow it, else 8.

Fields aligned to 16 bytes and to 8 only, an even and an odd number of cells, one
cell: what is read back is what was set, and its neighbours in memory are not.
"""
import numpy as np
import pytest

import synth
from tests.gpu_common import lapfoam

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape", [(1, 1, 1), (2, 1, 1), (9, 9, 9), (16, 9, 9)])
@pytest.mark.parametrize("offset", [0, 1])
def test_round_trip(shape, offset):
    import torch
    L = lapfoam()
    m = L.Mesh(synth.box_mesh(*shape))
    P = L.Problem(m, synth.fixed_x_bcs(), 1e-3, 1e-3)
    T = torch.arange(m.n_cells + 2 * offset, dtype=torch.float64, device="cuda") + 273.0
    field = T[offset:offset + m.n_cells]
    assert field.data_ptr() % 16 == 8 * offset
    P.set_T(field)
    assert np.array_equal(P.get_T(), field.cpu().numpy())
    P.close()
    m.close()
