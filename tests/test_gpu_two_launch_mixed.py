"""The precision form with two launches per inner iteration, at the edges of its rules.

Without a walk the inner kernels take one row per thread up to 2^18 rows, two up
to 2^21 and eight above, where one-workgroup kernels decide the start of a pass;
the mean of x0 is taken in the assembly up to 2^20 rows.  One step per size
against the oracle's from the same T (1e-8), and the same problems as members of
one group, bitwise the steps taken alone.
"""
import numpy as np
import pytest

import synth
from tests.gpu_common import lapfoam, max_rel

pytestmark = pytest.mark.gpu

SIZES = {"below_one_row": ((64, 64, 64), None), "two_rows": ((65, 64, 64), None), "two_rows_random": ((66, 65, 64), 3),
         "above_mean": ((103, 102, 101), None), "many_rows": ((129, 128, 128), None),
         "many_rows_random": ((130, 128, 127), 4), "line": ((700, 1, 1), None)}


def _mesh(name):
    shape, seed = SIZES[name]
    mesh = synth.box_mesh(*shape, z_ratio=1.0 if min(shape) == 1 else 2.0)
    return synth.renumber(mesh, synth.random_permutation(mesh.n_cells, seed)) if seed else mesh


def test_steps_and_group(oracle):
    import torch
    L = lapfoam()
    opts = L.make_opts(precision=L.LF_PREC_MIXED)
    meshes, probs, T0s, alone = [], [], [], []
    for i, name in enumerate(SIZES):
        mesh = _mesh(name)
        T0 = synth.initial_field(mesh.n_cells, 40 + i)
        m = L.Mesh(mesh)
        P = L.Problem(m, synth.fixed_x_bcs(), 1e-3, 1e-3, opts)
        assert P.amul_form() == 0
        P.set_T(T0)
        out = []
        for _ in range(2):
            stats, _ = P.step(1)
            out.append((P.get_T(), stats[0]))
        ref, _, _ = oracle.run(mesh, synth.fixed_x_bcs(), 1e-3, 1e-3, 1, T0)
        assert out[0][1]["converged"] == 1 and max_rel(out[0][0], ref) <= 1e-8, (name, max_rel(out[0][0], ref))
        # two steps in one call go on from the same sums of T
        P.set_T(T0)
        P.step(2)
        assert np.array_equal(P.get_T(), out[1][0]), name
        meshes.append(m)
        probs.append(P)
        T0s.append(torch.from_numpy(T0).cuda())
        alone.append(out)
    g = L.Group(len(probs))
    snaps = [torch.empty((2, t.numel()), dtype=torch.float64, device="cuda") for t in T0s]
    for P, t, s in zip(probs, T0s, snaps):
        g.add(P, 2, s, T0=t)
    left = len(probs)
    while left:
        for P, stats in g.poll():
            left -= 1
            k = probs.index(P)
            for a, (_, b) in zip(stats, alone[k]):
                assert all(a[key] == b[key] for key in ("initial_residual", "final_residual", "n_iter", "n_outer"))
    torch.cuda.synchronize()
    for name, s, out in zip(SIZES, snaps, alone):
        for j in range(2):
            assert np.array_equal(s[j].cpu().numpy(), out[j][0]), (name, j)
    g.close()
    for x in probs + meshes:
        x.close()
