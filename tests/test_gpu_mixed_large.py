"""The precision form without a walk where its two launches per inner iteration end.

In the row layout up to 3 * 2^19 rows, in the band layout up to 15 * 2^19, an inner
iteration is two launches, whose workgroups each sum all partials; above, five with
separate reductions (the direction is then a launch of its own, which the timers
show).  Both sides of the edge: one step against the oracle's (1e-8), and the row
layout's meshes as members of one group, bitwise the steps taken alone.
"""
import numpy as np
import pytest

import synth
from tests.gpu_common import lapfoam, max_rel

pytestmark = pytest.mark.gpu

ROWS = [((128, 128, 96), True), ((129, 128, 96), False)]
BANDS = [((199, 197, 200), True), ((201, 198, 198), False)]


def _problem(L, shape, seed, **opts):
    mesh = synth.box_mesh(*shape, z_ratio=2.0)
    if seed:
        mesh = synth.renumber(mesh, synth.random_permutation(mesh.n_cells, seed))
    m = L.Mesh(mesh)
    P = L.Problem(m, synth.fixed_x_bcs(), 1e-3, 1e-3, L.make_opts(precision=L.LF_PREC_MIXED, **opts))
    return mesh, m, P


def _has_direction_launches(L, P):
    L.lf_profile_enable(P.h, True)
    P.step(1)
    _, count = L.lf_profile_read(P.h, len(L.KERNEL_CLASSES))
    L.lf_profile_enable(P.h, False)
    return count[L.KERNEL_CLASSES.index("inner_direction")] > 0


def test_row_layout_alone_and_in_a_group(oracle):
    import torch
    L = lapfoam()
    meshes, probs, T0s, refs = [], [], [], []
    for i, (shape, two) in enumerate(ROWS):
        mesh, m, P = _problem(L, shape, 21 + i)
        T0 = synth.initial_field(mesh.n_cells, 50 + i)
        P.set_T(T0)
        assert _has_direction_launches(L, P) != two, shape
        P.set_T(T0)
        P.step(1)
        T = P.get_T()
        ref, _, _ = oracle.run(mesh, synth.fixed_x_bcs(), 1e-3, 1e-3, 1, T0)
        assert max_rel(T, ref) <= 1e-8, (shape, max_rel(T, ref))
        P.step(1)
        meshes.append(m)
        probs.append(P)
        T0s.append(torch.from_numpy(T0).cuda())
        refs.append((T, P.get_T()))
    g = L.Group(len(probs))
    snaps = [torch.empty((2, t.numel()), dtype=torch.float64, device="cuda") for t in T0s]
    for P, t, s in zip(probs, T0s, snaps):
        g.add(P, 2, s, T0=t)
    left = len(probs)
    while left:
        left -= len(g.poll())
    torch.cuda.synchronize()
    for s, ref in zip(snaps, refs):
        for j in range(2):
            assert np.array_equal(s[j].cpu().numpy(), ref[j]), j
    g.close()
    for x in probs + meshes:
        x.close()


@pytest.mark.parametrize("shape,two", BANDS)
def test_band_layout(oracle, shape, two):
    L = lapfoam()
    mesh, m, P = _problem(L, shape, 0, amul_walk=L.LF_WALK_OFF)
    T0 = synth.initial_field(mesh.n_cells, 60)
    P.set_T(T0)
    assert _has_direction_launches(L, P) != two
    P.set_T(T0)
    P.step(1)
    ref, _, _ = oracle.run(mesh, synth.fixed_x_bcs(), 1e-3, 1e-3, 1, T0)
    assert max_rel(P.get_T(), ref) <= 1e-8, max_rel(P.get_T(), ref)
    P.close()
    m.close()
