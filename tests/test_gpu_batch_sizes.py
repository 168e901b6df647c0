"""The batched kernel at the sizes where its vectors change place.

A problem of n rows in the band layout keeps min(4, floor(39 * 1024 / n)) of its
FP32 vectors in the LDS (none above 39,936 rows), and takes its rows in groups
that are inner ones only away from both ends.  One step from a random field on
boxes at both sides of every change, on thin boxes without an inner group and
on a few cells, against the oracle's step within the precision form's bar of
1e-8, with every workgroup size.
"""
import pytest

import synth
from tests.gpu_common import lapfoam, max_rel

pytestmark = pytest.mark.gpu

SHAPES = [(2, 2, 2), (130, 4, 4), (3, 3, 300), (21, 22, 21), (22, 22, 22), (24, 24, 23), (24, 24, 24),
          (27, 27, 27), (28, 27, 27), (34, 34, 34), (35, 34, 34)]


@pytest.mark.parametrize("threads", [256, 512, 1024])
def test_step_at_every_placement(oracle, threads):
    import torch
    L = lapfoam()
    meshes, probs, refs = [], [], []
    for i, shape in enumerate(SHAPES):
        mesh = synth.box_mesh(*shape, z_ratio=2.0)
        T0 = synth.initial_field(mesh.n_cells, 300 + i)
        m = L.Mesh(mesh)
        P = L.Problem(m, synth.fixed_x_bcs(), 1e-3, 1e-3, L.make_opts(precision=L.LF_PREC_MIXED))
        P.set_T(T0)
        meshes.append(m)
        probs.append(P)
        refs.append(oracle.run(mesh, synth.fixed_x_bcs(), 1e-3, 1e-3, 1, T0)[0])
    torch.cuda.synchronize()
    b = L.Batch(len(probs), 1)
    b.launch(probs, 1, block_threads=threads, n_workgroups=4)
    b.wait()
    stats, _ = b.stats()
    for shape, P, ref, st in zip(SHAPES, probs, refs, stats):
        assert st[0]["converged"] == 1, shape
        assert max_rel(P.get_T(), ref) <= 1e-8, (shape, max_rel(P.get_T(), ref))
    b.close()
    for x in probs + meshes:
        x.close()
