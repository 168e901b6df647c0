"""A problem's batched result does not depend on the launch's form.

A launch whose problems all have at most 4096 rows takes the form for small
problems, one larger problem in it the other: the same problems (a few cells, both
sides of a workgroup, exactly 4096 rows, the row layout) bitwise the same in both,
and within the precision form's bar of 1e-8 of the oracle's step.
"""
import numpy as np
import pytest

import synth
from tests.gpu_common import lapfoam, max_rel

pytestmark = pytest.mark.gpu

SHAPES = [(2, 2, 2), (4, 4, 4), (8, 8, 8), (9, 8, 8), (12, 12, 12), (16, 16, 16), (3, 3, 300)]


@pytest.mark.parametrize("threads", [256, 512, 1024])
def test_small_alone_and_beside_a_large_one(oracle, threads):
    import torch
    L = lapfoam()
    opts = L.make_opts(precision=L.LF_PREC_MIXED)
    host = [synth.box_mesh(*s, z_ratio=2.0) for s in SHAPES]
    host.append(synth.renumber(host[4], synth.random_permutation(host[4].n_cells, 3)))
    host.append(synth.box_mesh(17, 16, 16))          # 4352 rows: the large form
    T0 = [synth.initial_field(m.n_cells, 400 + i) for i, m in enumerate(host)]
    meshes = [L.Mesh(m) for m in host]
    probs = [L.Problem(m, synth.fixed_x_bcs(), 1e-3, 1e-3, opts) for m in meshes]
    b = L.Batch(len(probs), 2)
    out = []
    for n in (len(probs) - 1, len(probs)):
        for P, t in zip(probs, T0):
            P.set_T(t)
        torch.cuda.synchronize()
        b.launch(probs[:n], 2, block_threads=threads)
        b.wait()
        stats, _ = b.stats()
        out.append(([P.get_T() for P in probs], stats))
    for i in range(len(probs) - 1):
        assert np.array_equal(out[0][0][i], out[1][0][i]), i
        for x, y in zip(out[0][1][i], out[1][1][i]):
            assert all(x[k] == y[k] for k in ("initial_residual", "final_residual", "n_iter", "n_outer")), i
    for m, t, T in zip(host, T0, out[1][0]):
        ref = oracle.run(m, synth.fixed_x_bcs(), 1e-3, 1e-3, 2, t)[0]
        assert max_rel(T, ref) <= 1e-8, max_rel(T, ref)
    b.close()
    for x in probs + meshes:
        x.close()
