"""The second level's kernels on every padded grid size (16 T lines, T up to 5,
unequal between the planes' directions and the columns) and on the small grids
of one workgroup up to their limits (1,024 nodes, 16 lines; 384 nodes with the
gather inside), as in the other two-level tests.
"""

import numpy as np
import pytest
import torch

import paper_1601_07384_amd as P
import test_gpu_two_level as two
from stdg_inputs import kuhn_mesh

pytestmark = pytest.mark.gpu

BOXES = [(40, 4, 3), (5, 60, 4), (75, 3, 4), (3, 4, 70), (4, 3, 40), (20, 36, 3), (16, 16, 4), (16, 8, 3), (6, 8, 8)]


@pytest.mark.parametrize("n,p,pg", [(n, 1 + i % 3, i % 2) for i, n in enumerate(BOXES)])
def test_boxes(n, p, pg):
    size = tuple(k / 8 for k in n)
    two.test_two_level_solve((f"{n} p={p} pg={pg}", lambda: two.box_mesh(n, size), p, pg, True, size, True))


@pytest.mark.parametrize("n,p,pg", [(6, 2, 1), (7, 2, 0), (10, 1, 0)])
def test_cubes_with_walls(n, p, pg):
    two.test_two_level_solve((f"walls {n} p={p} pg={pg}", lambda: kuhn_mesh(n), p, pg, False, None, True))


@pytest.mark.parametrize("n,pg,periodic", [(4, 0, True), (5, 1, True), (8, 0, True), (8, 1, False), (9, 0, False)])
def test_p4(n, pg, periodic):
    """p = 4: runs of one class and of several, a last run that is not full.
    What a solve promises is its residual (the condition of these systems, up
    to 1e3 times that of the lower degrees, stands between it and the error):
    recomputed here with the mesh's blocks, whose rounding is a tenth of it."""
    print(f"two-level p=4 n={n} pg={pg} periodic={periodic}", flush=True)
    X, T = kuhn_mesh(n)
    m = P.Mesh(X, T, 4, pg, dt=1e-2, periodic=periodic)
    B, cls, nbr, C = m.blocks()

    def product(x):
        z = np.zeros_like(x)
        for k in range(5):
            t = np.arange(m.E) if k == 0 else nbr[:, k - 1]
            for c in range(m.n_classes):
                e = np.flatnonzero((cls == c) & (t >= 0))
                z[e] += x[t[e]] @ B[c, k].T
        return np.matmul(C, z)

    cent = X[T[m.permutation()]].mean(axis=1)
    x = np.random.default_rng(4).standard_normal((m.E, m.G, m.N)) * 0.01
    x += np.sin(2 * np.pi * (cent[:, 0] + 2 * cent[:, 1]) + 0.3)[:, None, None]
    b = product(x)
    bd = torch.tensor(b.ravel(), dtype=torch.float64, device=two.DEV)
    its = {}
    for pc in (P.STDG_PRECOND_BLOCK_JACOBI, P.STDG_PRECOND_NONE):
        xs = torch.zeros_like(bd)
        rep = m.solve(bd, xs, method=P.STDG_CG_TIME, precision=P.STDG_FP32, rtol=1e-11, inner_rtol=1e-5,
                      max_iter=20000, precond=pc)
        assert rep.status == 0 and rep.rel_residual <= 1e-11
        r = b - product(xs.cpu().numpy().reshape(x.shape))
        keep = np.ones(m.E * m.G * m.N, bool)          # the anchor's rows are not solved for
        keep.reshape(x.shape)[m.anchor_internal, :, 0] = False
        assert np.linalg.norm(r.ravel()[keep]) <= 1.1e-11 * np.linalg.norm(b.ravel()[keep])
        its[pc] = rep.inner_iters
    assert its[P.STDG_PRECOND_BLOCK_JACOBI] < 0.45 * its[P.STDG_PRECOND_NONE]
