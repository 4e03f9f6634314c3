"""Vertex coordinates with noise near the tolerance that joins them to a grid
line of the second level: every vertex must find its line (an index past the
last line would leave the tables) and two builds of one mesh must agree.  A
long thin box, whose volume hides the noise of its end face from the test that
the mesh fills it; the residual is checked against the mesh's host blocks.
"""

import numpy as np
import pytest
import torch

import paper_1601_07384_amd as P
from common import blocks_apply
from test_gpu_two_level import DEV, box_mesh

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("seed", [0, 1])
def test_noise_at_the_tolerance(seed):
    n, size = (70, 2, 2), (2500.0, 1.0, 1.0)
    print("two-level, noisy end face, seed", seed, flush=True)
    X, T = box_mesh(n, size)
    h = (np.prod(size) / np.prod(n)) ** (1 / 3)
    rng = np.random.default_rng(seed)
    end, inner = X[:, 0] == size[0], (X[:, 0] > 0) & (X[:, 0] < size[0])
    X[end, 0] += rng.uniform(-1.6e-6, 0.0, end.sum()) * h
    X[inner, 0] += rng.uniform(-4e-7, 4e-7, inner.sum()) * h
    out = []
    for _ in range(2):
        m = P.Mesh(X, T, 1, 0, dt=1e-2)
        x = np.random.default_rng(5).standard_normal((m.E, m.N))
        b = blocks_apply(m, x)
        bd = torch.tensor(b.ravel(), dtype=torch.float64, device=DEV)
        xs = torch.zeros_like(bd)
        rep = m.solve(bd, xs, method=P.STDG_CG, precision=P.STDG_FP32, rtol=1e-9, inner_rtol=1e-4, max_iter=50000)
        assert rep.status == 0
        r = b - blocks_apply(m, xs.cpu().numpy().reshape(m.E, m.N))
        keep = np.ones((m.E, m.N), bool)          # the anchor's row is not solved for
        keep[m.anchor_internal, 0] = False
        assert np.linalg.norm(r[keep]) <= 1.1e-9 * np.linalg.norm(b[keep])
        out.append(xs.cpu().numpy())
    assert np.array_equal(out[0], out[1])
