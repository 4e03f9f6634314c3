"""FP64 pressure operator on both sides of its split between 64-element runs of
one class and elements taken one by one: few elements (all of them one by
one), a last run that is not full, runs of several classes among uniform ones,
the input order (every run mixed), walls; every p with odd and even numbers of
time nodes, against the product with the mesh's own blocks on the host.

A row is a sum of 5 N G products of values of order one with the blocks: 1e-12
of the largest result leaves 20 times the rounding of 1,000 terms added one by
one.
"""

import numpy as np
import pytest
import torch

import paper_1601_07384_amd as P
from test_gpu_two_level import box_mesh

pytestmark = pytest.mark.gpu
DEV = "cuda:0"

CASES = [
    # hexahedra, p, p_gamma, periodic, reorder
    ((3, 3, 3), 1, 0, True, True), ((21, 21, 21), 1, 0, True, True), ((21, 20, 23), 1, 1, False, True),
    ((21, 20, 21), 1, 4, True, True), ((6, 6, 6), 1, 2, True, False),
    ((3, 4, 5), 2, 1, True, True), ((11, 12, 11), 2, 0, True, True), ((12, 12, 13), 2, 1, False, True),
    ((12, 11, 12), 2, 3, True, True), ((12, 12, 12), 2, 4, True, True), ((12, 12, 12), 2, 1, True, False),
    ((3, 3, 5), 3, 1, False, True), ((7, 7, 8), 3, 0, True, True), ((9, 9, 10), 3, 0, False, True),
    ((7, 7, 8), 3, 1, True, True), ((9, 10, 9), 3, 2, False, True), ((7, 7, 8), 3, 4, True, True),
    ((6, 7, 7), 3, 0, True, False),
    ((3, 3, 3), 4, 1, True, True), ((5, 5, 6), 4, 0, True, True), ((9, 9, 10), 4, 1, False, True),
    ((5, 5, 6), 4, 2, True, True), ((8, 8, 8), 4, 4, True, True), ((5, 5, 6), 4, 3, True, False),
]


@pytest.mark.parametrize("n,p,pg,periodic,reorder", CASES)
def test_apply_matches_blocks(n, p, pg, periodic, reorder):
    print(f"apply n={n} p={p} pg={pg} periodic={periodic} reorder={reorder}", flush=True)
    X, T = box_mesh(n, (1.0, 1.0, 1.0))
    m = P.Mesh(X, T, p, pg, dt=1e-2, periodic=periodic, reorder=reorder)
    B, cls, nbr, C = m.blocks()
    x = np.random.default_rng(7).standard_normal((m.E, m.G, m.N))
    z = np.zeros_like(x)
    for k in range(5):
        t = np.arange(m.E) if k == 0 else nbr[:, k - 1]
        for c in range(m.n_classes):
            e = np.flatnonzero((cls == c) & (t >= 0))
            z[e] += x[t[e]] @ B[c, k].T
    ref = np.matmul(C, z)
    xd = torch.tensor(x.ravel(), dtype=torch.float64, device=DEV)
    y = torch.full_like(xd, float("nan"))
    m.apply(xd, y)
    err = np.abs(y.cpu().numpy().reshape(ref.shape) - ref).max()
    assert err <= 1e-12 * np.abs(ref).max()


@pytest.mark.parametrize("n,p,pg,periodic", [((3, 3, 3), 3, 0, False), ((6, 7, 6), 3, 2, True), ((4, 5, 6), 4, 0, False),
                                             ((6, 6, 5), 4, 1, True), ((3, 4, 4), 4, 4, False)])
def test_apply_f32_matches_fp64(n, p, pg, periodic):
    """The FP32 operator element by element (p >= 3, few elements): 5 N products
    in FP32, 1e-5 of the largest result."""
    print(f"apply_f32 n={n} p={p} pg={pg} periodic={periodic}", flush=True)
    X, T = box_mesh(n, (1.0, 1.0, 1.0))
    m = P.Mesh(X, T, p, pg, dt=1e-2, periodic=periodic)
    xf = torch.tensor(np.random.default_rng(3).standard_normal(m.E * m.Nst), dtype=torch.float32, device=DEV)
    yf = torch.full_like(xf, float("nan"))
    m.apply_f32(xf, yf)
    y = torch.empty(m.E * m.Nst, dtype=torch.float64, device=DEV)
    m.apply(xf.double(), y)
    assert float((yf.double() - y).abs().max()) <= 1e-5 * float(y.abs().max())
