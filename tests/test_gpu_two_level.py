"""The two-level preconditioned inner CG (csrc/cg_coarse.hip) where it can go
wrong: grids through the vertices (periodic and with walls, unequal edges,
line counts that are no multiple of the matrix tiles), scattered vertices
(interpolated corners, with and without periodic wrap), more lines than the
grid may have, and a mesh that does not fill its bounding box (block Jacobi).

The right-hand side is S x for a known x, formed on the host in FP64 from the
library's blocks, so x (anchored) is the solution; 1e-8 relative as in the
other solve tests (rtol 1e-11 times the system's condition on these meshes).
"""

import numpy as np
import pytest
import torch

import paper_1601_07384_amd as P
from stdg_inputs import kuhn_mesh
from stdg_inputs.mesh import KUHN_PERMS

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def box_mesh(n, size):
    """Kuhn mesh of n[0] x n[1] x n[2] hexahedra on the box [0, size]."""
    m = [k + 1 for k in n]
    kk, jj, ii = np.meshgrid(*(np.arange(k) for k in m[::-1]), indexing="ij")
    X = np.stack([size[0] * ii.ravel() / n[0], size[1] * jj.ravel() / n[1], size[2] * kk.ravel() / n[2]], axis=1)
    step = np.array([1, m[0], m[0] * m[1]])
    ck, cj, ci = np.meshgrid(*(np.arange(k) for k in n[::-1]), indexing="ij")
    corner = (ci + m[0] * (cj + m[1] * ck)).ravel()
    off = np.array([[0, step[s[0]], step[s[0]] + step[s[1]], step.sum()] for s in KUHN_PERMS])
    return X, (corner[:, None, None] + off[None]).reshape(-1, 4)


def l_shape(n):
    """A cube of n^3 hexahedra without one octant."""
    X, T = kuhn_mesh(n)
    c = X[T].mean(axis=1)
    return X, T[~np.all(c > 0.5, axis=1)]


CASES = [
    # name, mesh, p, p_gamma, periodic, box, two-level
    ("periodic", lambda: kuhn_mesh(9), 3, 1, True, (1.0, 1.0, 1.0), True),
    ("periodic lines 16", lambda: kuhn_mesh(16), 1, 0, True, (1.0, 1.0, 1.0), True),
    ("walls lines 17", lambda: kuhn_mesh(16), 1, 0, False, None, True),
    ("walls", lambda: kuhn_mesh(9), 2, 2, False, None, True),
    ("walls, smallest", lambda: kuhn_mesh(4), 3, 0, False, None, True),
    ("unequal edges", lambda: box_mesh((18, 9, 5), (2.0, 0.5, 1.0)), 2, 0, True, (2.0, 0.5, 1.0), True),
    ("scattered periodic", lambda: kuhn_mesh(9, jitter=0.2, seed=3), 2, 1, True, (1.0, 1.0, 1.0), True),
    ("scattered walls", lambda: kuhn_mesh(9, jitter=0.2, seed=3), 1, 0, False, None, True),
    ("more lines than the grid", lambda: box_mesh((100, 3, 3), (20.0, 1.0, 1.0)), 1, 1, True, (20.0, 1.0, 1.0), True),
    ("not a box", lambda: l_shape(10), 2, 0, False, None, False),
]


@pytest.mark.parametrize("case", CASES, ids=[c[0] for c in CASES])
def test_two_level_solve(case):
    name, mesh, p, pg, periodic, box, two = case
    print("two-level", name, flush=True)
    X, T = mesh()
    m = P.Mesh(X, T, p, pg, dt=1e-2, periodic=periodic, box_hi=box or (1.0, 1.0, 1.0))
    B, cls, nbr, C = m.blocks()
    perm = m.permutation()
    nodes = np.random.default_rng(4).standard_normal((m.E, m.G, m.N)) * 0.01
    cent = X[T[perm]].mean(axis=1) / X.max(axis=0)
    x = nodes + np.sin(2 * np.pi * (cent[:, 0] + 2 * cent[:, 1]) + 0.3)[:, None, None]
    y = np.matmul(x, B[cls, 0].transpose(0, 2, 1))
    for f in range(4):
        k = nbr[:, f]
        y += np.where(k[:, None, None] >= 0, np.matmul(x[np.maximum(k, 0)], B[cls, 1 + f].transpose(0, 2, 1)), 0.0)
    b = torch.tensor((np.matmul(C, y)).ravel(), dtype=torch.float64, device=DEV)
    ref = x - x[m.anchor_internal, :, :1][None]
    out, its = [], {}
    for pc in (P.STDG_PRECOND_BLOCK_JACOBI, P.STDG_PRECOND_BLOCK_JACOBI, P.STDG_PRECOND_NONE):
        xs = torch.zeros_like(b)
        rep = m.solve(b, xs, method=P.STDG_CG_TIME, precision=P.STDG_FP32, rtol=1e-11, inner_rtol=1e-5,
                      max_iter=20000, precond=pc)
        assert rep.status == 0 and rep.rel_residual <= 1e-11
        out.append(xs.cpu().numpy().reshape(x.shape))
        its[pc] = rep.inner_iters
        assert np.abs(out[-1] - ref).max() <= 1e-8 * np.abs(ref).max()
    assert np.array_equal(out[0], out[1])
    print(f"  {m.E} elements, iterations: none {its[P.STDG_PRECOND_NONE]}, preconditioned "
          f"{its[P.STDG_PRECOND_BLOCK_JACOBI]}", flush=True)
    # block Jacobi alone needs more than half of the plain iterations on these meshes
    assert (its[P.STDG_PRECOND_BLOCK_JACOBI] < 0.45 * its[P.STDG_PRECOND_NONE]) == two
    # the iteration limit is kept and reported
    xs = torch.zeros_like(b)
    rep = m.solve(b, xs, method=P.STDG_CG_TIME, precision=P.STDG_FP32, rtol=1e-11, inner_rtol=1e-5, max_iter=7)
    assert rep.status == P.STDG_NOT_CONVERGED and rep.inner_iters <= 7
    # a zero and a non-finite right-hand side
    rep = m.solve(torch.zeros_like(b), xs, method=P.STDG_CG_TIME, precision=P.STDG_FP32)
    assert rep.status == 0 and float(xs.abs().max()) == 0.0
