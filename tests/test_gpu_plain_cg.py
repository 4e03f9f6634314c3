"""The plain FP64 CG where its reductions change: p.q from the operator's own
workgroups (at most 2,048 of them, and more), from a kernel of its own (meshes
whose elements carry their blocks), one workgroup of the vector kernels and
many; the polls one interval behind the queue and, in the no-allocation solve,
waiting.  b = S x for a known x through the mesh's own blocks on the host;
1e-8 relative as in the other solve tests (rtol 1e-11 times the system's
condition on these meshes).
"""

import numpy as np
import pytest
import torch

import paper_1601_07384_amd as P
from stdg_inputs import kuhn_mesh

pytestmark = pytest.mark.gpu
DEV = "cuda:0"

CASES = [
    # n, p, p_gamma, periodic, reorder, jitter
    (3, 1, 0, False, True, 0.0), (7, 2, 0, True, True, 0.0), (7, 2, 1, False, True, 0.0),
    (12, 4, 0, True, False, 0.0), (6, 3, 1, True, False, 0.0), (5, 2, 0, True, True, 0.2), (14, 1, 2, True, True, 0.0),
]


@pytest.mark.parametrize("n,p,pg,periodic,reorder,jitter", CASES)
def test_plain_cg(n, p, pg, periodic, reorder, jitter):
    print(f"plain CG n={n} p={p} pg={pg} periodic={periodic} reorder={reorder} jitter={jitter}", flush=True)
    X, T = kuhn_mesh(n, jitter=jitter, seed=3)
    m = P.Mesh(X, T, p, pg, dt=1e-2, periodic=periodic, reorder=reorder)
    B, cls, nbr, C = m.blocks()
    x = np.random.default_rng(4).standard_normal((m.E, m.G, m.N))
    z = np.zeros_like(x)
    for k in range(5):
        t = np.arange(m.E) if k == 0 else nbr[:, k - 1]
        for c in np.unique(cls):
            e = np.flatnonzero((cls == c) & (t >= 0))
            z[e] += x[t[e]] @ B[c, k].T
    b = torch.tensor(np.matmul(C, z).ravel(), dtype=torch.float64, device=DEV)
    ref = x - x[m.anchor_internal, :, :1][None]
    opts = dict(method=P.STDG_CG_TIME, precision=P.STDG_FP64, rtol=1e-11, max_iter=20000)
    its, out = [], []
    for solve, every in ((m.solve, 8), (m.solve, 8), (m.solve_noalloc, 8), (m.solve, 1)):
        xs = torch.zeros_like(b)
        rep = solve(b, xs, check_every=every, **opts)
        assert rep.status == 0 and rep.rel_residual <= 1e-11
        its.append(rep.inner_iters)
        out.append(xs.cpu().numpy().reshape(x.shape))
        assert np.abs(out[-1] - ref).max() <= 1e-8 * np.abs(ref).max()
    assert its[0] == its[1] == its[2] and np.array_equal(out[0], out[1]) and np.array_equal(out[0], out[2])
    # (a restart from the true residual may add an interval)
    assert its[3] <= its[0] <= its[3] + 16
    for solve in (m.solve, m.solve_noalloc):
        xs = torch.zeros_like(b)
        rep = solve(b, xs, method=P.STDG_CG_TIME, precision=P.STDG_FP64, rtol=1e-11, max_iter=13, check_every=8)
        assert rep.status == P.STDG_NOT_CONVERGED and rep.inner_iters == 13
    xs = torch.zeros_like(b)
    b[5] = float("nan")
    with pytest.raises(Exception):
        m.solve(b, xs, **opts)
