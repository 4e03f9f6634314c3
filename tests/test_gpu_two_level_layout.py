"""The two-level CG on a mesh of the run layout that is too large for the
one-kernel CG's partials (E G above 5.1 M), where the refinement once handed it
element-major vectors.  b = S x by the FP64 operator, so x (anchored) is the
solution; 1e-8 relative as in the other two-level tests.
"""

import numpy as np
import pytest
import torch

import paper_1601_07384_amd as P
from test_gpu_two_level import DEV, box_mesh

pytestmark = pytest.mark.gpu


def test_past_the_one_kernel_limit():
    X, T = box_mesh((56, 56, 56), (1.0, 1.0, 1.0))
    print("two-level, 1,053,696 elements, p=1, p_gamma=4", flush=True)
    m = P.Mesh(X, T, 1, 4, dt=1e-2, periodic=True)
    assert m.inner_layout == 1 and 2 * 8 * (m.E // 384 * m.G) > 1024 * 208
    cent = torch.tensor(X[T[m.permutation()]].mean(axis=1), device=DEV)
    g = torch.Generator(device=DEV).manual_seed(4)
    x = 0.01 * torch.randn(m.E, m.G, m.N, generator=g, dtype=torch.float64, device=DEV)
    x += torch.sin(2 * np.pi * (cent[:, 0] + 2 * cent[:, 1]) + 0.3)[:, None, None]
    b = torch.empty(m.E * m.Nst, dtype=torch.float64, device=DEV)
    m.apply(x.reshape(-1), b)
    xs = torch.zeros_like(b)
    rep = m.solve(b, xs, method=P.STDG_CG_TIME, precision=P.STDG_FP32, rtol=1e-11, inner_rtol=1e-5, max_iter=3000)
    assert rep.status == 0 and rep.rel_residual <= 1e-11
    ref = x - x[m.anchor_internal, :, :1][None]
    assert float((xs.view_as(x) - ref).abs().max()) <= 1e-8 * float(ref.abs().max())
