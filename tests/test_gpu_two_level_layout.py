"""The two-level CG on meshes of the run layout: one too large for the one-kernel
CG's partials (E G above 5.1 M), where the refinement once handed it
element-major vectors, and ones with more lines than the grid may have, whose
corners are interpolated.  b = S x by the FP64 operator, so x (anchored) is the
solution; 1e-8 relative as in the other two-level tests (p = 4: the residual).
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


@pytest.mark.parametrize("p,pg", [(1, 0), (2, 1), (3, 0), (4, 0), (4, 1)])
def test_interpolated_corners_in_the_run_layout(p, pg):
    n, size = (96, 4, 4), (24.0, 1.0, 1.0)
    print(f"two-level, run layout, interpolated corners, p={p} p_gamma={pg}", flush=True)
    X, T = box_mesh(n, size)
    m = P.Mesh(X, T, p, pg, dt=1e-2, periodic=True, box_hi=size)
    assert m.inner_layout == 1
    cent = torch.tensor(X[T[m.permutation()]].mean(axis=1) / X.max(axis=0), device=DEV)
    g = torch.Generator(device=DEV).manual_seed(4)
    x = 0.01 * torch.randn(m.E, m.G, m.N, generator=g, dtype=torch.float64, device=DEV)
    x += torch.sin(2 * np.pi * (cent[:, 0] + 2 * cent[:, 1]) + 0.3)[:, None, None]
    b = torch.empty(m.E * m.Nst, dtype=torch.float64, device=DEV)
    m.apply(x.reshape(-1), b)
    xs = torch.zeros_like(b)
    rep = m.solve(b, xs, method=P.STDG_CG_TIME, precision=P.STDG_FP32, rtol=1e-11, inner_rtol=1e-5, max_iter=3000,
                  check_every=64)
    print("  iterations:", rep.inner_iters, flush=True)
    assert rep.status == 0 and rep.rel_residual <= 1e-11
    assert rep.inner_iters % 64 != 0          # the two-level CG's count; polls elsewhere are 64 apart
    if p < 4:
        ref = x - x[m.anchor_internal, :, :1][None]
        assert float((xs.view_as(x) - ref).abs().max()) <= 1e-8 * float(ref.abs().max())
