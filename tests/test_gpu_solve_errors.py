"""A solve whose residual overflows on the way: the polls read behind the queue
then find it while iterations are still queued.  The error must not come back
before they have ended (they write x and the mesh's work vectors), and the mesh
must solve the next system as if nothing had been.
"""

import pytest
import torch

import paper_1601_07384_amd as P
from stdg_inputs import kuhn_mesh
from test_gpu_two_level import DEV

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision", [P.STDG_FP64, P.STDG_FP32])
def test_error_behind_the_queue(precision):
    print("solve error, precision", precision, flush=True)
    X, T = kuhn_mesh(12)
    m = P.Mesh(X, T, 2, 0, dt=1e-2, periodic=True)
    cent = torch.tensor(X[T[m.permutation()]].mean(axis=1), device=DEV)
    b = torch.sin(6.283185307179586 * (cent[:, 0] + 2 * cent[:, 1]))[:, None].repeat(1, m.N).reshape(-1)
    b -= b.mean()
    b /= b.norm()
    opts = dict(method=P.STDG_CG, precision=precision, rtol=1e-10, inner_rtol=1e-5, max_iter=20000)
    before, after = torch.zeros_like(b), torch.zeros_like(b)
    m.solve(b, before, **opts)
    torch.cuda.synchronize()
    # |b|^2 is representable, the residual of the first iterations (its square
    # grows sixfold) is not; refinement scales each inner system to norm one
    x = torch.zeros_like(b)
    if precision == P.STDG_FP64:
        with pytest.raises(P.StdgError, match="non-finite"):
            m.solve(9e153 * b, x, check_every=64, **opts)
    else:
        assert m.solve(9e153 * b, x, check_every=64, **opts).status == 0
    assert torch.cuda.current_stream().query()
    m.solve(b, after, **opts)
    assert torch.equal(before, after)


@pytest.mark.parametrize("bad", [float("nan"), float("inf")])
def test_non_finite_right_hand_side(bad):
    """An error at once, and nothing left behind for the two-level CG's next solve."""
    print("solve, right-hand side with", bad, flush=True)
    X, T = kuhn_mesh(12)
    m = P.Mesh(X, T, 2, 1, dt=1e-2, periodic=True)
    x = torch.randn(m.E * m.Nst, generator=torch.Generator(device=DEV).manual_seed(1), dtype=torch.float64, device=DEV)
    b = torch.empty_like(x)
    m.apply(x, b)
    opts = dict(method=P.STDG_CG_TIME, precision=P.STDG_FP32, rtol=1e-10, inner_rtol=1e-5)
    before, after = torch.zeros_like(b), torch.zeros_like(b)
    m.solve(b, before, **opts)
    wrong = b.clone()
    wrong[b.numel() // 2] = bad
    with pytest.raises(P.StdgError, match="non-finite"):
        m.solve(wrong, torch.zeros_like(b), **opts)
    assert torch.cuda.current_stream().query()
    m.solve(b, after, **opts)
    assert torch.equal(before, after)
