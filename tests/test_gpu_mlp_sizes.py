"""The model's matrix products where their tiles and loads change: hidden units
and outputs that are no multiple of four (one value at a time instead of four),
one unit, one row, row counts around the 64-row tile and the split of the batch
between weight-gradient slices.  Against the oracle in the tolerances of the
other model tests (1e-12 / 1e-11 relative to the largest value in FP64, 1e-5 /
1e-4 in FP32).
"""

import numpy as np
import pytest
import torch

import paper_1601_07384_amd as P
from oracle import mlp
from stdg_inputs import kuhn_mesh

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def dev(a):
    return torch.tensor(np.ascontiguousarray(a, dtype=np.float64).ravel(), device=DEV)


@pytest.mark.parametrize("precision", [P.STDG_FP64, P.STDG_FP32])
@pytest.mark.parametrize("p,pg,hidden,n", [(1, 0, 1, 1), (1, 0, 67, 63), (2, 2, 66, 65), (2, 0, 33, 257),
                                           (3, 0, 128, 530), (1, 1, 192, 1040)])
def test_gradient_sizes(precision, p, pg, hidden, n):
    print(f"mlp sizes precision={precision} p={p} pg={pg} hidden={hidden} n={n}", flush=True)
    X, T = kuhn_mesh(3)
    m = P.Mesh(X, T, p, pg, dt=1e-2, periodic=True)
    model = P.Model(m, hidden=hidden, precision=precision, batch=2048)
    rng = np.random.default_rng(21)
    shapes = mlp.shapes(model.n_in, hidden, model.n_out)
    theta = mlp.flatten([rng.standard_normal(s) / np.sqrt(s[0]) for s in shapes])
    model.set_params(theta)
    F = rng.standard_normal((n, model.n_in))
    R = rng.standard_normal((n, model.n_out))
    Y = torch.empty(n * model.n_out, dtype=torch.float64, device=DEV)
    model.forward(dev(F), Y)
    Yo, _ = mlp.forward(theta, F, hidden, model.n_out)
    tol_f, tol_g = (1e-12, 1e-11) if precision == P.STDG_FP64 else (1e-5, 1e-4)
    assert np.abs(Y.cpu().numpy().reshape(Yo.shape) - Yo).max() <= tol_f * np.abs(Yo).max()
    loss = model.loss_grad(dev(F), dev(R))
    lo, go = mlp.loss_and_grad(theta, F, R, hidden, model.n_out)
    assert abs(loss - lo) <= tol_f * lo
    gg = model.grads()
    o = 0
    for s in shapes:
        k = int(np.prod(s))
        assert np.abs(gg[o:o + k] - go[o:o + k]).max() <= tol_g * np.abs(go[o:o + k]).max(), s
        o += k
