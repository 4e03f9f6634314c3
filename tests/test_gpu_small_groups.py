"""Groups of few elements of one class, cut where the class changes: meshes
with walls and periodic ones whose classes are no multiple of 64 elements,
every p, against the general kernels on the same mesh (in the input order no
two neighbouring elements share a class).  Tolerances as in the tests of whole
runs: the transfers' rounding, and for a step 1e3 times the residuals of its
solves.
"""

import numpy as np
import pytest
import torch

import paper_1601_07384_amd as P
import test_gpu_class_runs as runs
from stdg_inputs import fourier_modes, fourier_velocity, kuhn_mesh, node_coordinates

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,p,pg,periodic", [(3, 1, 0, False), (4, 2, 1, False), (5, 2, 0, True), (3, 3, 0, False),
                                             (5, 3, 1, True), (4, 3, 2, False), (4, 4, 0, False), (3, 4, 1, True)])
def test_transfers(n, p, pg, periodic):
    runs.test_transfers_match_general_kernels(n, p, pg, periodic)


@pytest.mark.parametrize("n,p,pg,periodic", [(4, 1, 1, False), (5, 2, 0, False), (5, 2, 1, True), (4, 2, 3, False),
                                             (4, 3, 0, False), (5, 3, 0, True), (3, 3, 1, False), (3, 4, 0, False),
                                             (4, 2, 4, True), (3, 3, 2, False), (3, 3, 3, True), (4, 4, 0, True),
                                             (3, 4, 1, False)])
def test_step(n, p, pg, periodic):
    print(f"small groups n={n} p={p} pg={pg} periodic={periodic}", flush=True)
    X, T = kuhn_mesh(n)
    v = fourier_velocity(node_coordinates(X, T, p), fourier_modes(seed=5, n_modes=6, kmax=2))
    v0 = np.transpose(v, (2, 0, 1))[:, :, None, :] * (1.0 + 0.1 * np.arange(pg + 1))[None, None, :, None]
    out = []
    for reorder in (True, False):
        m = P.Mesh(X, T, p, pg, dt=2e-3, nu=2e-2, periodic=periodic, reorder=reorder)
        vbar = runs.dev(v0[:, m.permutation()])
        vhat = torch.empty(3 * m.n_face * m.Nst, dtype=torch.float64, device=runs.DEV)
        m.dual_from_main(vbar, vhat)
        p0 = torch.zeros(m.E * m.Nst, dtype=torch.float64, device=runs.DEV)
        # the walls move with the flow's own velocity
        rep = m.picard_step(vhat, vbar, p0, None if periodic else vbar.clone(), opts=P.step_opts(
            n_picard=2,
            pressure={"method": P.STDG_CG_TIME, "precision": P.STDG_FP32, "rtol": 1e-12, "inner_rtol": 1e-5,
                      "max_iter": 50000},
            viscous={"method": P.STDG_BICGSTAB, "restart": 10, "rtol": 1e-12, "check_every": 1}))
        assert rep.max_viscous_residual <= 1e-12 and rep.max_pressure_residual <= 1e-10
        out.append((runs.back(vbar, m, 3), runs.back(p0, m, 1)))
    for a, b in zip(*out):
        err = np.abs(a - b).max() / np.abs(b).max()
        print(f"  step difference {err:.2e}", flush=True)
        assert err <= 1e-9
