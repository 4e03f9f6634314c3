"""Meshes of many geometry classes on both sides of the line from which kernels
take groups of one class (each kernel has its own): transfers and a time step
against the same mesh in the input order, where no two neighbouring elements
share a class and the general kernels serve.  Tolerances as in the tests of
small groups.
"""

import numpy as np
import pytest
import torch

import paper_1601_07384_amd as P
import test_gpu_class_runs as runs
from stdg_inputs import fourier_modes, fourier_velocity, node_coordinates
from test_gpu_two_level_graded import graded_mesh

pytestmark = pytest.mark.gpu


def lines(n, seed):
    """n cells of unequal widths: classes of their own in this direction."""
    x = np.cumsum(np.concatenate([[0.0], 1.0 + 0.3 * np.random.default_rng(seed).random(n)]))
    return x / x[-1]


@pytest.mark.parametrize("nx,ny,p,pg", [(4, 9, 1, 1), (8, 9, 1, 4), (4, 9, 2, 2), (8, 9, 2, 2), (4, 12, 2, 1),
                                        (4, 9, 3, 1)])
def test_many_classes(nx, ny, p, pg):
    print(f"group rule nx={nx} ny={ny} p={p} pg={pg}", flush=True)
    X, T = graded_mesh([np.linspace(0.0, 1.0, nx + 1), lines(ny, 1), lines(ny, 2)])
    rng = np.random.default_rng(8)
    v = fourier_velocity(node_coordinates(X, T, p), fourier_modes(seed=5, n_modes=6, kmax=2))
    v0 = np.transpose(v, (2, 0, 1))[:, :, None, :] * (1.0 + 0.1 * np.arange(pg + 1))[None, None, :, None]
    got, steps, vh = [], [], None
    for reorder in (True, False):
        m = P.Mesh(X, T, p, pg, dt=2e-3, nu=2e-2, periodic=True, reorder=reorder)
        if vh is None:
            vb = rng.standard_normal((3, m.E, m.Nst))
            vh = rng.standard_normal((3, m.n_face, m.Nst))
        perm, order = m.permutation(), np.argsort(runs.face_keys(m))
        rank = np.empty_like(order)
        rank[order] = np.arange(m.n_face)
        vbar, vhat = runs.dev(vb[:, perm]), runs.dev(vh[:, rank])
        dual, main = torch.empty_like(vhat), torch.empty_like(vbar)
        div = torch.empty(m.E * m.Nst, dtype=torch.float64, device=runs.DEV)
        m.dual_from_main(vbar, dual)
        m.main_from_dual(vhat, main)
        m.divergence(vhat, div)
        got.append((dual.cpu().numpy().reshape(3, m.n_face, m.Nst)[:, order], runs.back(main, m, 3),
                    runs.back(div, m, 1)))
        steps.append(runs.step(m, 2, v0))
    for a, b in zip(*got):
        assert np.abs(a - b).max() <= 1e-12 * np.abs(b).max()
    for a, b in zip(*steps):
        err = np.abs(a - b).max() / np.abs(b).max()
        print(f"  step difference {err:.2e}", flush=True)
        assert err <= 1e-9
