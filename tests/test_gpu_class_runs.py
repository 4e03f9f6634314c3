"""Kernels for meshes whose 64-element runs share a geometry class against the
general ones, on the same mesh: in the library's element order every run of
these periodic cubes is one class; in the input order (reorder = 0) every run
mixes the six Kuhn classes, so the general kernels serve it.

A time step solves its systems to 1e-12 (viscous) and 1e-12 (pressure)
relative residuals, whose errors on these meshes stay within 1e3 times that.
"""

import numpy as np
import pytest
import torch

import paper_1601_07384_amd as P
from stdg_inputs import fourier_modes, fourier_velocity, kuhn_mesh, node_coordinates

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def dev(a):
    return torch.tensor(np.ascontiguousarray(a).ravel(), dtype=torch.float64, device=DEV)


def back(t, m, comps):
    """Device element vector -> input element order."""
    v = t.cpu().numpy().reshape(comps, m.E, m.Nst)
    out = np.empty_like(v)
    out[:, m.permutation()] = v
    return out


def step(m, n_pic, v0):
    """A step on one mesh from nodal values v0 [3, E, G, N] in input order."""
    perm = m.permutation()
    vbar = dev(v0[:, perm])
    vhat = torch.empty(3 * m.n_face * m.Nst, dtype=torch.float64, device=DEV)
    m.dual_from_main(vbar, vhat)
    p = torch.zeros(m.E * m.Nst, dtype=torch.float64, device=DEV)
    rep = m.picard_step(vhat, vbar, p, None, opts=P.step_opts(
        n_picard=n_pic,
        pressure={"method": P.STDG_CG_TIME, "precision": P.STDG_FP32, "rtol": 1e-12, "inner_rtol": 1e-5,
                  "max_iter": 50000},
        viscous={"method": P.STDG_BICGSTAB, "restart": 10, "rtol": 1e-12, "check_every": 1}))
    assert rep.max_viscous_residual <= 1e-12 and rep.max_pressure_residual <= 1e-10
    return back(vbar, m, 3), back(p, m, 1)


@pytest.mark.parametrize("n,p,pg", [(4, 1, 0), (4, 1, 4), (8, 1, 1), (4, 2, 0), (4, 2, 1), (4, 2, 3), (4, 2, 4),
                                    (4, 3, 0), (8, 3, 0), (4, 3, 1), (4, 3, 2), (4, 4, 0), (4, 4, 1)])
def test_class_runs_match_general_kernels(n, p, pg):
    print(f"class runs n={n} p={p} pg={pg}", flush=True)
    X, T = kuhn_mesh(n)
    v = fourier_velocity(node_coordinates(X, T, p), fourier_modes(seed=5, n_modes=6, kmax=2))
    v0 = np.transpose(v, (2, 0, 1))[:, :, None, :] * (1.0 + 0.1 * np.arange(pg + 1))[None, None, :, None]
    out = []
    for reorder in (True, False):
        m = P.Mesh(X, T, p, pg, dt=2e-3, nu=2e-2, periodic=True, reorder=reorder)
        out.append(step(m, 2, v0))
    for a, b in zip(*out):
        err = np.abs(a - b).max() / np.abs(b).max()
        print(f"  step difference {err:.2e}", flush=True)
        assert err <= 1e-9


def face_keys(m):
    """A number per face that does not depend on the element order."""
    left, lf, right, rf = m.faces()
    perm = m.permutation()
    a = perm[left] * 4 + lf
    return np.where(right >= 0, np.minimum(a, perm[np.maximum(right, 0)] * 4 + rf), a)


@pytest.mark.parametrize("n,p,pg,periodic", [(4, 1, 0, True), (8, 1, 4, True), (4, 2, 0, True), (8, 2, 1, True),
                                             (4, 2, 4, True), (4, 3, 0, True), (8, 3, 1, True), (4, 3, 3, True),
                                             (4, 4, 0, True), (4, 4, 1, True), (4, 4, 4, True), (16, 1, 0, False),
                                             (16, 2, 1, False)])
def test_transfers_match_general_kernels(n, p, pg, periodic):
    """Dual from main, main from dual and the divergence of random fields, each
    from the same input on both orders; walls (whole and mixed runs and face
    groups, one-sided faces) against the input order too.  Sums of at most
    12 N products of random sign: 1e-12 of the largest value; at p = 4 the
    blocks themselves (conditions up to 3e9, extended precision) differ by up
    to 1e-13 between representatives: 1e-11."""
    print(f"transfers n={n} p={p} pg={pg} periodic={periodic}", flush=True)
    X, T = kuhn_mesh(n)
    rng = np.random.default_rng(8)
    got = []
    vb = vh = None
    for reorder in (True, False):
        m = P.Mesh(X, T, p, pg, dt=2e-3, nu=2e-2, periodic=periodic, reorder=reorder)
        if vb is None:
            vb = rng.standard_normal((3, m.E, m.Nst))
            vh = rng.standard_normal((3, m.n_face, m.Nst))
        perm, order = m.permutation(), np.argsort(face_keys(m))
        rank = np.empty_like(order)
        rank[order] = np.arange(m.n_face)
        vbar, vhat = dev(vb[:, perm]), dev(vh[:, rank])
        dual, main = torch.empty_like(vhat), torch.empty_like(vbar)
        div = torch.empty(m.E * m.Nst, dtype=torch.float64, device=DEV)
        m.dual_from_main(vbar, dual)
        m.main_from_dual(vhat, main)
        m.divergence(vhat, div)
        got.append((dual.cpu().numpy().reshape(3, m.n_face, m.Nst)[:, order], back(main, m, 3), back(div, m, 1)))
    for a, b in zip(*got):
        assert np.abs(a - b).max() <= (1e-12 if p < 4 else 1e-11) * np.abs(b).max()
