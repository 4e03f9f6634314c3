"""The two-level CG on meshes whose vertices are graded towards a corner and
scattered: a few grid nodes then hold most of the corners.
"""

import numpy as np
import pytest
import torch

import paper_1601_07384_amd as P
from test_gpu_two_level import DEV, KUHN_PERMS

pytestmark = pytest.mark.gpu


def graded_lines(n, ratio, two_sided=False):
    """n cells on [0, 1] in geometric progression, widest / narrowest = ratio."""
    e = np.arange(n) / (n - 1)
    if two_sided:
        e = np.minimum(np.arange(n), np.arange(n)[::-1]) / ((n - 1) // 2)
    x = np.concatenate([[0.0], np.cumsum(ratio ** e)])
    return x / x[-1]


def graded_mesh(lines, jitter=0.0):
    """Kuhn mesh on the lines, interior vertices moved by up to jitter times the
    narrower of the spacings beside them."""
    m = [len(l) for l in lines]
    kk, jj, ii = np.meshgrid(*(np.arange(k) for k in m[::-1]), indexing="ij")
    at = [a.ravel() for a in (ii, jj, kk)]
    X = np.stack([l[a] for l, a in zip(lines, at)], axis=1)
    inside = np.all([(a > 0) & (a < k - 1) for a, k in zip(at, m)], axis=0)
    u = np.random.default_rng(7).uniform(-jitter, jitter, size=X.shape)
    for d in range(3):
        h = np.diff(lines[d])
        a = at[d][inside]
        X[inside, d] += np.minimum(h[a - 1], h[a]) * u[inside, d]
    step = np.array([1, m[0], m[0] * m[1]])
    ck, cj, ci = np.meshgrid(*(np.arange(k - 1) for k in m[::-1]), indexing="ij")
    corner = (ci + m[0] * (cj + m[1] * ck)).ravel()
    off = np.array([[0, step[s[0]], step[s[0]] + step[s[1]], step.sum()] for s in KUHN_PERMS])
    return X, (corner[:, None, None] + off[None]).reshape(-1, 4)


def system(m, X, T):
    """(x, b = S x) on the device, x smooth with a little noise."""
    cent = torch.tensor(X[T[m.permutation()]].mean(axis=1) / X.max(axis=0), device=DEV)
    g = torch.Generator(device=DEV).manual_seed(4)
    x = 0.01 * torch.randn(m.E, m.G, m.N, generator=g, dtype=torch.float64, device=DEV)
    x += torch.sin(2 * np.pi * (cent[:, 0] + 2 * cent[:, 1]) + 0.3)[:, None, None]
    b = torch.empty(m.E * m.Nst, dtype=torch.float64, device=DEV)
    m.apply(x.reshape(-1).contiguous(), b)
    return x, b


@pytest.mark.parametrize("ratio", [10, 1000])
def test_memory_of_the_tables(ratio):
    """What the second level adds to a mesh: at most 32 corner weights per
    element (256 bytes), positions, work vectors and the grid, however unevenly
    the nodes share the corners; 2.5 KB and more if every node's entries were
    padded to the fullest's.  A mesh with one corner pulled out by a thousandth
    of the spacing does not fill its box and has none."""
    print("two-level, graded and scattered, ratio", ratio, flush=True)
    X, T = graded_mesh([graded_lines(14, ratio)] * 3, 0.2)
    used = []
    for pull in (1.0, 1.0, 0.0):      # (the first build also loads the kernels)
        Y = X.copy()
        Y[0] -= pull * 1e-3 * X[X[:, 0] > 0, 0].min()
        torch.cuda.synchronize()
        free = torch.cuda.mem_get_info()[0]
        m = P.Mesh(Y, T, 1, 0, dt=1e-2)
        used.append(free - torch.cuda.mem_get_info()[0])
        del m
    print("  bytes per element:", [round(u / len(T)) for u in used], flush=True)
    assert used[2] - used[1] <= 1024 * len(T)


CASES = [
    # name, n per direction, grading per direction (sign: two-sided), jitter, p, p_gamma, periodic, second level
    ("scattered, 10", (8, 8, 8), (10, 10, 10), 0.2, 2, 0, False, True),
    ("scattered, 30", (8, 8, 8), (30, 30, 30), 0.2, 1, 0, False, False),
    ("scattered, 30 both ends", (8, 8, 8), (-30, -30, -30), 0.2, 2, 0, False, False),
    ("scattered, 100", (8, 8, 8), (100, 100, 100), 0.2, 3, 0, False, False),
    ("scattered, 100 both ends", (8, 8, 8), (-100, -100, -100), 0.2, 2, 1, False, False),
    ("scattered, 300", (8, 8, 8), (300, 300, 300), 0.2, 1, 0, False, False),
    ("scattered periodic, 10", (8, 8, 8), (10, 10, 10), 0.2, 1, 0, True, False),
    ("tensor, 100 in z", (8, 8, 8), (1, 1, 100), 0.0, 2, 0, False, True),
    ("tensor, 1e4 in z", (6, 6, 6), (1, 1, 1e4), 0.0, 3, 0, False, False),
    ("tensor, 1000", (4, 4, 4), (1000, 1000, 1000), 0.0, 1, 0, False, False),
    ("tensor periodic, 4 in z", (8, 8, 16), (1, 1, 4), 0.0, 2, 1, True, True),
    ("tensor periodic, 64 in z", (8, 8, 16), (1, 1, 64), 0.0, 2, 1, True, False),
    ("tensor periodic, p = 4, 64 in z", (8, 8, 8), (1, 1, 64), 0.0, 4, 0, True, True),
]


@pytest.mark.parametrize("case", CASES, ids=[c[0] for c in CASES])
def test_second_level_only_where_it_pays(case):
    """With the polls 64 iterations apart block Jacobi alone takes a multiple of
    64, the two-level CG the iterations that it needs.  Where the second level is
    used it has to halve the iterations, or nearly (an iteration takes about
    twice as long), of the same mesh with its corners pulled out by a thousandth
    of a spacing, which no longer fills its box and so has block Jacobi alone."""
    name, n, grading, jitter, p, pg, periodic, second = case
    print("two-level,", name, flush=True)
    X, T = graded_mesh([graded_lines(k, abs(g), g < 0) for k, g in zip(n, grading)], jitter)
    its = []
    for pull in (0.0, 1.0) if second else (0.0,):
        Y = X.copy()
        corner = np.all((X == 0.0) | (X == 1.0), axis=1)
        Y[corner if periodic else 0] -= pull * 1e-3 * X[X > 0].min()
        m = P.Mesh(Y, T, p, pg, dt=1e-2, periodic=periodic)
        x, b = system(m, Y, T)
        xs = torch.zeros_like(b)
        rep = m.solve(b, xs, method=P.STDG_CG_TIME, precision=P.STDG_FP32, rtol=1e-8, inner_rtol=1e-4,
                      max_iter=64000, check_every=64)
        assert rep.status == 0 and rep.rel_residual <= 1e-8
        its.append(rep.inner_iters)
    print(f"  {m.E} elements, iterations: {its}", flush=True)
    assert (its[0] % 64 != 0) == second
    if second:
        assert its[1] % 64 == 0 and its[0] < 0.55 * its[1]


@pytest.mark.parametrize("n,p,pg,second", [(6, 2, 0, False), (7, 2, 0, True), (7, 2, 1, False), (9, 2, 1, True),
                                           (9, 1, 2, False), (8, 3, 2, True)])
def test_least_elements_of_periodic_meshes(n, p, pg, second):
    """Runs that mix classes (all but n = 8): from 2,000 elements per time node."""
    print(f"two-level, periodic n={n} p={p} pg={pg}", flush=True)
    X, T = graded_mesh([graded_lines(n, 1.0)] * 3)
    m = P.Mesh(X, T, p, pg, dt=1e-2, periodic=True)
    x, b = system(m, X, T)
    xs = torch.zeros_like(b)
    rep = m.solve(b, xs, method=P.STDG_CG_TIME, precision=P.STDG_FP32, rtol=1e-8, inner_rtol=1e-4, check_every=64)
    assert rep.status == 0 and rep.rel_residual <= 1e-8
    print("  iterations:", rep.inner_iters, flush=True)
    assert (rep.inner_iters % 64 != 0) == second
