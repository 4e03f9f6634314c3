"""The second level's kernels on every padded grid size (16 T lines, T up to 5,
unequal between the planes' directions and the columns) and on the small grids
of one workgroup up to their limits (1,024 nodes, 16 lines; 384 nodes with the
gather inside), as in the other two-level tests.
"""

import pytest

import test_gpu_two_level as two
from stdg_inputs import kuhn_mesh

pytestmark = pytest.mark.gpu

BOXES = [(40, 4, 3), (5, 60, 4), (75, 3, 4), (3, 4, 70), (4, 3, 40), (20, 36, 3), (16, 16, 4), (16, 8, 3), (6, 8, 8)]


@pytest.mark.parametrize("n,p,pg", [(n, 1 + i % 3, i % 2) for i, n in enumerate(BOXES)])
def test_boxes(n, p, pg):
    size = tuple(k / 8 for k in n)
    two.test_two_level_solve((f"{n} p={p} pg={pg}", lambda: two.box_mesh(n, size), p, pg, True, size, True))


@pytest.mark.parametrize("n,p,pg", [(6, 2, 1), (7, 2, 0), (10, 1, 0)])
def test_cubes_with_walls(n, p, pg):
    two.test_two_level_solve((f"walls {n} p={p} pg={pg}", lambda: kuhn_mesh(n), p, pg, False, None, True))
