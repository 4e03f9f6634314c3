"""FP64 pressure operator at p = 1 on both sides of the size from which meshes
of whole 64-element runs take an element per lane (100,000 elements), and a mesh
that large whose last runs mix classes; at p = 4 with four and five time nodes on
both sides of the numbers of groups from which rows leave eight elements at a time
(256, and at five not between 600 and 768); against the product with the mesh's
own blocks, as in the tests of smaller meshes.
"""

import pytest

import test_gpu_apply_runs as runs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,pg", [((28, 26, 24), 0), ((28, 26, 24), 1), ((27, 26, 24), 1), ((28, 26, 20), 0),
                                  ((28, 26, 24), 2)])
def test_apply_matches_blocks(n, pg):
    runs.test_apply_matches_blocks(n, 1, pg, True, True)


@pytest.mark.parametrize("n,pg", [((10, 10, 9), 3), ((14, 14, 15), 3), ((14, 14, 15), 4), ((19, 19, 19), 4)])
def test_apply_of_rows_in_parts(n, pg):
    runs.test_apply_matches_blocks(n, 4, pg, True, True)
