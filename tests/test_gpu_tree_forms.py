"""The tile trees in rows (nx = 1, 2) and on the matrix cores (nx = 3) at the edges of a tile, against the float64
oracle at the repository's tolerances.
"""
import pytest
import torch

from test_gpu_fold import test_fold_sizes as check

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32], ids=["f64", "f32"])
@pytest.mark.parametrize("nx,ny", [(1, 1), (2, 1), (2, 2), (3, 1)])
@pytest.mark.parametrize("N", [1, 2, 31, 255, 257, 513, 3 * 256 + 130])
def test_tree_forms(N, nx, ny, dtype):
    check(N, nx, ny, dtype)
