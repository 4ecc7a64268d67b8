"""The gradient's statistics at window lengths around its 32-step LDS tables (one step, a full table, a second
table of one step, three tables) and at 4 to 74 sums per tile. Against central differences of the float64
reference at the repository's tolerance for them.
"""
import pytest
import torch

from test_gpu_loglik import test_loglik_and_gradient_against_finite_differences as check

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nx,ny,L,N", [(1, 1, 40, 300), (2, 2, 33, 60), (3, 2, 32, 50), (4, 1, 65, 30), (6, 1, 33, 40), (6, 1, 1, 70)])
def test_table_steps(nx, ny, L, N):
    check(nx, ny, L, N, 500 + L, torch.float64)
