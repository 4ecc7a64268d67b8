"""The recovery's split of a tile's fast steps over workgroups, at the numbers of tiles where the rule changes
(8 parts of every tile, fewer, the end tiles alone, tiles that do not settle) and at window lengths with fewer
steps than parts, a remainder, and more steps than one LDS table holds. Against the float64 oracle, at the
repository's tolerances (1e-8 float64, 1e-3 float32 on the rounded inputs).
"""
import numpy as np
import pytest
import torch

import oracle
from paper_2410_00627_amd import workloads as wl
from test_gpu_lag1 import lag1_error
from test_gpu_settled import TOL, _check

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32], ids=["f64", "f32"])
@pytest.mark.parametrize("nx,ny,L,N", [(4, 2, 33, 5 * 256), (3, 1, 6, 16 * 256 + 1), (2, 1, 9, 43 * 256), (1, 1, 3, 65 * 256 + 255),
                                       (1, 1, 7, 256 * 256), (6, 1, 9, 3 * 256 + 2), (6, 1, 34, 5 * 256), (6, 1, 3, 86 * 256)])
def test_parts(nx, ny, L, N, dtype):
    m = wl.random_stable_model(nx, ny, L, 40 + L)
    _check(m, wl.simulate(m, N, 41 + L), dtype, n=N)


@pytest.mark.parametrize("L,N", [(10, 8 * 256), (25, 5 * 256 + 3)])
def test_parts_inputs(L, N):
    m = wl.random_stable_model(4, 2, L, 50)
    B, u = wl.random_inputs(4, 2, L, N, 51)
    _check(m, wl.simulate(m, N, 52, B=B, u=u), torch.float64, B, u, n=N)


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32], ids=["f64", "f32"])
@pytest.mark.parametrize("nx,L,N", [(4, 13, 12 * 256 + 9), (4, 3, 44 * 256), (6, 5, 6 * 256 + 1)])
def test_parts_lag1(nx, L, N, dtype):
    from paper_2410_00627_amd import srtm
    m = wl.random_stable_model(nx, 1, L, 60)
    y = wl.simulate(m, N, 61)
    args = [t.to(dtype) for t in srtm.model_tensors(m, "cuda", torch.float64)]
    yt = torch.as_tensor(y, device="cuda").to(dtype)
    out = srtm.smooth(*args[:4], L, *args[4:], yt, lag1=True)
    a = [t.double().cpu().numpy() for t in (*args, yt)]
    ref = oracle.srtm_smoother(a[0], a[1], a[2], a[3], L, a[4], a[5], a[6], lag1=True)
    assert np.max(lag1_error(out["Cs_fast"].double().cpu().numpy(), ref["Cs_fast"], ref["Ps_fast"])) <= TOL[dtype]
