"""A measurement that is not a number: the filter's outputs before it depend on no later data, and the blocks
of every window's covariances on no data at all, whether the outputs are asked for alone or together.
"""
import numpy as np
import pytest
import torch

from paper_2410_00627_amd import workloads as wl

pytestmark = pytest.mark.gpu
N, BAD = 6 * 256 + 77, 5 * 256 + 40  # settled tiles before the bad window


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32], ids=["f64", "f32"])
@pytest.mark.parametrize("value", [np.nan, np.inf], ids=["nan", "inf"])
@pytest.mark.parametrize("nx,ny", [(1, 1), (2, 1), (2, 2), (3, 1), (3, 2), (4, 1), (4, 2), (6, 1)])
def test_filter_before_it_is_unchanged(nx, ny, value, dtype):
    from paper_2410_00627_amd import srtm
    m = wl.random_stable_model(nx, ny, 5, 21)
    F, Q, H, R, m0, P0 = (t.to(dtype) for t in srtm.model_tensors(m, "cuda", torch.float64))
    y = torch.as_tensor(wl.simulate(m, N, 22), device="cuda").to(dtype)
    bad = y.clone()
    bad[BAD, 0] = value
    for call, keys in ((lambda t: srtm.smooth(F, Q, H, R, 5, m0, P0, t, with_filter=True, check=False), ("mf", "Pf")),
                       (lambda t: srtm.filter(F, Q, H, R, 5, m0, P0, t, check=False), ("m", "P"))):
        good, out = call(y), call(bad)
        assert int(good["info"].item()) == 0 and int(out["info"].item()) & 8
        for k in (f"{keys[0]}_fast", f"{keys[0]}_slow"):
            assert torch.equal(out[k][:BAD], good[k][:BAD]), k
        for k in out:
            if k.startswith("P"):
                assert torch.equal(out[k], good[k]), k
