"""Batches around the numbers of tiles and sequences where the recovery's split of the end tiles changes (5, 3, 2
parts and none), with sequences shorter than the tiles that may be split: bitwise equal to one call per sequence.
"""
import pytest
import torch

from paper_2410_00627_amd import workloads as wl

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32], ids=["f64", "f32"])
@pytest.mark.parametrize("nx,nseq,N", [(4, 2, 3000), (4, 4, 3000), (4, 7, 3001), (4, 8, 3000), (4, 15, 3000), (4, 17, 3000),
                                       (4, 33, 2000), (2, 4, 3000), (2, 15, 3000), (2, 17, 3000), (3, 9, 2500)])
def test_batch_equals_single_calls(nx, nseq, N, dtype):
    from paper_2410_00627_amd import srtm
    L, probs = 9, []
    for j in range(nseq):
        m = wl.random_stable_model(nx, 1, L, 70 + j)
        n = N if j % 3 else max(1, N // (1 + j % 7))
        F, Q, H, R, m0, P0 = (t.to(dtype) for t in srtm.model_tensors(m, "cuda", torch.float64))
        probs.append((F, Q, H, R, L, m0, P0, torch.as_tensor(wl.simulate(m, n, 71 + j), device="cuda").to(dtype)))
    got = srtm.smooth_batch(probs)
    for p, g in zip(probs, got):
        one = srtm.smooth(*p)
        for k in ("ms_fast", "Ps_fast", "ms_slow", "Ps_slow"):
            assert torch.equal(g[k], one[k]), k
