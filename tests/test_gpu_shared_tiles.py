"""Settled tiles: far from the ends of a sequence that settles, the fold shares one set of matrices among the 256 windows
of a tile, so their covariances are the same to the last bit; near the ends, and for models that don't settle within the
sequence, every window has its own.
"""
import pytest
import torch

from paper_2410_00627_amd import srtm
from paper_2410_00627_amd import workloads as wl

pytestmark = pytest.mark.gpu

NT = 12
N = NT * 256 + 40


def covariances(m, dtype):
    y = torch.as_tensor(wl.simulate(m, N, 1)).cuda().to(dtype)
    a = [t.to(dtype) for t in srtm.model_tensors(m, "cuda", torch.float64)]
    out = srtm.smooth(*a[:4], m.L, *a[4:], y, with_filter=True)
    out.update(Cs_fast=srtm.smooth(*a[:4], m.L, *a[4:], y, lag1=True)["Cs_fast"])
    return {k: out[k] for k in ("Pf_fast", "Ps_fast", "Cs_fast")}


def shared(P, tile):
    P = P[tile * 256:(tile + 1) * 256]
    return bool((P == P[:1]).all())


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32], ids=["f64", "f32"])
@pytest.mark.parametrize("nx,ny", [(2, 1), (2, 2), (3, 1), (3, 2), (4, 1), (4, 2)])
def test_middle_tiles_share(nx, ny, dtype):
    # spectral radius 0.99: after six tiles the start is forgotten to 0.99^(2 * 5 * 1536) < 1e-66
    for name, P in covariances(wl.random_stable_model(nx, ny, 5, 3), dtype).items():
        assert shared(P, 6), name
        assert not shared(P, 0), name
        if name != "Pf_fast":
            assert not shared(P, NT), name  # the last 40 windows


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32], ids=["f64", "f32"])
@pytest.mark.parametrize("nx,ny", [(2, 1), (3, 2), (4, 2)])
def test_slow_models_share_nothing(nx, ny, dtype):
    # hardly any noise of the process: over the whole sequence the start is forgotten to 0.9999^(2 * 2 * 3112) = 0.29
    for name, P in covariances(wl.random_stable_model(nx, ny, 2, 0, rho=0.9999, q=1e-10, r=0.1), dtype).items():
        for tile in range(NT):
            assert not shared(P, tile), (name, tile)
