"""Priors much wider than what the measurements leave, and measurements much more accurate than the filter's
prediction: the later windows' information then shrinks a window's covariance many times over (J P >> 1),
which the smoother has to do without losing the digits in between. Against the float64 oracle, at the
repository's tolerances (1e-8 float64, 1e-3 float32 on the rounded inputs).
"""
import numpy as np
import pytest
import torch

import oracle
from paper_2410_00627_amd import workloads as wl
from test_gpu_lag1 import lag1_error
from test_gpu_settled import TOL, _errors

pytestmark = pytest.mark.gpu


def _model(kind, nx, ny, L, seed, wide, r):
    m = (wl.random_stable_model if kind == "stable" else wl.random_general_model)(nx, ny, L, seed)
    m.P0, m.R = wide * m.P0, r * m.R
    return m


def _run(m, N, seed, dtype, **kw):
    from paper_2410_00627_amd import srtm
    args = [t.to(dtype) for t in srtm.model_tensors(m, "cuda", torch.float64)]
    yt = torch.as_tensor(wl.simulate(m, N, seed), device="cuda").to(dtype)
    out = srtm.smooth(*args[:4], m.L, *args[4:], yt, **kw)
    a = [t.double().cpu().numpy() for t in (*args, yt)]
    return out, oracle.srtm_smoother(a[0], a[1], a[2], a[3], m.L, a[4], a[5], a[6], with_filter=True, lag1=True)


COVARIANCES = [  # P^s was 2e-8 .. 1e-5 off in float64, 6e-3 in float32, with W in the element type and its upper half mirrored
    ("stable", 3, 2, 10, 0, 1e4, 1.0, 30, torch.float64), ("stable", 4, 1, 1, 2, 100.0, 1.0, 30, torch.float64),
    ("stable", 4, 2, 10, 1, 1e4, 1.0, 30, torch.float64), ("stable", 6, 1, 1, 1, 100.0, 1.0, 30, torch.float64),
    ("general", 4, 2, 4, 5, 1e4, 1e-2, 30, torch.float64), ("stable", 4, 2, 4, 3, 1e4, 1.0, 5 * 256 + 19, torch.float64),
    ("stable", 6, 1, 4, 3, 1e4, 1.0, 5 * 256 + 19, torch.float64), ("stable", 3, 2, 10, 0, 100.0, 1.0, 30, torch.float32),
]


@pytest.mark.parametrize("kind,nx,ny,L,seed,wide,r,N,dtype", COVARIANCES)
def test_smoothed_covariances(kind, nx, ny, L, seed, wide, r, N, dtype):
    out, ref = _run(_model(kind, nx, ny, L, seed, wide, r), N, 60 + seed, dtype)
    P, Pr = out["Ps_fast"].double().cpu().numpy(), ref["Ps_fast"]
    assert np.max(np.linalg.norm(P - Pr, axis=(-2, -1)) / np.linalg.norm(Pr, axis=(-2, -1))) <= TOL[dtype]
    assert torch.equal(out["Ps_fast"], out["Ps_fast"].mT)


STATES = [  # the filter's means and covariances were 2e-8 .. 1e-6 off in float64, 2e-3 .. 7e-2 in float32
    ("general", 2, 1, 4, 4, 1e4, 1.0, torch.float64), ("stable", 2, 1, 10, 1, 1e4, 1.0, torch.float64),
    ("general", 3, 1, 1, 5, 1e4, 1e-2, torch.float64), ("stable", 4, 2, 1, 1, 1e4, 1.0, torch.float64),
    ("stable", 4, 1, 10, 0, 1e4, 1.0, torch.float64), ("stable", 4, 1, 1, 1, 100.0, 1.0, torch.float32),
    ("stable", 4, 2, 1, 1, 100.0, 1.0, torch.float32),
]


@pytest.mark.parametrize("N", [30, 2 * 256 + 17])
@pytest.mark.parametrize("kind,nx,ny,L,seed,wide,r,dtype", STATES)
def test_filter_states(kind, nx, ny, L, seed, wide, r, dtype, N):
    from paper_2410_00627_amd import srtm
    m = _model(kind, nx, ny, L, seed, wide, r)
    out, ref = _run(m, N, 60 + seed, dtype, with_filter=True)
    args = [t.to(dtype) for t in srtm.model_tensors(m, "cuda", torch.float64)]
    alone = srtm.filter(*args[:4], L, *args[4:], torch.as_tensor(wl.simulate(m, N, 60 + seed), device="cuda").to(dtype))
    for o, k, rk in ((out, "ms_fast", "ms_fast"), (out, "mf_fast", "m_fast"), (out, "mf_slow", "m_slow"),
                     (alone, "m_fast", "m_fast"), (alone, "m_slow", "m_slow")):
        P, Pr = o[k.replace("m", "P", 1)], ref[rk.replace("m", "P", 1)]
        e = _errors(o[k], P, ref[rk], Pr)
        assert e[0] <= TOL[dtype] and (k == "ms_fast" or e[1] <= TOL[dtype]), (k, e)


@pytest.mark.parametrize("r", [1e-3, 1e-4])
def test_accurate_measurements_float32(r):
    """J P about 700 in every window, settled tiles and the others. From the second window on: the first one's
    filter covariance, of which 1/500 is left, is itself 5e-6 off, the rounding of its prior."""
    out, ref = _run(_model("general", 2, 1, 1, 4, 1.0, r), 6 * 256 + 5, 91, torch.float32, lag1=True)
    e = _errors(out["ms_fast"][1:], out["Ps_fast"][1:], ref["ms_fast"][1:], ref["Ps_fast"][1:])
    assert max(e) <= TOL[torch.float32]
    C = out["Cs_fast"][1:].double().cpu().numpy()
    assert lag1_error(C, ref["Cs_fast"][1:], ref["Ps_fast"][1:]) <= TOL[torch.float32]


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32], ids=["f64", "f32"])
@pytest.mark.parametrize("nx,ny,L", [(2, 1, 1), (4, 2, 4), (3, 1, 2)])
def test_slow_filter_means_are_the_last_fast_step(nx, ny, L, dtype):
    """The mean of x_{k,L} given y_{1:k} twice, as the slow-rate output and as the last fast step of the same window
    update: equal to the rounding of its sums (some 20 terms each, 64 units allowed). The slow-rate covariance, which
    is not taken from that update, against the float64 oracle: in float32 it keeps digits that the update's loses."""
    from paper_2410_00627_amd import srtm
    m = _model("general", nx, ny, L, 4, 1.0, 1e-4)
    N = 6 * 256 + 5
    args = [t.to(dtype) for t in srtm.model_tensors(m, "cuda", torch.float64)]
    yt = torch.as_tensor(wl.simulate(m, N, 91), device="cuda").to(dtype)
    out = srtm.smooth(*args[:4], L, *args[4:], yt, with_filter=True)
    P = out["Pf_fast"][:, -1].double().cpu().numpy()
    e = _errors(out["mf_slow"], out["Pf_slow"], out["mf_fast"][:, -1].double().cpu().numpy(), P)
    assert e[0] <= 64 * torch.finfo(dtype).eps
    a = [t.double().cpu().numpy() for t in (*args, yt)]
    ref = oracle.srtm_smoother(a[0], a[1], a[2], a[3], L, a[4], a[5], a[6], with_filter=True)
    assert _errors(out["mf_slow"], out["Pf_slow"], ref["m_slow"], ref["P_slow"])[1] <= 1e-2 * TOL[dtype]


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32], ids=["f64", "f32"])
@pytest.mark.parametrize("nx,ny,L,nu", [(2, 1, 1, 0), (4, 2, 4, 0), (3, 1, 20, 3), (6, 1, 40, 0)])
def test_slow_filter_outputs_beside_smoothed_ones(nx, ny, L, nu, dtype):
    """Without the fast filter outputs the slow ones come from another kernel (or, at nx = 6 with long windows, from a
    second pass): the same numbers as with them, to the rounding of their sums (64 units allowed)."""
    from paper_2410_00627_amd import srtm
    m, N = wl.random_stable_model(nx, ny, L, 4), 2 * 256 + 9
    args = [t.to(dtype) for t in srtm.model_tensors(m, "cuda", torch.float64)]
    B, u = wl.random_inputs(nx, nu, L, N, 32) if nu else (None, None)
    yt = torch.as_tensor(wl.simulate(m, N, 91, B=B, u=u), device="cuda").to(dtype)
    kw = dict(B=torch.as_tensor(B, device="cuda").to(dtype), u=torch.as_tensor(u, device="cuda").to(dtype)) if nu else {}
    all_ = srtm.smooth(*args[:4], L, *args[4:], yt, with_filter=True, **kw)
    out = {k: torch.empty_like(all_[k]) for k in ("ms_fast", "Ps_fast", "ms_slow", "Ps_slow", "mf_slow", "Pf_slow")}
    srtm.smooth(*args[:4], L, *args[4:], yt, out=out, **kw)
    for mk, pk in (("mf_slow", "Pf_slow"), ("ms_slow", "Ps_slow"), ("ms_fast", "Ps_fast")):
        e = _errors(out[mk], out[pk], all_[mk].double().cpu().numpy(), all_[pk].double().cpu().numpy())
        assert max(e) <= 64 * torch.finfo(dtype).eps, (mk, e)
