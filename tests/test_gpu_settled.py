"""Settled tiles (windows that share their covariances) and the split of the end tiles: window lengths
around the recovery's step groups, records that do not divide a cache line, filter and smoother outputs
together, known inputs, and models that must not be taken for settled. N spans 9 tiles with a partial
last one, so the middle tiles settle and the ends do not. Against the float64 oracle, at the
repository's tolerances (1e-8 float64, 1e-3 float32 on the rounded inputs).
"""
import numpy as np
import pytest
import torch

import oracle
from paper_2410_00627_amd import workloads as wl

pytestmark = pytest.mark.gpu
TOL = {torch.float64: 1e-8, torch.float32: 1e-3}
N = 8 * 256 + 77


def _errors(m, P, mr, Pr):
    m, P = m.double().cpu().numpy(), P.double().cpu().numpy()
    nm = np.maximum(np.linalg.norm(mr, axis=-1), np.sqrt(np.trace(Pr, axis1=-2, axis2=-1)))
    return (float(np.max(np.linalg.norm(m - mr, axis=-1) / nm)),
            float(np.max(np.linalg.norm(P - Pr, axis=(-2, -1)) / np.linalg.norm(Pr, axis=(-2, -1)))))


def _check(model, y, dtype, B=None, u=None, slow_only=False, n=N):
    from paper_2410_00627_amd import srtm
    L = model.L
    F, Q, H, R, m0, P0 = (t.to(dtype) for t in srtm.model_tensors(model, "cuda", torch.float64))
    yt = torch.as_tensor(y, device="cuda").to(dtype)
    kw = {} if B is None else dict(B=torch.as_tensor(B, device="cuda").to(dtype), u=torch.as_tensor(u, device="cuda").to(dtype))
    a = [t.double().cpu().numpy() for t in (F, Q, H, R, m0, P0, yt)]
    rkw = {k: v.double().cpu().numpy() for k, v in kw.items()}
    ref = oracle.srtm_smoother(a[0], a[1], a[2], a[3], L, a[4], a[5], a[6], with_filter=True, **rkw)
    both = srtm.smooth(F, Q, H, R, L, m0, P0, yt, with_filter=True, fast=not slow_only, **kw)
    filt = srtm.filter(F, Q, H, R, L, m0, P0, yt, fast=not slow_only, **kw)
    only = srtm.smooth(F, Q, H, R, L, m0, P0, yt, fast=not slow_only, **kw)
    pairs = [(o, mk, pk, mk, pk) for o in (both, only) for mk, pk in (("ms_fast", "Ps_fast"), ("ms_slow", "Ps_slow"))]
    pairs += [(both, "mf_fast", "Pf_fast", "m_fast", "P_fast"), (both, "mf_slow", "Pf_slow", "m_slow", "P_slow")]
    pairs += [(filt, k, k.replace("m_", "P_"), k, k.replace("m_", "P_")) for k in ("m_fast", "m_slow")]
    for o, mk, pk, rm, rp in pairs:
        if mk not in o:
            continue
        e = _errors(o[mk], o[pk], ref[rm], ref[rp])
        assert max(e) <= TOL[dtype], (mk, e)
        assert torch.equal(o[pk], o[pk].mT), pk
    return both


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32], ids=["f64", "f32"])
@pytest.mark.parametrize("nx,ny,L", [(4, 2, 1), (4, 2, 7), (4, 1, 24), (4, 2, 25), (4, 2, 49), (3, 1, 5), (3, 2, 32), (2, 2, 20),
                                     (1, 1, 3), (6, 1, 10)])
def test_settled_sizes(nx, ny, L, dtype):
    m = wl.random_general_model(nx, ny, L, 700 + 10 * nx + L)
    _check(m, wl.simulate(m, N, 701 + L), dtype)


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32], ids=["f64", "f32"])
@pytest.mark.parametrize("nx,ny,L,nu", [(4, 2, 20, 2), (3, 1, 9, 4), (2, 1, 26, 1)])
def test_settled_inputs(nx, ny, L, nu, dtype):
    m = wl.random_stable_model(nx, ny, L, 31 + nu)
    B, u = wl.random_inputs(nx, nu, L, N, 32)
    _check(m, wl.simulate(m, N, 33, B=B, u=u), dtype, B, u)


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32], ids=["f64", "f32"])
def test_settled_slow_outputs_only(dtype):
    m = wl.random_stable_model(4, 2, 20, 5)
    _check(m, wl.simulate(m, N, 6), dtype, slow_only=True)


@pytest.mark.parametrize("turn", [0.0, np.pi / 2, 2 * np.pi / 256, 1e-3], ids=["still", "quarter", "tile", "slow"])
def test_unobserved_modes_do_not_pass_for_settled(turn):
    """An undriven, unobserved rotation keeps the covariance turning for ever (by a quarter a window, once
    per tile, slowly, or not at all): its windows differ unless it stands still."""
    c, s = np.cos(turn), np.sin(turn)
    A = np.zeros((4, 4))
    A[:2, :2] = [[0.9, 0.1], [-0.2, 0.8]]
    A[2:, 2:] = [[c, -s], [s, c]]
    Q = np.zeros((4, 4))
    Q[:2, :2] = 0.02 * np.eye(2)
    Q[2:, 2:] = 1e-12 * np.eye(2)  # keeps the prediction covariance positive definite
    m = wl.Model(A, Q, np.array([[1.0, 0.5, 0.0, 0.0]]), np.array([[0.1]]), 1, np.array([0.1, 0.2, 1.0, -1.0]),
                 np.diag([1.0, 1.0, 4.0, 0.25]))
    _check(m, wl.simulate(m, N, 8), torch.float64)


def test_slowly_settling_model():
    """A mode that takes tens of thousands of windows to settle: no tile of this length may share."""
    A = np.diag([0.99999, 0.5])
    m = wl.Model(A, np.diag([1e-9, 0.1]), np.array([[1.0, 1.0]]), np.array([[1.0]]), 2, np.zeros(2), np.diag([1.0, 1.0]))
    _check(m, wl.simulate(m, N, 9), torch.float64)
    _check(m, wl.simulate(m, N, 9), torch.float32)
