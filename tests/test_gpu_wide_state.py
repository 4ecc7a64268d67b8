"""Six states on the matrix cores (the level chain, the tile-level and wave-level steps of the fold, the
information of the last windows): states of very different scales, whose matrix I + D J needs its rows
exchanged in the elimination, and lengths around the waves of the last tile. Against the float64 oracle at
the repository's tolerances (1e-8 float64, 1e-3 float32 on the rounded inputs), errors taken in the unscaled
coordinates.
"""
import numpy as np
import pytest
import torch

import oracle
from paper_2410_00627_amd import workloads as wl

pytestmark = pytest.mark.gpu
TOL = {torch.float64: 1e-8, torch.float32: 1e-3}


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32], ids=["f64", "f32"])
@pytest.mark.parametrize("N", [63, 64, 129, 255, 256 + 64, 512 + 191, 5 * 256 + 192])
@pytest.mark.parametrize("scaled", [False, True], ids=["plain", "scaled"])
def test_six_states(N, scaled, dtype):
    from paper_2410_00627_amd import srtm
    L = 2
    m = wl.random_general_model(6, 1, L, 300 + N)
    s = 2.0 ** np.array([9.0, -8.0, 0.0, 6.0, -3.0, 4.0]) if scaled else np.ones(6)  # exact in both types
    m = wl.Model(m.A * s[:, None] / s, m.Q * np.outer(s, s), m.C / s, m.R, L, m.m0 * s, m.P0 * np.outer(s, s))
    y = wl.simulate(m, N, 301 + N)
    args = [t.to(dtype) for t in srtm.model_tensors(m, "cuda", torch.float64)]
    yt = torch.as_tensor(y, device="cuda").to(dtype)
    out = srtm.smooth(*args[:4], L, *args[4:], yt, with_filter=True)
    a = [t.double().cpu().numpy() for t in (*args, yt)]
    ref = oracle.srtm_smoother(a[0], a[1], a[2], a[3], L, a[4], a[5], a[6], with_filter=True)
    for mk, pk, rm, rp in (("ms_fast", "Ps_fast", "ms_fast", "Ps_fast"), ("mf_fast", "Pf_fast", "m_fast", "P_fast")):
        g, P = out[mk].double().cpu().numpy() / s, out[pk].double().cpu().numpy() / np.outer(s, s)
        gr, Pr = ref[rm] / s, ref[rp] / np.outer(s, s)
        nm = np.maximum(np.linalg.norm(gr, axis=-1), np.sqrt(np.trace(Pr, axis1=-2, axis2=-1)))
        assert np.max(np.linalg.norm(g - gr, axis=-1) / nm) <= TOL[dtype], mk
        assert np.max(np.linalg.norm(P - Pr, axis=(-2, -1)) / np.linalg.norm(Pr, axis=(-2, -1))) <= TOL[dtype], pk
