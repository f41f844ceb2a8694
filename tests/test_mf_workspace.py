"""Workspace of the filter forward: the query is the least, so that a shape has one
result; the static scratch takes calls whose query it does not hold, by their shape."""
import ctypes

import numpy as np
import pytest
import torch

from synth import freq_grid


@pytest.mark.parametrize("n_meas,n_freq,n_q", [(64, 32, 4096), (3200, 64, 500), (1, 33, 1), (1024, 64, 1 << 20), (256, 64, 1 << 21)])
@pytest.mark.parametrize("two", [0, 1])
def test_less_than_the_query_is_refused(n_meas, n_freq, n_q, two):
    """Few points (splits of the measurements), many (cells) and neither; nothing is enqueued."""
    from paper_2605_29097_amd import rfvr as R
    L = R.lib()
    v, ws = ctypes.c_void_p(4096), ctypes.c_void_p(256)
    ap = R.CAperture(n_meas, v, None, 77e9, 1e6, n_freq)
    need = L.rfvr_mf_forward_ws_bytes(ctypes.byref(ap), n_q, two)
    assert need > 0
    s2, o2 = (v, v) if two else (None, None)
    assert L.rfvr_mf_forward(ctypes.byref(ap), v, n_q, 0, v, v, v, s2, o2, o2, ws, need - 1, None) == -2


@pytest.mark.gpu
@pytest.mark.parametrize("n_meas,two", [(30001, False), (30801, False), (30831, False), (15001, True)])
def test_static_scratch_with_room_for_some_splits(dev, n_meas, two):
    """500 points and as many measurements as leave the scratch room for 222, 10, 2 and 228 of the 1024 splits (the
    measurements are no multiple of them).  Tolerance as where the series meet the per-frequency kernels: phases rounded to FP32
    on either side and sums of 30001 terms at 2^-24 sqrt(n) = 1.0e-5."""
    from paper_2605_29097_amd import rfvr as R
    rng = np.random.default_rng(3)
    f0, df = freq_grid(33)
    t = lambda a: torch.from_numpy(np.ascontiguousarray(a, np.float32)).to(dev)
    ap = R.Aperture(tx=t(np.concatenate([rng.uniform(-0.04, 0.04, (n_meas, 2)), np.zeros((n_meas, 1))], 1)), f0=f0, df=df, n_freq=33)
    x = t(rng.uniform(-0.05, 0.05, (500, 3)) + [0.0, 0.0, 0.3])
    sig = [t(rng.normal(size=(n_meas, 33, 2))) for _ in range(2 if two else 1)]
    query = R.lib().rfvr_mf_forward_ws_bytes(ctypes.byref(ap.c()), 500, int(two))
    assert query > R.MF_STATIC_SCRATCH_BYTES
    got, want = R.mf_forward_static(ap, x, *sig), R.mf_forward(ap, x, *sig, flags=R.TERMS_DIRECT)
    full = R.mf_forward(ap, x, *sig)
    again = R.mf_forward_static(ap, x, *sig)
    for a, b, c, d in zip(got, want, full, again):
        assert float((a.double() - b.double()).norm() / b.double().norm()) < 1.5e-5
        assert float((c.double() - b.double()).norm() / b.double().norm()) < 1.5e-5
        assert torch.equal(a, d)
