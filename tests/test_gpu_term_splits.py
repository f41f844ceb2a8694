"""The moment kernels at the sizes where their splits and tables end: points
around the 64- and 256-lane groups and the 32-point splits, measurement counts
around 8 (the least of a measurement split), 64 and 256, and more than 256
frequencies (two table blocks), one- and two-antenna paths, against the float64
oracle.

Tolerances (RMS relative): the series is cut at 1e-6 of the sum of the term
magnitudes, the phases are rounded to FP32 after their FP64 reduction (4e-7 rad
rms) and sums of some thousand FP32 terms round at 2^-24 sqrt(n) = 4e-6: 1e-5
for sums, and 5e-5 for the adjoints that chain two of them with cancelling
factors."""
import numpy as np
import pytest
import torch

from gpu_common import Case, as_complex, rel_rms
from oracle import render as orc
from synth import Sphere, freq_grid, line_points, scene_fields

pytestmark = pytest.mark.gpu


def _case(n_meas, n_freq, lines, n_z, bi, seed=0):
    rng = np.random.default_rng(seed)
    f0, df = freq_grid(n_freq)
    tx = np.concatenate([rng.uniform(-0.03, 0.03, (n_meas, 2)), np.zeros((n_meas, 1))], 1).astype(np.float32)
    rx = tx + np.float32([0.01, 0.0, 0.0]) if bi else None
    xyz, _ = line_points((0.0, 0.0, 0.30), 0.10, lines[0], lines[1], n_z)
    sdf, grad, refl = scene_fields(Sphere((0.002, 0.001, 0.30), 0.03, 0.8), xyz)
    return Case(tx, f0, df, n_freq, xyz, sdf, grad, refl, s=64.0, rx=rx)


@pytest.mark.parametrize("n_meas,n_freq,lines,n_z,bi", [
    (1, 25, (1, 1), 31, False), (7, 33, (8, 1), 32, False), (8, 45, (3, 3), 29, True), (9, 64, (5, 5), 41, False),
    (63, 101, (5, 13), 63, True), (65, 257, (4, 4), 65, False), (130, 300, (9, 3), 33, False), (257, 32, (16, 16), 17, False)])
def test_term_sums_at_split_edges(dev, n_meas, n_freq, lines, n_z, bi):
    from paper_2605_29097_amd import rfvr as R
    c = _case(n_meas, n_freq, lines, n_z, bi)
    ap, sm, fl = c.g(dev)
    assert R.term_order(ap, sm.xyz) > 0
    oap, F, x = c.o_ap(), c.o_fields(), c.xyz.astype(np.float64)
    rng = np.random.default_rng(7)
    sig = R.render_forward(ap, sm, fl)
    so = orc.render(oap, x, F)
    assert rel_rms(as_complex(sig), so) < 1e-5
    # the oracle's signal from here on, so that each call is seen by itself
    t = lambda a: torch.from_numpy(np.ascontiguousarray(a, np.float32)).to(dev)
    s32 = np.stack([so.real, so.imag], -1).astype(np.float32)
    s2 = rng.normal(size=s32.shape).astype(np.float32)
    cpx = lambda a: a[..., 0].astype(np.float64) + 1j * a[..., 1]
    z, p, z2, p2 = R.mf_forward(ap, sm.xyz, t(s32), t(s2))
    z1, _ = R.mf_forward(ap, sm.xyz, t(s32))
    zo, po = orc.mf(oap, x.reshape(-1, 3), cpx(s32))
    zo2, po2 = orc.mf(oap, x.reshape(-1, 3), cpx(s2))
    for got, ref in ((z, zo), (z1, zo), (z2, zo2)):
        assert rel_rms(as_complex(got), ref) < 1e-5
    assert rel_rms(p.cpu().numpy(), po) < 1e-5 and rel_rms(p2.cpu().numpy(), po2) < 1e-5
    gp = rng.normal(size=po.shape).astype(np.float32)
    zc = np.stack([zo.real, zo.imag], -1)
    g = R.mf_backward(ap, sm.xyz, t(zc), t(po), t(gp))
    go = orc.mf_adjoint(oap, x.reshape(-1, 3), zo, po, gp.astype(np.float64))
    assert rel_rms(as_complex(g), go) < 1e-5
    gr = R.render_backward(ap, sm, fl, t(s2))
    gro = orc.render_adjoint(oap, x, F, cpx(s2))
    for k in ("sdf", "grad", "refl"):
        assert rel_rms(gr[k].cpu().numpy(), gro[k]) < 5e-5, k
