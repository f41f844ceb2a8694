"""Large term calls, which sort their points into cells, against the
per-frequency kernels on the same inputs: points on a regular grid and scattered
ones, a flat and a long box, counts that fill neither a work-group nor a batch of
256 measurements, sizes where only one kind of sum has cells, one and two antenna
paths, segments of lines, one and two signals, accumulation, and a filter whose
workspace leaves no room for the cells.

Tolerances (RMS relative) as where the series meet the float64 oracle: the two
truncations stay below 1.5e-6 of the sum of the term magnitudes, phases are
rounded to FP32 after their FP64 reduction (4e-7 rad rms, on either side) and sums of some
thousand FP32 terms round at 2^-24 sqrt(n) = 4e-6: 1.5e-5 for sums, 5e-5 for the
adjoints, which chain two of them."""
import numpy as np
import pytest
import torch

from synth import freq_grid

pytestmark = pytest.mark.gpu


def _points(rng, kind, n_ray, n_z):
    n = n_ray * n_z
    if kind == "cube":
        x = rng.uniform(-0.1, 0.1, (n, 3))
    elif kind == "flat":
        x = rng.uniform(-0.1, 0.1, (n, 3)) * [1.0, 1.0, 0.0]
    elif kind == "long":
        x = rng.uniform(-0.1, 0.1, (n, 3)) * [1.5, 0.05, 0.02]
    elif kind == "clumped":                      # most cells empty, a few very full
        x = rng.normal(size=(n, 3)) * 0.004 + rng.integers(0, 2, (n, 1)) * 0.15 - 0.075
    else:                                        # lines along z
        u = np.stack(np.meshgrid(np.linspace(-0.1, 0.1, n_ray // 16), np.linspace(-0.1, 0.1, 16), indexing="ij"), -1)
        x = np.concatenate([np.repeat(u.reshape(-1, 1, 2), n_z, 1),
                            np.tile(np.linspace(-0.1, 0.1, n_z)[None, :, None], (n_ray, 1, 1))], 2)
    return (x.reshape(n_ray, n_z, 3) + [0.0, 0.0, 0.30]).astype(np.float32)


@pytest.mark.parametrize("kind,n_ray,n_z,n_meas,n_freq,bi,flags", [
    ("cube", 8200, 64, 512, 64, False, 0), ("lines", 2048, 257, 513, 40, True, 0),
    ("flat", 2057, 255, 515, 45, False, 0x1), ("long", 16385, 32, 700, 101, True, 0x2),
    ("clumped", 2100, 250, 1031, 64, False, 0x2), ("cube", 16384, 64, 257, 33, True, 0),
    ("cube", 1024, 64, 2049, 33, False, 0)])
def test_cells_match_per_frequency(dev, kind, n_ray, n_z, n_meas, n_freq, bi, flags):
    from paper_2605_29097_amd import rfvr as R
    rng = np.random.default_rng(n_ray)
    t = lambda a: torch.from_numpy(np.ascontiguousarray(a, np.float32)).to(dev)
    n = lambda *shape: rng.normal(size=shape)
    f0, df = freq_grid(n_freq)
    tx = np.concatenate([rng.uniform(-0.08, 0.08, (n_meas, 2)), np.zeros((n_meas, 1))], 1)
    ap = R.Aperture(tx=t(tx), f0=f0, df=df, n_freq=n_freq, rx=t(tx + [0.02, 0.01, 0.0]) if bi else None)
    sm = R.Samples(xyz=t(_points(rng, kind, n_ray, n_z)), ray_weight=t(rng.uniform(0.5, 1.5, n_ray)))
    # surfaces halfway along each line, a few samples wide
    sdf = 0.05 * np.linspace(1.0, -1.0, n_z) + 0.002 * n(n_ray, n_z)
    fl = R.Fields(sdf=t(sdf), grad=t(n(n_ray, n_z, 3) + [0.0, 0.0, -2.0]), refl=t(rng.uniform(0.2, 1.0, (n_ray, n_z))),
                  s=64.0, phi_ray=t(n(n_ray)), phi_tx=t(n(n_meas)), phi_rx=t(n(n_meas)) if bi else None)
    rms = lambda a, b: float((a.double() - b.double()).norm() / b.double().norm())
    D = R.TERMS_DIRECT
    order = R.term_order(ap, sm.xyz)
    assert order > 0
    for fw in (flags,) if bi else (flags, flags | R.WEIGHT_SEGMENT):
        sig, ref = R.render_forward(ap, sm, fl, flags=fw), R.render_forward(ap, sm, fl, flags=fw | D)
        assert rms(sig, ref) < 1.5e-5
        assert torch.equal(sig, R.render_forward(ap, sm, fl, flags=fw))
        gs = t(n(n_meas, n_freq, 2))
        g, gd = R.render_backward(ap, sm, fl, gs, flags=fw), R.render_backward(ap, sm, fl, gs, flags=fw | D)
        for k in ("sdf", "grad", "refl"):
            # without the specular factor there is no gradient in the normals
            assert rms(g[k], gd[k]) < 5e-5 if bool(gd[k].any()) else not bool(g[k].any()), k
    s2 = t(n(n_meas, n_freq, 2))
    got, want = R.mf_forward(ap, sm.xyz, ref, s2), R.mf_forward(ap, sm.xyz, ref, s2, flags=D)
    for a, b in zip(got, want):
        assert rms(a, b) < 1.5e-5
    z, p = R.mf_forward(ap, sm.xyz, ref)
    assert rms(z, want[0]) < 1.5e-5 and rms(p, want[1]) < 1.5e-5
    gp = t(n(n_ray * n_z))
    base = t(n(n_meas, n_freq, 2))
    for acc in (0, R.ACCUMULATE):
        a = R.mf_backward(ap, sm.xyz, want[0], want[1], gp, flags=acc, out=base.clone())
        b = R.mf_backward(ap, sm.xyz, want[0], want[1], gp, flags=acc | D, out=base.clone())
        assert rms(a, b) < 1.5e-5


def test_filter_without_room_for_cells(dev):
    """2^23 points and 32 measurements: the static scratch (32 MiB) holds no
    permutation, so that call takes the series over the whole box."""
    from paper_2605_29097_amd import rfvr as R
    g = torch.Generator(device="cpu").manual_seed(3)
    f0, df = freq_grid(64)
    tx = (torch.rand(32, 3, generator=g) - 0.5) * 0.1
    tx[:, 2] = 0.0
    xyz = ((torch.rand(1 << 23, 3, generator=g) - 0.5) * 0.2 + torch.tensor([0.0, 0.0, 0.3])).to(dev)
    ap = R.Aperture(tx=tx.to(dev), f0=f0, df=df, n_freq=64)
    sig = torch.randn(32, 64, 2, generator=g).to(dev)
    full, static, ref = R.mf_forward(ap, xyz, sig), R.mf_forward_static(ap, xyz, sig), R.mf_forward(ap, xyz, sig, flags=R.TERMS_DIRECT)
    for a, b, c in zip(full, static, ref):
        assert float((a.double() - c.double()).norm() / c.double().norm()) < 1.5e-5
        assert float((b.double() - c.double()).norm() / c.double().norm()) < 1.5e-5


def test_cells_with_points_that_are_no_numbers(dev):
    """NaN coordinates leave the other points' results as they are."""
    from paper_2605_29097_amd import rfvr as R
    rng = np.random.default_rng(5)
    f0, df = freq_grid(33)
    t = lambda a: torch.from_numpy(np.ascontiguousarray(a, np.float32)).to(dev)
    ap = R.Aperture(tx=t(np.concatenate([rng.uniform(-0.05, 0.05, (1024, 2)), np.zeros((1024, 1))], 1)), f0=f0, df=df, n_freq=33)
    x = _points(rng, "cube", 530000, 1).reshape(-1, 3)
    sig = t(rng.normal(size=(1024, 33, 2)))
    z, _ = R.mf_forward(ap, t(x), sig)
    bad = x.copy()
    bad[7:-1:4099] = np.nan
    keep = torch.from_numpy(~np.isnan(bad[:, 0])).to(dev)
    zb, _ = R.mf_forward(ap, t(bad), sig)
    assert float((zb[keep].double() - z[keep].double()).norm() / z[keep].double().norm()) < 1.5e-5
    assert bool(torch.isnan(zb[~keep]).all())
