"""Error of the large reductions over points against 64 bits, beside the tests that
compare their kernels with each other."""
import numpy as np
import pytest
import torch

from synth import freq_grid

pytestmark = pytest.mark.gpu
C = 299792458.0


@pytest.mark.parametrize("n_pts,bi", [(1 << 19, False), ((1 << 19) + 4321, True)])
def test_point_reduction_error(dev, n_pts, bi):
    """The filter adjoint of 1024 measurements over points of a 25 cm cube, random weights.  Tolerance: without cells
    this launch sums splits of 1024 points, and a sum of n random terms in FP32 is off by 2^-24 / sqrt(12) sqrt(n / 2)
    of its size, 3.9e-7; the normalised range, rounded to 2^-25, is multiplied by up to 2 pi 2 GHz 2 h / c = 18 in the
    phases (3e-7), which are rounded to FP32 themselves (1.1e-7).  Together 5.1e-7: cells may not be worse."""
    from paper_2605_29097_amd import rfvr as R
    rng = np.random.default_rng(17)
    f0, df = freq_grid(64)
    tx = np.concatenate([rng.uniform(-0.04, 0.04, (1024, 2)), np.zeros((1024, 1))], 1).astype(np.float32)
    rx = (tx + np.float32([0.01, 0.0, 0.0])) if bi else None
    x = (rng.uniform(-0.125, 0.125, (n_pts, 3)) + [0.0, 0.0, 0.30]).astype(np.float32)
    z = rng.normal(size=(n_pts, 2)).astype(np.float32)
    t = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to(dev)
    ap = R.Aperture(tx=t(tx), f0=f0, df=df, n_freq=64, rx=None if rx is None else t(rx))
    # with power = 1 and g_power = 1 the weights are z itself
    one = torch.ones(n_pts, device=dev)
    got = R.mf_backward(ap, t(x), t(z), one, one)[:8].double()
    w, p = torch.view_as_complex(t(z).double()), t(x).double()
    want = torch.zeros(8, 64, dtype=torch.complex128, device=dev)
    for i in range(8):
        r = (p - t(tx[i]).double()).norm(dim=1)
        r = 2 * r if rx is None else r + (p - t(rx[i]).double()).norm(dim=1)
        for n in range(64):
            turn = (r * ((f0 + n * df) / C)).remainder(1.0)
            want[i, n] = (w * torch.polar(torch.ones_like(turn), -2 * np.pi * turn)).sum()
    want = torch.view_as_real(want)
    err = float((got - want).norm() / want.norm())
    assert err < 5.1e-7, err
