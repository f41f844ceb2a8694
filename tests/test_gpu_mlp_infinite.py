"""Infinities, and numbers that BF16 has no room for, in the FP32 network's split
products: they propagate as in plain FP32, and only where they are met."""
import numpy as np
import pytest
import torch

from synth import MLPSpec, mlp_init, mlp_layout

pytestmark = pytest.mark.gpu


def _net(spec, p, beta):
    from paper_2605_29097_amd import rfvr as R
    return R.MLP(params=torch.from_numpy(p).cuda(), n_layers=spec.n_layers, width=spec.width, pe_octaves=spec.pe_octaves,
                 head_width=spec.head_width, head_layers=spec.head_layers, beta=beta, centre=(0.0, 0.0, 0.0), half_size=1.0)


def _block(spec, name):
    o, sh = mlp_layout(spec)[name]
    return slice(o, o + int(np.prod(sh))), sh


@pytest.mark.parametrize("value", [np.inf, -np.inf, 3.395e38, -3.395e38])
@pytest.mark.parametrize("n,width", [(1, 64), (200, 64), (50001, 256)])
def test_weight_in_the_gradient_sweep(n, width, value):
    """One layer on the bare coordinates: grad_x f = W_0^T (sp'(Z) w_out), whose component 1 meets W_0[5][1]."""
    from paper_2605_29097_amd import rfvr as R
    spec = MLPSpec(n_layers=1, width=width, pe_octaves=0, head_width=64, head_layers=1)
    rng = np.random.default_rng(1)
    p = (mlp_init(spec, 0) + rng.normal(0, 0.1, mlp_init(spec, 0).shape)).astype(np.float32)
    q, sh = _block(spec, "W0")
    W = p[q].reshape(sh)
    W[5, 1] = value
    x = rng.uniform(0.1, 1.0, (n, 3)).astype(np.float32)
    x[:, 1] *= np.sign(value)                    # so that unit 5 is on
    w_out = p[_block(spec, "w_out")[0]]
    w_out[5] = 0.25
    with np.errstate(all="ignore"):
        z = x.astype(np.float64) @ W.T.astype(np.float64) + p[_block(spec, "b0")[0]]
        s = w_out / (1.0 + np.exp(-100.0 * z))
        assert (s[:, 5] == 0.25).all()
        want = np.stack([(s * W[:, d].astype(np.float64)).sum(1) for d in range(3)], 1)
    _, g, _ = R.mlp_forward(_net(spec, p, 100.0), torch.from_numpy(x).cuda())
    g = g.cpu().numpy()
    if np.isinf(value):
        assert (g[:, 1] == value).all()
    else:
        assert np.abs(g[:, 1] / want[:, 1] - 1).max() < 1e-6
    for d in (0, 2):
        # 64 to 256 FP32 terms and the sigmoid's rounding of 1e-7
        assert np.abs(g[:, d] - want[:, d]).max() < 256 * 2.0 ** -23 * np.abs(w_out).max() * np.abs(W[:, d]).max()


@pytest.mark.parametrize("pair", [True, False])
@pytest.mark.parametrize("n,width,head", [(3, 64, 64), (300, 128, 128), (50001, 256, 256)])
def test_upstream_gradient_in_the_head(n, width, head, pair):
    """g_refl infinite at one point.  Only unit 3 of the head's second layer is on, so its first layer's adjoint there is
    the infinity times Wh1[3], for the units that are on, and Wh0's gradient that times positive activations."""
    from paper_2605_29097_amd import rfvr as R
    spec = MLPSpec(n_layers=2, width=width, pe_octaves=2, head_width=head, head_layers=2)
    rng = np.random.default_rng(2)
    p = (mlp_init(spec, 0) + rng.normal(0, 0.02, mlp_init(spec, 0).shape)).astype(np.float32)
    b1 = p[_block(spec, "bh1")[0]]
    b1[:] = -100.0
    b1[3] = 1.0
    wo = p[_block(spec, "wh_out")[0]]
    wo[3] = -0.5
    W1 = p[_block(spec, "Wh1")[0]].reshape(_block(spec, "Wh1")[1])
    W1 *= 0.01                                   # so that unit 3 is on everywhere
    W1[np.abs(W1) < 1e-6] = 1e-6
    net = _net(spec, p, 10.0)                    # a soft softplus: activations above zero
    x = torch.from_numpy(rng.uniform(-1, 1, (n, 3)).astype(np.float32)).cuda()
    ga = torch.from_numpy(rng.normal(size=n).astype(np.float32)).cuda()
    at = n // 2
    keep = torch.arange(n, device="cuda") != at
    res = R.mlp_reserve(net, n, "cuda")
    R.mlp_forward(net, x, reserve=res)
    up = lambda b: (b + 255) // 256 * 256
    y0 = res.view(torch.uint8)[4 * up(4 * n * width):][:4 * n * head].view(torch.float32).view(n, head)
    on = (y0[at] > 0).cpu().numpy()
    assert on.any() and not on.all()
    bad = ga.clone()
    bad[at] = float("inf")
    got = R.mlp_backward(net, x, None, None, bad, reserve=res if pair else None).cpu().numpy()
    q, sh = _block(spec, "Wh0")
    rows = got[q].reshape(sh)
    want = np.where(np.sign(wo[3] * W1[3]) > 0, np.inf, -np.inf)
    assert (rows[on] == want[on, None]).all()
    zero = ga.clone()
    zero[at] = 0.0
    res2 = R.mlp_reserve(net, n, "cuda")
    R.mlp_forward(net, x, reserve=res2)
    ref = R.mlp_backward(net, x, None, None, zero, reserve=res2 if pair else None).cpu().numpy()[q].reshape(sh)
    # the units that are off there: as if the point had no gradient, bit for bit
    assert np.isfinite(ref[~on]).all() and np.array_equal(rows[~on], ref[~on])
