"""The FP32 network's arithmetic, apart from the tests that bound its error as a whole.

Values: every layer's products are chains of FP32 fused multiply-adds in the order
that the FP32 matrix instruction takes them, bit for bit.  The signs of the head's
pre-activations are its ReLU masks; another rounding of the values flips some of
them, and each flip shows in the parameter gradient whatever its own products are
worth."""
import numpy as np
import pytest
import torch

from synth import MLPSpec, mlp_init, mlp_layout

pytestmark = pytest.mark.gpu


def _inputs(spec, n, seed):
    rng = np.random.default_rng(seed)
    p = (mlp_init(spec, seed) + rng.normal(0, 2e-3, mlp_init(spec, seed).shape)).astype(np.float32)
    x = (np.array(spec.centre) + spec.half_size * rng.uniform(-1, 1, (n, 3))).astype(np.float32)
    return p, x


def _net(spec, p, beta=100.0):
    from paper_2605_29097_amd import rfvr as R
    return R.MLP(params=torch.from_numpy(p).cuda(), n_layers=spec.n_layers, width=spec.width, pe_octaves=spec.pe_octaves,
                 head_width=spec.head_width, head_layers=spec.head_layers, beta=beta, centre=spec.centre,
                 half_size=spec.half_size)


def _reserve_arrays(res, spec, n):
    """Views of the reserve: H per layer, S per layer, the head's outputs before the relu."""
    up = lambda b: (b + 255) // 256 * 256
    a, h = up(4 * n * spec.width), up(4 * n * spec.head_width)
    res = res.view(torch.uint8)
    take = lambda o, w: res[o:o + 4 * n * w].view(torch.float32).view(n, w)
    L = spec.n_layers
    return ([take(i * a, spec.width) for i in range(L)], [take((L + i) * a, spec.width) for i in range(L)],
            [take(2 * L * a + k * h, spec.head_width) for k in range(spec.head_layers)])


def _matrices(p, spec):
    return {k: p[o:o + int(np.prod(sh))].reshape(sh) for k, (o, sh) in mlp_layout(spec).items() if not k.startswith("_")}


def _chain(h, w, b):
    """h w^T + b by FP32 fused multiply-adds: 16 k at a time, in them k = 4 g + s with s outer and g inner.  A product of
    two FP32 numbers is exact in float64, whose sum is within 2^-53 of the one that is rounded to FP32."""
    acc = np.zeros((h.shape[0], w.shape[0]))
    for k in [kk + 4 * g + s for kk in range(0, h.shape[1], 16) for s in range(4) for g in range(4)]:
        acc = (h[:, k, None].astype(np.float64) * w[None, :, k] + acc).astype(np.float32).astype(np.float64)
    return acc.astype(np.float32) + b


@pytest.mark.parametrize("n,width,head,layers", [(65, 64, 64, 2), (129, 192, 128, 3), (4133, 256, 64, 2),
                                                 (24001, 256, 192, 2), (49157, 128, 64, 1), (70001, 256, 192, 2)])
def test_values_are_fp32_multiply_add_chains(n, width, head, layers):
    """With a softplus so sharp that it is a relu beyond |z| = 2e-4, H shows the trunk's pre-activations too.  Sizes on
    both sides of the rule for 64- and 128-point tiles; the first and the last rows are compared."""
    from paper_2605_29097_amd import rfvr as R
    spec = MLPSpec(n_layers=3, width=width, pe_octaves=4, head_width=head, head_layers=layers)
    p, x = _inputs(spec, n, 5)
    net, xt = _net(spec, p, beta=1e6), torch.from_numpy(x).cuda()
    res = R.mlp_reserve(net, n, "cuda")
    R.mlp_forward(net, xt, reserve=res)
    H, _, Y = _reserve_arrays(res, spec, n)
    rows = torch.from_numpy(np.unique(np.r_[0:32, n - 32:n].clip(0, n - 1))).cuda()
    H, Y = [[a[rows].cpu().numpy() for a in v] for v in (H, Y)]
    P = _matrices(p, spec)
    for i in range(1, spec.n_layers):
        z = _chain(H[i - 1], P[f"W{i}"], P[f"b{i}"])
        far = np.abs(z) > 2e-4
        assert far.mean() > 0.9 and np.array_equal(H[i][far], np.maximum(z, 0)[far]), i
    for k in range(layers):
        assert np.array_equal(Y[k], _chain(np.maximum(Y[k - 1], 0) if k else H[-1], P[f"Wh{k}"], P[f"bh{k}"])), k


def _grad64(p, spec, x, up, masks):
    """Parameter gradient of sum(g_f f + g_grad . grad_x f + g_a a) in float64 with the head's relu masks given, at the
    normalised points that the FP32 encoding starts from (their rounding is no product's)."""
    P64 = torch.from_numpy(p).cuda().double().requires_grad_(True)
    P = {k: P64[o:o + int(np.prod(sh))].view(*sh) for k, (o, sh) in mlp_layout(spec).items() if not k.startswith("_")}
    half = float(np.float32(spec.half_size))
    xn = (x - torch.tensor(spec.centre, dtype=torch.float32, device="cuda")) * float(np.float32(1.0) / np.float32(half))
    total = torch.zeros_like(P64)
    for q in torch.arange(x.shape[0], device="cuda").split(1 << 13):
        xh = xn[q].double().requires_grad_(True)
        h = [xh]
        for k in range(spec.pe_octaves):
            h += [torch.sin(2.0 ** k * np.pi * xh), torch.cos(2.0 ** k * np.pi * xh)]
        h = torch.cat(h, -1)
        for i in range(spec.n_layers):
            h = torch.nn.functional.softplus(h @ P[f"W{i}"].T + P[f"b{i}"], beta=100.0, threshold=1e9)
        f = half * (h @ P["w_out"] + P["b_out"])
        for k in range(spec.head_layers):
            h = (h @ P[f"Wh{k}"].T + P[f"bh{k}"]) * masks[k][q]
        a = torch.sigmoid(h @ P["wh_out"] + P["bh_out"])
        g = torch.autograd.grad(f.sum(), xh, create_graph=True)[0] / half
        total += torch.autograd.grad((up[0][q] * f).sum() + (up[1][q] * g).sum() + (up[2][q] * a).sum(), P64)[0]
    return total


# sizes by the tiles that the products take: 64 x 64; 128 x 128 with all output tiles at a time (up to 512
# work-groups) or in halves; a ragged last tile everywhere, a partial second column block at width 192.  No fewer
# points: the activations' own rounding (1e-7 of softplus', point by point) averages out over many
SIZES = [(23003, 256, 64, 2), (24001, 256, 192, 2), (32700, 256, 64, 1), (40001, 192, 128, 3), (65613, 256, 64, 2)]


@pytest.mark.parametrize("n,width,head,layers", SIZES)
@pytest.mark.parametrize("precision,tol", [("fp32", 4 * 2.0 ** -24), ("bf16x3", 4 * 2.0 ** -16)])
@pytest.mark.parametrize("pair", [True, False])
def test_gradient_apart_from_mask_changes(n, width, head, layers, precision, tol, pair):
    """The products of the parameter gradient, on adjoints as a render returns them: largest near a surface, a mean and as
    much that differs from point to point.  Tolerance: every entry above the first layer's weights sums products of an
    adjoint and an activation, and of an adjoint and a tangent; each factor and the sum are good to a rounding of the
    operands' form, four of those in all.  A mean error of the products, however
    small, adds up over layers and points and shows here; operands in two parts where FP32 is asked for show tenfold."""
    from paper_2605_29097_amd import rfvr as R
    spec = MLPSpec(n_layers=8, width=width, pe_octaves=6, head_width=head, head_layers=layers)
    p, x = _inputs(spec, n, 11)
    net, xt = _net(spec, p), torch.from_numpy(x).cuda()
    net.precision = R.PREC_FP32 if precision == "fp32" else R.PREC_BF16X3
    g = torch.Generator(device="cuda").manual_seed(12)
    near = torch.exp(-(((xt - torch.tensor(spec.centre, device="cuda")).norm(dim=-1) - 0.05) / 0.03) ** 2)
    up = [1e-2 * near * (1 + torch.randn(n, generator=g, device="cuda")),
          1e-3 * near[:, None] * (1 + torch.randn(n, 3, generator=g, device="cuda")),
          1e-2 * near * (1 + torch.randn(n, generator=g, device="cuda"))]
    res = R.mlp_reserve(net, n, "cuda")
    R.mlp_forward(net, xt, reserve=res)
    masks = [y > 0 for y in _reserve_arrays(res, spec, n)[2]]
    got = R.mlp_backward(net, xt, *up, reserve=res if pair else None).double()
    want = _grad64(p, spec, xt, [u.double() for u in up], masks)
    first = mlp_layout(spec)["W1"][0]
    err = float((got - want)[first:].norm() / want[first:].norm())
    assert err < tol, err
