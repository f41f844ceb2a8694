"""The FP32 network products on operands split in three BF16 parts, at the sizes
where their tiles end: point counts around the 64- and 128-point tiles, widths
with full and partial 128-column blocks, encodings padded to 32, 64 and 96.

Tolerances: a product over K terms of FP32 operands, each partial sum rounded to
FP32, is within 2^-24 sqrt(K) of its norm (rounding errors of either sign); 8
layers of K = 256 give 8 e-6 for f and a.  The gradients pass every layer twice
and the encoding multiplies them by up to 2^k pi: 16 times that."""
import numpy as np
import pytest
import torch

from oracle import mlp as omlp
from synth import MLPSpec, mlp_init

TOL_F, TOL_G = 8e-6, 1.3e-4


def rel(x, y):
    x, y = np.asarray(x, np.float64).ravel(), np.asarray(y, np.float64).ravel()
    return float(np.linalg.norm(x - y) / np.linalg.norm(y))


def net(spec, seed=3):
    from paper_2605_29097_amd import rfvr as R
    rng = np.random.default_rng(seed)
    p = mlp_init(spec, seed)
    p = (p + rng.normal(0, 0.01, p.shape)).astype(np.float32)
    m = R.MLP(params=torch.from_numpy(p).cuda(), n_layers=spec.n_layers, width=spec.width, pe_octaves=spec.pe_octaves,
              head_width=spec.head_width, head_layers=spec.head_layers, centre=spec.centre, half_size=spec.half_size)
    return p, m


def inputs(n, seed=4):
    rng = np.random.default_rng(seed)
    x = np.array([0.0, 0.0, 0.3]) + rng.uniform(-0.1, 0.1, (n, 3))
    return [a.astype(np.float32) for a in (x, rng.normal(1, 1, n), rng.normal(0.1, 0.1, (n, 3)), rng.normal(1, 1, n))]


@pytest.mark.gpu
@pytest.mark.parametrize("n,width,octaves,head,layers", [
    (1, 64, 2, 64, 1), (63, 64, 4, 64, 2), (64, 128, 6, 64, 2), (65, 192, 10, 128, 3), (127, 256, 6, 192, 2),
    (128, 256, 0, 64, 1), (129, 256, 12, 256, 4), (1000, 192, 6, 64, 2), (4133, 256, 6, 64, 2)])
@pytest.mark.parametrize("pair", [True, False])
def test_split_products_match_oracle(n, width, octaves, head, layers, pair):
    from paper_2605_29097_amd import rfvr as R
    spec = MLPSpec(n_layers=4, width=width, pe_octaves=octaves, head_width=head, head_layers=layers)
    p, m = net(spec)
    x, gf, gg, ga = inputs(n)
    t = [torch.from_numpy(a).cuda() for a in (x, gf, gg, ga)]
    res = R.mlp_reserve(m, n, "cuda") if pair else None
    f, g, a = R.mlp_forward(m, t[0], reserve=res)
    gp = R.mlp_backward(m, t[0], t[1], t[2], t[3], reserve=res)
    fo, go, ao = omlp.forward(p, spec, x)
    gpo = omlp.backward(p, spec, x, gf, gg, ga)
    # the encoding's own rounding: x_hat carries 2^-24, which octave k multiplies by 2^k pi
    pe = 2.0 ** -24 * np.pi * 2.0 ** octaves
    errs = [rel(f.cpu(), fo), rel(a.cpu(), ao), rel(g.cpu(), go), rel(gp.cpu(), gpo)]
    assert errs[0] < TOL_F + pe and errs[1] < TOL_F + pe and errs[2] < TOL_G + 4 * pe and errs[3] < TOL_G + 4 * pe, errs


@pytest.mark.gpu
def test_split_products_scale_exactly():
    """The parts of an operand scale with it: gradients scaled by a power of two come out scaled bit for bit."""
    from paper_2605_29097_amd import rfvr as R
    spec = MLPSpec()
    _, m = net(spec)
    x, *g = [torch.from_numpy(a).cuda() for a in inputs(700)]
    res = R.mlp_reserve(m, 700, "cuda")
    R.mlp_forward(m, x, reserve=res)
    one = R.mlp_backward(m, x, *g, reserve=res)
    for k in (-40, 30):
        got = R.mlp_backward(m, x, *[v * 2.0 ** k for v in g], reserve=res)
        assert torch.equal(got * 2.0 ** -k, one), k


@pytest.mark.gpu
def test_nan_stays_in_its_row():
    from paper_2605_29097_amd import rfvr as R
    spec = MLPSpec()
    _, m = net(spec)
    x = torch.from_numpy(inputs(300)[0]).cuda()
    want = R.mlp_forward(m, x)
    bad = x.clone()
    bad[77, 1] = float("nan")
    got = R.mlp_forward(m, bad)
    keep = torch.arange(300, device="cuda") != 77
    for w, v in zip(want, got):
        assert torch.equal(w[keep], v[keep])
    # f and grad_x f carry it; the head's relu (fmaxf) does not
    assert bool(torch.isnan(got[0][77])) and bool(torch.isnan(got[1][77]).all())


@pytest.mark.gpu
@pytest.mark.parametrize("n,octaves,layers,shift", [(1, 0, 1, 0), (15, 5, 2, 1), (17, 4, 2, 0), (31, 2, 2, 2), (33, 5, 1, 3),
                                                    (64, 4, 2, 0), (65, 3, 2, 1), (129, 5, 2, 0)])
def test_narrow_products_match_oracle(n, octaves, layers, shift):
    """The proposal network's 64 x 64 and 64 x 32 weight gradients (64 x 64 tiles), encoding and ReLU adjoint around
    their 32- and 64-point chunks and 16-row groups, with parameters at any 4-byte alignment.  Tolerance: three
    passes over at most 64 FP32 terms, and the encoding's rounding as above."""
    from paper_2605_29097_amd import rfvr as R
    from oracle import proposal as op
    from synth import ProposalSpec, proposal_init
    spec = ProposalSpec(pe_octaves=octaves, layers=layers)
    rng = np.random.default_rng(n)
    p = (proposal_init(spec, 3) + 0.1 * rng.normal(size=proposal_init(spec, 3).shape)).astype(np.float32)
    x = (np.array(spec.centre) + rng.uniform(-1.0, 1.0, (n, 3)) * spec.half_size).astype(np.float32)
    g = rng.normal(size=n).astype(np.float32)
    buf = torch.zeros(p.size + 4, device="cuda")
    buf[shift:shift + p.size] = torch.from_numpy(p).cuda()
    m = R.Proposal(params=buf[shift:shift + p.size], pe_octaves=octaves, width=spec.width, layers=layers,
                   centre=spec.centre, half_size=spec.half_size)
    xt, gt = torch.from_numpy(x).cuda(), torch.from_numpy(g).cuda()
    p64 = p.astype(np.float64)
    z = R.proposal_forward(m, xt).cpu()
    gp = R.proposal_backward(m, xt, gt).cpu()
    pe = 2.0 ** -24 * np.pi * 2.0 ** octaves
    errs = [rel(z, op.forward(p64, spec, x.astype(np.float64))),
            rel(gp, op.backward(p64, spec, x.astype(np.float64), g.astype(np.float64)))]
    assert max(errs) < 3 * 2.0 ** -24 * 8 + pe, errs


@pytest.mark.gpu
@pytest.mark.parametrize("n,width,octaves,head,layers", [
    (1, 64, 2, 64, 1), (63, 128, 4, 64, 2), (65, 192, 10, 128, 3), (128, 256, 0, 64, 1), (129, 256, 12, 256, 4), (4133, 256, 6, 64, 2)])
@pytest.mark.parametrize("pair", [True, False])
def test_two_part_products_match_oracle(n, width, octaves, head, layers, pair):
    """BF16X3 on the same tiles: two parts hold 16 bits, so an operand is within 2^-17 and a product of K terms with
    errors of either sign within 2^-16 of its norm; 8 layers give 1.3e-4 for f and a at most, 16 times that for the
    gradients as above."""
    from paper_2605_29097_amd import rfvr as R
    spec = MLPSpec(n_layers=4, width=width, pe_octaves=octaves, head_width=head, head_layers=layers)
    p, m = net(spec)
    m.precision = R.PREC_BF16X3
    x, gf, gg, ga = inputs(n)
    t = [torch.from_numpy(a).cuda() for a in (x, gf, gg, ga)]
    res = R.mlp_reserve(m, n, "cuda") if pair else None
    f, g, a = R.mlp_forward(m, t[0], reserve=res)
    gp = R.mlp_backward(m, t[0], t[1], t[2], t[3], reserve=res)
    fo, go, ao = omlp.forward(p, spec, x)
    gpo = omlp.backward(p, spec, x, gf, gg, ga)
    pe = 2.0 ** -24 * np.pi * 2.0 ** octaves
    errs = [rel(f.cpu(), fo), rel(a.cpu(), ao), rel(g.cpu(), go), rel(gp.cpu(), gpo)]
    assert max(errs[:2]) < 1.3e-4 + pe and max(errs[2:]) < 2e-3 + 4 * pe, errs
