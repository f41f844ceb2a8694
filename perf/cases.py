"""Performance cases of librfvr: the calls that a reconstruction spends its time in.

Every case is one pass through the public entry points (``rfvr``
and ``autograd``) on inputs that a program has in hand on the GPU.  Five kinds:

``net``       the SDF network: the training pair (forward and backward through a
              reserve), the plain forward, or the plain forward and backward by
              autograd;
``render``    signal tracing forward and its adjoint;
``mf``        the matched filter of one or two signals and its adjoint;
``chain``     render, filter, loss and both adjoints, as one training step calls them
              between the network's forward and backward;
``sampler``   the learned proposal: logits, importance samples, targets, BCE and
              the proposal's gradient.

A step's network and chain are separate cases: opacities are differences of
neighbouring samples' distances and the filter's sums all but cancel, so a
last-bit change of the network is seen a thousand times larger in a whole
step's gradient.

``listed()`` names the sizes that matter, ``draw()`` gives more of the same
ranges, ``exact()`` is the 64-bit value of every output in plain torch.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2605_29097_amd import rfvr as R
from paper_2605_29097_amd.autograd import MLPFn

C = 299792458.0
F_LO, F_HI = 77e9, 81e9
PITCH = 2e-3
CENTRE = (0.0, 0.0, 0.30)
PRECISIONS = {"fp32": R.PREC_FP32, "bf16": R.PREC_BF16, "bf16x3": R.PREC_BF16X3, "f16": R.PREC_F16}
FLAGS = {"clamp": R.SPEC_CLAMP, "raw": R.SPEC_RAW, "off": R.SPEC_OFF}

# the network of the 2^20-point workload, and that of the published configuration
NET = dict(layers=8, width=256, octaves=6, head_width=64, head_layers=2)
PAPER_NET = dict(layers=8, width=256, octaves=10, head_width=256, head_layers=4)


def listed():
    return [
        # the small parity scene (8x8 aperture, 32 frequencies, 16^3 points): launches and latency
        dict(name="chain_small", kind="chain", ax=8, ay=8, freqs=32, lx=16, ly=16, nz=16, side=0.10, spec="clamp",
             bistatic=False, segment=False, shift=False),
        # odd sizes, separate receivers, raw specular factor, lensless shift and ray weights on
        dict(name="chain_bistatic_ragged", kind="chain", ax=21, ay=17, freqs=101, lx=37, ly=29, nz=70, side=0.16,
             spec="raw", bistatic=True, segment=False, shift=True),
        # the published configuration: 1024 rays x 32 depths, 3200 antennas, 64 frequencies
        dict(name="chain_published", kind="chain", ax=64, ay=50, freqs=64, lx=32, ly=32, nz=32, side=0.20, spec="clamp",
             bistatic=False, segment=False, shift=False),
        # the 2^20-point step's signal tracing, forward and adjoint
        dict(name="render_full", kind="render", ax=32, ay=32, freqs=128, lx=64, ly=64, nz=256, side=0.20,
             spec="clamp", bistatic=False, segment=False, shift=True),
        # the 2^20-point step's filter, forward and adjoint
        dict(name="mf_full", kind="mf", ax=32, ay=32, freqs=128, lx=64, ly=64, nz=256, side=0.20, two=False,
             bistatic=False),
        # one scene of the eight-scene workload: importance samples weighted by segments, 45x45 aperture, 256 frequencies
        dict(name="render_scene_segment", kind="render", ax=45, ay=45, freqs=256, lx=128, ly=128, nz=64, side=0.25,
             spec="clamp", bistatic=False, segment=True, shift=False),
        # Phi at the 4096 ray origins and 1024 antennas: the small plain forward of every step
        dict(name="net_origins", kind="net", mode="forward", points=5120, precision="fp32", **NET),
        # the published configuration's network (10 octaves, 4x256 head) at its 32768 samples, training pair
        dict(name="net_pair_published", kind="net", mode="pair", points=32768, precision="fp32", **PAPER_NET),
        # the 2^20-point step's network, training pair, FP32
        dict(name="net_pair_full", kind="net", mode="pair", points=1 << 20, precision="fp32", **NET),
        # the same in the FP16 form
        dict(name="net_pair_full_f16", kind="net", mode="pair", points=1 << 20, precision="f16", **NET),
        # autograd's plain forward and backward, split BF16, an odd count
        dict(name="net_autograd_bf16x3", kind="net", mode="autograd", points=150001, precision="bf16x3", **NET),
        # the proposal sampler of 64x64 rays: 64 bins, 16 + 4 depths
        dict(name="sampler_torus", kind="sampler", lx=64, ly=64, bins=64, imp=16, uni=4, octaves=4, layers=2),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["net", "net", "render", "mf", "chain", "sampler"])
    if kind == "net":
        mode = rng.choice(["pair", "pair", "forward", "autograd"])
        width = rng.choice([128, 192, 256, 256])
        return dict(kind="net", mode=mode, points=_log(rng, 3000, 600000), precision=rng.choice(sorted(PRECISIONS)),
                    layers=rng.randint(3, 8), width=width, octaves=rng.randint(2, 10), head_width=rng.choice([64, 128]),
                    head_layers=rng.randint(1, 3))
    if kind == "sampler":
        return dict(kind="sampler", lx=rng.randint(16, 128), ly=rng.randint(16, 96), bins=rng.randint(16, 64),
                    imp=rng.randint(8, 48), uni=rng.randint(4, 16), octaves=rng.randint(2, 5), layers=rng.randint(1, 3))
    geo = dict(kind=kind, ax=rng.randint(6, 40), ay=rng.randint(5, 32), freqs=rng.randint(32, 200),
               lx=rng.randint(12, 64), ly=rng.randint(12, 64), nz=_log(rng, 16, 256),
               side=round(rng.uniform(0.08, 0.25), 3), bistatic=rng.random() < 0.3)
    if kind == "mf":
        return dict(geo, two=rng.random() < 0.5)
    return dict(geo, spec=rng.choice(sorted(FLAGS)), segment=not geo["bistatic"] and rng.random() < 0.4,
                shift=rng.random() < 0.5)


# ----------------------------------------------------------------------------
# inputs
# ----------------------------------------------------------------------------
def _gen(seed):
    return torch.Generator(device="cuda").manual_seed(int(seed))


def _rand(g, *shape, lo=0.0, hi=1.0):
    return lo + (hi - lo) * torch.rand(*shape, generator=g, device="cuda", dtype=torch.float32)


def _randn(g, *shape):
    return torch.randn(*shape, generator=g, device="cuda", dtype=torch.float32)


def _aperture(case, g):
    """Planar aperture in z = 0 with antennas off the grid by up to 0.1 mm; receivers 5 mm beside."""
    nx, ny = case["ax"], case["ay"]
    ix = (torch.arange(nx, device="cuda", dtype=torch.float32) - (nx - 1) / 2) * PITCH
    iy = (torch.arange(ny, device="cuda", dtype=torch.float32) - (ny - 1) / 2) * PITCH
    yy, xx = torch.meshgrid(iy, ix, indexing="ij")
    tx = torch.stack([xx.reshape(-1), yy.reshape(-1), torch.zeros(nx * ny, device="cuda")], 1)
    tx = tx + _rand(g, nx * ny, 3, lo=-1e-4, hi=1e-4)
    rx = None
    if case.get("bistatic"):
        rx = (tx + torch.tensor([5e-3, 0.0, 0.0], device="cuda")).contiguous()
    nf = case["freqs"]
    return R.Aperture(tx=tx.contiguous(), f0=F_LO, df=(F_HI - F_LO) / (nf - 1), n_freq=nf, rx=rx)


def _points(case):
    xyz, _, _ = R.sample_points(CENTRE, case["side"] / 2, (0.0, 0.0, 1.0), case["lx"], case["ly"], case["nz"])
    return xyz


def _object(case, g, xyz):
    """Signed distance, gradient and reflectiveness of a box of seeded size, place and turn, slightly disturbed."""
    half = case["side"] * _rand(g, 3, lo=0.12, hi=0.25)
    c = torch.tensor(CENTRE, device="cuda") + case["side"] * _rand(g, 3, lo=-0.05, hi=0.05)
    t = float(_rand(g, 1, lo=0.0, hi=0.6))
    rot = torch.tensor([[math.cos(t), 0.0, -math.sin(t)], [0.0, 1.0, 0.0], [math.sin(t), 0.0, math.cos(t)]], device="cuda")
    q = (xyz - c) @ rot.T
    d = q.abs() - half
    out = d.clamp(min=0.0)
    far = out.norm(dim=-1)
    face = torch.nn.functional.one_hot(d.argmax(-1), 3).float()
    n = torch.where(far[..., None] > 1e-9, out / far.clamp(min=1e-9)[..., None], face) * torch.where(q < 0, -1.0, 1.0)
    sdf = far + d.amax(-1).clamp(max=0.0)
    grad = n @ rot + 0.05 * _randn(g, *xyz.shape)
    return sdf.contiguous(), grad.contiguous(), _rand(g, *sdf.shape, lo=0.5, hi=0.9)


def _scene(case, seed):
    g = _gen(seed)
    ap = _aperture(case, g)
    xyz = _points(case)
    sdf, grad, refl = _object(case, g, xyz)
    phi = [None, None, None]
    w = None
    if case["shift"]:
        phi[0] = _rand(g, xyz.shape[0], lo=0.97, hi=1.0)
        phi[1] = _rand(g, ap.n_meas, lo=0.97, hi=1.0)
        phi[2] = _rand(g, ap.n_meas, lo=0.97, hi=1.0) if ap.rx is not None else None
        w = _rand(g, xyz.shape[0], lo=0.5, hi=1.5)
    fl = R.Fields(sdf=sdf, grad=grad, refl=refl, s=64.0, amp=1.0, phi_ray=phi[0], phi_tx=phi[1], phi_rx=phi[2])
    flags = FLAGS[case["spec"]] | (R.WEIGHT_SEGMENT if case["segment"] else 0)
    return dict(ap=ap, sm=R.Samples(xyz=xyz, ray_weight=w), fl=fl, flags=flags, g=g)


def _echoes(ap, g, side):
    """The signal of 48 seeded point scatterers in the cube with 10 dB noise, as a radar measures it."""
    p = torch.tensor(CENTRE, device="cuda") + side * _rand(g, 48, 3, lo=-0.4, hi=0.4)
    a = _rand(g, 48, lo=0.3, hi=1.0).double()
    d = (p[None] - ap.tx[:, None]).double().norm(dim=-1)
    d = 2 * d if ap.rx is None else d + (p[None] - ap.rx[:, None]).double().norm(dim=-1)
    f = ap.f0 + ap.df * torch.arange(ap.n_freq, device="cuda", dtype=torch.float64)
    s = torch.zeros(ap.n_meas, ap.n_freq, dtype=torch.complex128, device="cuda")
    for k in range(48):
        turn = (d[:, k, None] * f / C).remainder(1.0)
        s += a[k] * torch.polar(torch.ones_like(turn), -2 * math.pi * turn)
    s = torch.view_as_real(s).float()
    return (s + 0.3 * s.std() * _randn(g, *s.shape)).contiguous()


def _net_params(case, seed):
    """Weights as of a network under way: the geometric start (distance of a sphere) with every weight moved."""
    from synth.mlp_init import MLPSpec, mlp_init, mlp_layout
    spec = MLPSpec(n_layers=case["layers"], width=case["width"], pe_octaves=case["octaves"],
                   head_width=case["head_width"], head_layers=case["head_layers"], centre=CENTRE, half_size=0.10)
    rng = np.random.default_rng(int(seed))
    p = mlp_init(spec, int(seed)).astype(np.float64)
    lay = mlp_layout(spec)
    off, shape = lay["W0"]
    first = np.zeros(shape)
    for k in range(spec.pe_octaves):    # octaves learnt with falling weight
        first[:, 3 + 6 * k:9 + 6 * k] = rng.normal(0.0, 0.02 * 0.5 ** k, (shape[0], 6))
    p[off:off + first.size] += first.ravel()
    p += rng.normal(0.0, 2e-3, p.size)
    return torch.from_numpy(p.astype(np.float32)).cuda(), spec


def _net(case, seed):
    p, spec = _net_params(case, seed)
    return R.MLP(params=p, n_layers=spec.n_layers, width=spec.width, pe_octaves=spec.pe_octaves,
                 head_width=spec.head_width, head_layers=spec.head_layers, beta=100.0, centre=CENTRE, half_size=0.10,
                 precision=PRECISIONS[case["precision"]])


def prepare(case, seed):
    kind = case["kind"]
    if kind == "net":
        g = _gen(seed)
        n = case["points"]
        net = _net(case, seed)
        xyz = torch.tensor(CENTRE, device="cuda") + 0.10 * _rand(g, n, 3, lo=-1.0, hi=1.0)
        if case["mode"] == "forward":
            # ray origins and antennas: the plane z = 0, outside the cube
            xyz = torch.cat([0.10 * _rand(g, n, 2, lo=-1.0, hi=1.0), torch.zeros(n, 1, device="cuda")], 1).contiguous()
        # adjoints as the render returns them: largest near the surface, a mean and as much that differs from point to point
        near = torch.exp(-(((xyz - torch.tensor(CENTRE, device="cuda")).norm(dim=-1) - 0.05) / 0.03) ** 2)
        return dict(net=net, xyz=xyz.contiguous(), gf=1e-2 * near * (1 + _randn(g, n)),
                    gg=1e-3 * near[:, None] * (1 + _randn(g, n, 3)), ga=1e-2 * near * (1 + _randn(g, n)), mode=case["mode"],
                    reserve=R.mlp_reserve(net, n, "cuda") if case["mode"] == "pair" else None)
    if kind == "render":
        s = _scene(case, seed)
        # the measured signal of a loss 1/2 sum |s - s*|^2
        s["target"] = _echoes(s["ap"], s["g"], case["side"])
        return s
    if kind == "mf":
        g = _gen(seed)
        ap = _aperture(case, g)
        xyz = _points(case)
        n = xyz.shape[0] * xyz.shape[1]
        return dict(ap=ap, xyz=xyz, sig=_echoes(ap, g, case["side"]), sig2=_echoes(ap, g, case["side"]) if case["two"] else None,
                    g_p=1e-3 * _randn(g, n))
    if kind == "chain":
        s = _scene(case, seed)
        # the measured heatmap, of the size of the rendered one (an aperture focused on a surface)
        s["p_star"] = 50.0 * _rand(s["g"], s["sm"].xyz.shape[0] * s["sm"].xyz.shape[1])
        return s
    from synth.mlp_init import ProposalSpec, proposal_init
    g = _gen(seed)
    spec = ProposalSpec(case["octaves"], 64, case["layers"], CENTRE, 0.10)
    net = R.Proposal(params=torch.from_numpy(proposal_init(spec, int(seed))).cuda(), pe_octaves=case["octaves"],
                     layers=case["layers"], centre=CENTRE, half_size=0.10)
    bins, _, _ = R.sample_points(CENTRE, 0.10, (0.0, 0.0, 1.0), case["lx"], case["ly"], case["bins"])
    k = case["imp"] + case["uni"]
    # the blend weights of a render at depths drawn before: one opaque surface per ray
    n_ray = case["lx"] * case["ly"]
    u = (0.20 + 0.20 * _rand(g, n_ray, k)).sort(dim=-1).values.contiguous()
    alpha = torch.exp(-((u - _rand(g, n_ray, 1, lo=0.25, hi=0.35)) / 0.01) ** 2) * 0.8
    trans = torch.cumprod(torch.cat([torch.ones(n_ray, 1, device="cuda"), 1 - alpha[:, :-1]], 1), 1)
    return dict(net=net, bins=bins, case=case, u=u, alpha=alpha.contiguous(), trans=trans.contiguous(), seed=int(seed))


# ----------------------------------------------------------------------------
# one pass
# ----------------------------------------------------------------------------
def run(state):
    if "net" in state and "mode" in state:
        net, xyz = state["net"], state["xyz"]
        if state["mode"] == "forward":
            f, g, a = R.mlp_forward(net, xyz)
            return dict(f=f, grad=g, a=a)
        if state["mode"] == "pair":
            f, g, a = R.mlp_forward(net, xyz, reserve=state["reserve"])
            gp = R.mlp_backward(net, xyz, state["gf"], state["gg"], state["ga"], reserve=state["reserve"])
            return dict(f=f, grad=g, a=a, g_params=gp)
        p = net.params.detach().requires_grad_(True)
        f, g, a = MLPFn.apply(p, xyz, net)
        (gp,) = torch.autograd.grad([f, g, a], [p], [state["gf"], state["gg"], state["ga"]])
        return dict(f=f, grad=g, a=a, g_params=gp)
    if "bins" in state:
        c, net = state["case"], state["net"]
        z = R.proposal_forward(net, state["bins"]).view(c["lx"] * c["ly"], c["bins"])
        xyz, u, o = R.sample_importance(CENTRE, 0.10, (0.0, 0.0, 1.0), c["lx"], c["ly"], z, c["imp"], c["uni"],
                                        seed=state["seed"])
        t = R.proposal_targets(state["u"], state["alpha"], state["trans"], 0.20, 0.40, c["bins"])
        loss, g_z = R.bce(z, t)
        gp = R.proposal_backward(net, state["bins"], g_z)
        return dict(logits=z, xyz=xyz, u=u, origins=o, targets=t, loss=loss, g_params=gp)
    ap = state["ap"]
    if "target" in state:
        sig, alpha, trans = R.render_forward(ap, state["sm"], state["fl"], flags=state["flags"], want_alpha=True)
        gr = R.render_backward(ap, state["sm"], state["fl"], sig - state["target"], flags=state["flags"])
        return dict(signal=sig, alpha=alpha, trans=trans, **_used(gr))
    if "g_p" in state:
        out = R.mf_forward(ap, state["xyz"], state["sig"], state["sig2"])
        g = R.mf_backward(ap, state["xyz"], out[0], out[1], state["g_p"])
        return dict(zip(("z", "p", "z2", "p2"), out), g_sig=g)
    sm, fl, flags = state["sm"], state["fl"], state["flags"]
    sig = R.render_forward(ap, sm, fl, flags=flags)
    z, p = R.mf_forward(ap, sm.xyz, sig)
    loss, g_p = R.loss_l2(p, state["p_star"])
    g_sig = R.mf_backward(ap, sm.xyz, z, p, g_p)
    gr = R.render_backward(ap, sm, fl, g_sig, flags=flags)
    return dict(signal=sig, z=z, p=p, loss=loss, g_sig=g_sig, **_used(gr))


def _used(gr):
    """The gradients that a step with a fixed sharpness s uses (the default): fields and amplitude.  The one in s is a
    scalar sum over both sides of the surface that all but cancels."""
    return {"g_" + k: v for k, v in gr.items() if k != "s"}


# ----------------------------------------------------------------------------
# work that a pass cannot do without
# ----------------------------------------------------------------------------
def _net_work(case, n):
    w, in0, hw = case["width"], 3 + 6 * case["octaves"], case["head_width"]
    trunk = w * in0 + (case["layers"] - 1) * w * w + w
    head = hw * w + (case["head_layers"] - 1) * hw * hw + hw
    params = trunk + head + case["layers"] * w + case["head_layers"] * hw + 2
    fwd = 2.0 * n * (2 * trunk + head)                   # the value, and grad_x f by one sweep
    # parameter gradient: tangent and adjoint chains and two weight products per trunk layer, the head's pair
    bwd = 2.0 * n * (4 * trunk + 2 * head)
    return fwd, bwd, params


def _term_work(case, n, passes):
    """Signal-side and point-side arrays once; per (point, measurement) pair a range, a phase and a complex product."""
    m = case["ax"] * case["ay"]
    pairs = float(n) * m
    return dict(bytes=4.0 * (passes * (2 * m * case["freqs"]) + 3 * m) + passes * 32.0 * n, flops=passes * 40.0 * pairs)


def work(case):
    kind = case["kind"]
    if kind == "net":
        n = case["points"]
        fwd, bwd, params = _net_work(case, n)
        if case["mode"] == "forward":
            return dict(bytes=4.0 * (params + 8 * n), flops=fwd)
        return dict(bytes=4.0 * (2 * params + 16 * n), flops=fwd + bwd)
    if kind == "sampler":
        n_ray = case["lx"] * case["ly"]
        n = n_ray * case["bins"]
        in0 = 3 + 6 * case["octaves"]
        par = 64 * in0 + (case["layers"] - 1) * 4096 + 64
        k = case["imp"] + case["uni"]
        return dict(bytes=4.0 * (3 * n + 4 * n + 4 * n_ray * k + 3 * n_ray * k + 2 * par), flops=2.0 * n * par * 3)
    n = case["lx"] * case["ly"] * case["nz"]
    return _term_work(case, n, 2 if kind in ("render", "mf") else 4)


# ----------------------------------------------------------------------------
# 64-bit values, plain torch
# ----------------------------------------------------------------------------
def _path(tx, rx, m, x):
    """Of measurements m and points x: ranges to transmitter and receiver, vectors along the path, the mean range."""
    d = x[None] - tx[m, None]
    rt = d.norm(dim=-1)
    if rx is None:
        return rt, rt, d, -d, rt
    e = rx[m, None] - x[None]
    rr = e.norm(dim=-1)
    return rt, rr, d, e, 0.5 * (rt + rr)


def _wave(r, f, sign):
    t = (r * (2.0 * f / C)).remainder(1.0)
    return torch.polar(torch.ones_like(t), sign * 2 * math.pi * t)


def _over_points(c, r, ap):
    """sum_j c_ij exp(-j 2 pi f_n 2 r_ij / c) for every n."""
    p, w = c * _wave(r, ap.f0, -1.0), _wave(r, ap.df, -1.0)
    out = []
    for _ in range(ap.n_freq):
        out.append(p.sum(-1))
        p.mul_(w)
    return torch.stack(out, -1)


def _over_freqs(g, r, ap):
    """sum_n g_in exp(+j 2 pi f_n 2 r_ij / c) for every j, by Horner's rule."""
    w = _wave(r, ap.df, 1.0)
    s = torch.zeros_like(w)
    for n in range(ap.n_freq - 1, -1, -1):
        s.mul_(w).add_(g[:, n, None])
    return s.mul_(_wave(r, ap.f0, 1.0))


def _blend(sdf, s, segment):
    """alpha and T of every sample."""
    p = torch.sigmoid(s * sdf)
    al = ((p[:, :-1] - p[:, 1:]) / (p[:, :-1] + 1e-5)).clamp(0.0, 1.0)
    al = torch.cat([al, torch.zeros_like(al[:, :1])], 1)
    t = torch.cumprod(torch.cat([torch.ones_like(al[:, :1]), 1 - al[:, :-1]], 1), 1)
    return al, t


class _Exact:
    """Render and filter of one scene in 64 bits, a few measurements at a time."""

    def __init__(self, s):
        self.ap = s["ap"]
        self.tx = self.ap.tx.double()
        self.rx = None if self.ap.rx is None else self.ap.rx.double()

    def blocks(self, n):
        step = max(1, (1 << 20) // max(n, 1))
        return [slice(k, k + step) for k in range(0, self.ap.n_meas, step)]

    def render_leaves(self, xyz, w, sdf, grad, refl, amp, sharp, phi, flags):
        """Per-point weight b, transmittance t, normal n and position, as functions of the fields."""
        seg = bool(flags & R.WEIGHT_SEGMENT)
        al, t = _blend(sdf, sharp, seg)
        x = xyz.double()
        b = amp * (1.0 if w is None else w.double()[:, None]) * refl * al
        tp = t
        if seg:
            x = torch.cat([0.5 * (x[:, :-1] + x[:, 1:]), x[:, -1:]], 1)
            b = b * t
            tp = t * (1 - 0.5 * al)
        if phi[0] is not None and phi[1] is not None:
            tp = tp - phi[0].double()[:, None]
        n = grad / grad.norm(dim=-1, keepdim=True).clamp(min=1e-12)
        return al, t, b.reshape(-1), tp.reshape(-1), n.reshape(-1, 3), x.reshape(-1, 3)

    def amplitude(self, m, b, tp, n, x, phi, flags):
        rt, rr, d, e, r = _path(self.tx, self.rx, m, x)
        shift = phi[0] is not None and phi[1] is not None
        tt = (tp + (phi[1][m, None].double() if shift else 0.0)).clamp(0.0, 1.0)
        if flags & R.WEIGHT_SEGMENT:
            tr = 1.0
        elif self.rx is None:
            tr = tt
        else:
            tr = (tp + (phi[2][m, None].double() if shift else 0.0)).clamp(0.0, 1.0)
        spec = 1.0
        if (flags & 3) != R.SPEC_OFF:
            wi, wr = d / rt[..., None], e / rr[..., None]
            spec = (wi * wr).sum(-1) - 2 * (n * wi).sum(-1) * (n * wr).sum(-1)
            if (flags & 3) == R.SPEC_CLAMP:
                spec = spec.clamp(min=0.0)
        return b * tt * tr * spec / (rt * rr), r

    def render(self, leaves, phi, flags):
        _, _, b, tp, n, x = leaves
        with torch.no_grad():
            live = b.nonzero().reshape(-1)      # points without weight add nothing
            b, tp, n, x = b[live], tp[live], n[live], x[live]
            return torch.cat([_over_points(*self.amplitude(m, b, tp, n, x, phi, flags), self.ap) for m in self.blocks(x.shape[0])])

    def render_adjoint(self, leaves, inputs, phi, flags, g_sig):
        """Gradients of Re(sum conj(g) s) with respect to `inputs`, which `leaves` are functions of."""
        _, _, b, tp, n, x = leaves
        mid = [v.detach().requires_grad_(True) for v in (b, tp, n)]
        acc = [torch.zeros_like(v) for v in mid]
        for m in self.blocks(x.shape[0]):
            c, r = self.amplitude(m, *mid, x, phi, flags)
            with torch.no_grad():
                g = _over_freqs(g_sig[m], r, self.ap).real
            for a, v in zip(acc, torch.autograd.grad(c, mid, g, allow_unused=True)):
                if v is not None:
                    a += v
        return torch.autograd.grad([b, tp, n], inputs, acc, allow_unused=True)

    def filter(self, xyz, sig):
        x = xyz.reshape(-1, 3).double()
        z = torch.zeros(x.shape[0], dtype=torch.complex128, device=x.device)
        for m in self.blocks(x.shape[0]):
            z += _over_freqs(sig[m], _path(self.tx, self.rx, m, x)[4], self.ap).sum(0)
        return z

    def filter_adjoint(self, xyz, z, g_p):
        x = xyz.reshape(-1, 3).double()
        p = z.abs()
        c = torch.where(p > 0, g_p * z / p.clamp(min=1e-300), torch.zeros_like(z))
        return torch.cat([_over_points(c, _path(self.tx, self.rx, m, x)[4], self.ap) for m in self.blocks(x.shape[0])])


def _cplx(t):
    return torch.view_as_complex(t.double().contiguous())


def _real(t):
    return torch.view_as_real(t.contiguous())


def _exact_render(s):
    """(_Exact, signal, alpha, trans, adjoint as a function of g_sig) of a scene's state."""
    fl, ex = s["fl"], _Exact(s)
    leaf = lambda t: t.double().requires_grad_(True)
    sdf, grad, refl = leaf(fl.sdf), leaf(fl.grad), leaf(fl.refl)
    amp = torch.tensor([float(fl.amp)], dtype=torch.float64, device="cuda", requires_grad=True)
    phi = (fl.phi_ray, fl.phi_tx, fl.phi_rx)
    lv = ex.render_leaves(s["sm"].xyz, s["sm"].ray_weight, sdf, grad, refl, amp, float(fl.s), phi, s["flags"])
    sig = ex.render(lv, phi, s["flags"])

    def adjoint(g):
        ins = [sdf, grad, refl, amp]
        got = ex.render_adjoint(lv, ins, phi, s["flags"], g)
        return {"g_" + k: torch.zeros_like(t) if v is None else v
                for k, t, v in zip(("sdf", "grad", "refl", "amp"), ins, got)}

    return ex, sig, lv[0].detach(), lv[1].detach(), adjoint


def _net64(p, case, x):
    """(f, a) of the network at x, differentiable."""
    from synth.mlp_init import MLPSpec, mlp_layout
    spec = MLPSpec(n_layers=case["layers"], width=case["width"], pe_octaves=case["octaves"],
                   head_width=case["head_width"], head_layers=case["head_layers"], centre=CENTRE, half_size=0.10)
    P = {k: p[o:o + int(np.prod(sh))].view(*sh) for k, (o, sh) in mlp_layout(spec).items() if not k.startswith("_")}
    half = float(np.float32(0.10))
    xh = (x - torch.tensor([float(np.float32(c)) for c in CENTRE], dtype=torch.float64, device=x.device)) / half
    h = [xh]
    for k in range(case["octaves"]):
        h += [torch.sin(2.0 ** k * math.pi * xh), torch.cos(2.0 ** k * math.pi * xh)]
    h = torch.cat(h, -1)
    for i in range(case["layers"]):
        z = 100.0 * (h @ P["W%d" % i].T + P["b%d" % i])
        h = (z.clamp(min=0.0) + torch.log1p(torch.exp(-z.abs()))) / 100.0
    f = half * (h @ P["w_out"] + P["b_out"])
    for k in range(case["head_layers"]):
        h = torch.relu(h @ P["Wh%d" % k].T + P["bh%d" % k])
    return f, torch.sigmoid(h @ P["wh_out"] + P["bh_out"])


def _exact_net(params, case, xyz, gf=None, gg=None, ga=None, chunk=1 << 15):
    """(f, grad_x f, a) and, with upstream gradients, the parameter gradient."""
    p = params.double().requires_grad_(gf is not None)
    fs, gs, as_, gp = [], [], [], torch.zeros_like(p)
    for k in range(0, xyz.shape[0], chunk):
        x = xyz[k:k + chunk].double().requires_grad_(True)
        f, a = _net64(p, case, x)
        (g,) = torch.autograd.grad(f.sum(), x, create_graph=gf is not None)
        if gf is not None:
            q = slice(k, k + chunk)
            j = (gf[q].double() * f).sum() + (gg[q].double() * g).sum() + (ga[q].double() * a).sum()
            gp += torch.autograd.grad(j, p)[0]
        fs.append(f.detach()), gs.append(g.detach()), as_.append(a.detach())
    return torch.cat(fs), torch.cat(gs), torch.cat(as_), gp.detach()


def _exact_sampler(s):
    c = s["case"]
    n_ray = c["lx"] * c["ly"]
    p = s["net"].params.double().requires_grad_(True)
    half = float(np.float32(0.10))
    x = s["bins"].reshape(-1, 3).double()
    xh = (x - torch.tensor([float(np.float32(v)) for v in CENTRE], dtype=torch.float64, device="cuda")) / half
    h = [xh]
    for k in range(c["octaves"]):
        h += [torch.sin(2.0 ** k * math.pi * xh), torch.cos(2.0 ** k * math.pi * xh)]
    h, o = torch.cat(h, -1), 0
    for i in range(c["layers"]):
        fin = h.shape[1]
        w, o = p[o:o + 64 * fin].view(64, fin), o + 64 * fin
        b, o = p[o:o + 64], o + 64
        h = torch.relu(h @ w.T + b)
    z = h @ p[o:o + 64] + p[o + 64]
    # targets: each depth's weight spread over the bins that its segment overlaps
    lo, hi = float(np.float32(0.20)), float(np.float32(0.40))
    u, w = s["u"].double(), s["alpha"].double() * s["trans"].double()
    edge = lo + (hi - lo) / c["bins"] * torch.arange(c["bins"] + 1, device="cuda", dtype=torch.float64)
    W = torch.zeros(n_ray, c["bins"], dtype=torch.float64, device="cuda")
    for k in range(u.shape[1] - 1):
        a, b = u[:, k, None], u[:, k + 1, None]
        over = (torch.minimum(b, edge[1:]) - torch.maximum(a, edge[:-1])).clamp(min=0.0)
        W += w[:, k, None] * over / (b - a).clamp(min=1e-300)
    at = ((u[:, -1] - lo) / (hi - lo) * c["bins"]).floor().long().clamp(0, c["bins"] - 1)
    W.scatter_add_(1, at[:, None], w[:, -1:])
    t = (W / W.amax(-1, keepdim=True).clamp(min=1e-3)).clamp(max=1.0).reshape(-1)
    loss = torch.nn.functional.binary_cross_entropy_with_logits(z, t)
    (gp,) = torch.autograd.grad(loss, p)
    # the drawn depths follow the 32-bit logits through a sort: no 64-bit value is given for them
    return dict(logits=z.detach().view(n_ray, c["bins"]), xyz=None, u=None, origins=None, targets=t.view(n_ray, c["bins"]),
                loss=loss.detach().reshape(1), g_params=gp)


def exact(case, seed):
    kind = case["kind"]
    if kind in ("render", "mf", "chain") and case["ax"] * case["ay"] * case["lx"] * case["ly"] * case["nz"] > 2.2e9:
        return None
    s = prepare(case, seed)
    if kind == "net":
        full = case["mode"] != "forward"
        f, g, a, gp = _exact_net(s["net"].params, case, s["xyz"], *((s["gf"], s["gg"], s["ga"]) if full else ()))
        return dict(f=f, grad=g, a=a, **(dict(g_params=gp) if full else {}))
    if kind == "sampler":
        return _exact_sampler(s)
    if kind == "render":
        _, sig, al, t, adjoint = _exact_render(s)
        return dict(signal=_real(sig), alpha=al, trans=t, **adjoint(sig - _cplx(s["target"])))
    if kind == "mf":
        ex = _Exact(s)
        out = {}
        for k in ("", "2") if case["two"] else ("",):
            z = ex.filter(s["xyz"], _cplx(s["sig" + k]))
            out.update({"z" + k: _real(z), "p" + k: z.abs()})
        return dict(out, g_sig=_real(ex.filter_adjoint(s["xyz"], _cplx(out["z"]), s["g_p"].double())))
    ex, sig, _, _, adjoint = _exact_render(s)
    z = ex.filter(s["sm"].xyz, sig)
    d = z.abs() - s["p_star"].double()
    g_sig = ex.filter_adjoint(s["sm"].xyz, z, 2 * d / d.numel())
    return dict(signal=_real(sig), z=_real(z), p=z.abs(), loss=(d * d).mean().reshape(1), g_sig=_real(g_sig), **adjoint(g_sig))
