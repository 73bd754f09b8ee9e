"""The workloads this library is timed on.

A case is a dict of plain values; `kind` names the call sequence a program
makes and the other entries are its sizes and options:

  solve    cold start and a fixed budget of iterations of one problem through
           ot_dyn_init + ot_dyn_solve (the refined first iterations and the
           residual checks included): small problems, where launches count;
  step     ten steady iterations (ot_dyn_step) of one plan past its refined
           start: what a long solve spends its time on;
  hue      a batch of 1D periodic hue problems of uneven sizes through
           ot_dyn_batch_solve with balanced steps, and its packed result;
  recolor  a new image: hues, histogram, strict order and one frame;
  frames   the frames of a whole path from a prepared image;
  predict  the learned warm start of a group of pairs: restriction,
           prolongation, network input, network, solver state;
  grad     loss and gradient of the warm-start network on one batch.

listed() holds the sizes of this repository's own configurations (16 x 16 x 3
x 8, 64 x 64 x 3 x 16, the paper's 100 x 100 x 3 x 32, 256 x 256 x 3 x 32, 1024
hue histograms, 3840 x 2160 images, the 64 x 64 network) plus one problem of
odd sides and one larger than the caches; draw() spreads over the ranges
around them.  exact() computes the same in float64 with plain torch.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_1501_04840_amd import otdyn, othue, otnet

DEV = "cuda:0"
WARM_ITERS = 64          # past the refined start of the carried potential
STEP_ITERS = 10
HUE_BINS = (64, 128, 180, 256, 360)
HUE_STEPS = (16, 32)


def listed():
    return [
        # the smallest configuration: every kernel is a few microseconds
        dict(name="solve 16x16x3x8", kind="solve", X=16, Y=16, C=3, P=8, iters=100),
        # one RGB pair of the warm-start size
        dict(name="solve 64x64x3x16", kind="solve", X=64, Y=64, C=3, P=16, iters=200),
        # a data-generation group of them as one batched plan
        dict(name="step 32 of 64x64x3x16", kind="step", X=64, Y=64, C=3, P=16, batch=32, refine=3, perx=False),
        # the paper's image size
        dict(name="step 100x100x3x32", kind="step", X=100, Y=100, C=3, P=32, batch=1, refine=3, perx=False),
        # an image of odd sides (no fast transform length) and odd time steps
        dict(name="step 173x131x3x12", kind="step", X=173, Y=131, C=3, P=12, batch=1, refine=3, perx=False),
        # the throughput configuration
        dict(name="step 256x256x3x32", kind="step", X=256, Y=256, C=3, P=32, batch=1, refine=3, perx=False),
        # larger than any cache
        dict(name="step 512x512x3x32", kind="step", X=512, Y=512, C=3, P=32, batch=1, refine=3, perx=False),
        # the batched hue configuration, its first checks
        dict(name="hue 1024", kind="hue", count=1024, iters=300, chunk=100),
        # a new photograph, one recoloured frame
        dict(name="recolor 3840x2160", kind="recolor", W=3840, H=2160, bins=360),
        # the 33 time levels of a path
        dict(name="frames 33 of 3840x2160", kind="frames", W=3840, H=2160, bins=360, frames=33),
        # the learned warm start of a group of pairs
        dict(name="predict 64", kind="predict", m=64, X=64, Y=64, C=3, P=16, Pc=8),
        # one training batch
        dict(name="grad 32", kind="grad", H=64, W=64, in_ch=195, out_ch=189, base=32, levels=4, batch=32),
    ]


def _log(rng, a, b):
    return int(round(math.exp(rng.uniform(math.log(a), math.log(b)))))


def draw(rng):
    kind = rng.choice(["solve", "step", "step", "step", "hue", "recolor", "frames", "predict", "grad"])
    if kind == "solve":
        return dict(kind=kind, X=_log(rng, 8, 128), Y=_log(rng, 8, 128), C=rng.choice([1, 3]), P=rng.choice([8, 10, 16, 32]),
                    iters=50 * rng.randint(2, 4))
    if kind == "step":
        side = rng.choice(["fast", "odd", "odd"])
        while True:
            if side == "fast":
                X, Y = rng.choice([64, 100, 128, 180, 256, 360]), rng.choice([64, 100, 128, 256])
            else:
                X, Y = _log(rng, 24, 420), _log(rng, 24, 420)
            C, P, batch = rng.choice([1, 3, 3]), rng.choice([8, 12, 16, 20, 32]), rng.choice([1, 1, 4])
            if X * Y * C * P * batch <= 8_000_000:
                return dict(kind=kind, X=X, Y=Y, C=C, P=P, batch=batch, refine=rng.choice([3, 3, 3, 1]),
                            perx=rng.choice([False, False, True]))
    if kind == "hue":
        return dict(kind=kind, count=_log(rng, 4, 900), iters=100 * rng.randint(2, 3), chunk=100)
    if kind == "recolor":
        return dict(kind=kind, W=_log(rng, 300, 3800), H=_log(rng, 200, 2160), bins=_log(rng, 60, 1024))
    if kind == "frames":
        return dict(kind=kind, W=_log(rng, 300, 3800), H=_log(rng, 200, 2160), bins=_log(rng, 60, 1024),
                    frames=rng.choice([1, 9, 17, 33]))
    if kind == "predict":
        return dict(kind=kind, m=_log(rng, 1, 60), X=64, Y=64, C=3, P=16, Pc=8)
    s = rng.choice([32, 48, 64])
    return dict(kind=kind, H=s, W=s, in_ch=rng.choice([6, 99, 195]), out_ch=rng.choice([93, 189]), base=rng.choice([16, 32]),
                levels=rng.choice([3, 4]), batch=_log(rng, 1, 32))


# ---- inputs ---------------------------------------------------------------------

def _gen(seed):
    return torch.Generator(device=DEV).manual_seed(int(seed) * 1_000_003 + 17)


def _smooth(gen, n, Y, X, sigma):
    """n standardised Gaussian random fields [n, Y, X], float64, correlated over sigma pixels."""
    z = torch.randn(n, Y, X, generator=gen, device=DEV, dtype=torch.float64)
    ky = torch.fft.fftfreq(Y, device=DEV, dtype=torch.float64)[:, None]
    kx = torch.fft.rfftfreq(X, device=DEV, dtype=torch.float64)[None, :]
    z = torch.fft.irfft2(torch.fft.rfft2(z) * torch.exp(-2 * (math.pi * sigma) ** 2 * (ky * ky + kx * kx)), s=(Y, X))
    z = z - z.mean(dim=(1, 2), keepdim=True)
    return z / z.std(dim=(1, 2), keepdim=True).clamp_min(1e-12)


def _densities(seed, B, C, Y, X):
    """Two mean-one densities [B, C, Y, X] (float32): exponentiated smooth fields."""
    gen, out = _gen(seed), []
    for _ in range(2):
        d = torch.exp(_smooth(gen, B * C, Y, X, 4.0)).reshape(B, C, Y, X)
        out.append((d / d.mean(dim=(1, 2, 3), keepdim=True)).float())
    return out


def _hue_problems(case, seed):
    """(bins, steps, h0, h1) per problem: von Mises mixtures, mean one."""
    sizes, rng, out = np.random.default_rng(401), np.random.default_rng([seed, 401]), []
    for _ in range(case["count"]):
        n, T, hs = int(sizes.choice(HUE_BINS)), int(sizes.choice(HUE_STEPS)), []
        for _ in range(2):
            k = int(rng.integers(1, 5))
            mu, kappa, w = rng.uniform(0, 1, k), rng.uniform(1, 20, k), rng.dirichlet(np.ones(k))
            th = (np.arange(n) + 0.5) / n
            g = (w[:, None] * np.exp(kappa[:, None] * (np.cos(2 * np.pi * (th[None] - mu[:, None])) - 1))).sum(0)
            g = g / g.max() + 1e-4
            hs.append((g / g.mean()).astype(np.float32))
        out.append((n, T, hs[0], hs[1]))
    return out


def _image(seed, H, W):
    """An 8-bit RGB image [H, W, 3] of smooth channels with a grey corner."""
    z = _smooth(_gen(seed), 3, H, W, 24.0 if min(H, W) > 500 else 6.0)
    lo, hi = z.amin(dim=(1, 2), keepdim=True), z.amax(dim=(1, 2), keepdim=True)
    img = torch.round(255 * (z - lo) / (hi - lo)).to(torch.uint8).permute(1, 2, 0).contiguous()
    img[: H // 8, : W // 8, :] = img[: H // 8, : W // 8, :1]
    return img


def _targets(seed, frames, n):
    """Hue densities along a path [frames, n]: mixtures of two von Mises histograms."""
    rng = np.random.default_rng([seed, 77])
    th = (np.arange(n) + 0.5) / n
    mu, kappa = rng.uniform(0, 1, 2), rng.uniform(1, 20, 2)
    h = np.exp(kappa[:, None] * (np.cos(2 * np.pi * (th[None] - mu[:, None])) - 1)) + 1e-4
    t = np.linspace(0.0, 1.0, frames)[:, None]
    return torch.from_numpy(((1 - t) * h[0] + t * h[1]).astype(np.float32)).to(DEV)


def _desc(case):
    d = otdyn.ot_dyn_default_desc(case["X"], case["Y"], case["C"], case["P"])
    d.batch = case.get("batch", 1)
    d.refine = case.get("refine", otdyn.OT_REFINE_CARRY)
    if case.get("perx"):
        d.bc[0] = otdyn.OT_BC_PERIODIC
    return d


def _net_layers(in_ch, out_ch, base, levels):
    widths, layers, c = [base << l for l in range(levels)], [], in_ch
    for w in widths:
        layers += [(3, c, w), (3, w, w)]
        c = w
    for w in reversed(widths[:-1]):
        layers += [(3, c + w, w), (3, w, w)]
        c = w
    return layers + [(1, c, out_ch)]


def _net_params(seed, layers):
    """He-normal weights and small biases, flat float32 on the GPU."""
    gen, parts = _gen(seed), []
    for k, ci, co in layers:
        parts.append(torch.randn(k * k * ci * co, generator=gen, device=DEV) * math.sqrt(2.0 / (k * k * ci)))
        parts.append(0.02 * torch.randn(co, generator=gen, device=DEV))
    return torch.cat(parts)


def _net(in_ch, out_ch, H, W, base, levels, max_batch, params):
    d = otnet.ot_net_default_desc(H, W, in_ch, out_ch, max_batch)
    d.base, d.levels = base, levels
    net = otnet.Net(d, DEV)
    net.set_params(params)
    return net


def _coarse(case, seed):
    """A coarse solver state (F [m, Pc+1, C, Y/2, X/2], M [3, m, Pc, ...]) near a linear path."""
    m, C, Y, X, Pc = case["m"], case["C"], case["Y"] // 2, case["X"] // 2, case["Pc"]
    f0, f1 = _densities(seed, m, C, Y, X)
    t = (torch.arange(Pc + 1, device=DEV) / Pc).reshape(1, Pc + 1, 1, 1, 1)
    F = ((1 - t) * f0[:, None] + t * f1[:, None]).contiguous()
    M = 0.1 * _smooth(_gen(seed + 5), 3 * m * Pc * C, Y, X, 2.0).float().reshape(3, m, Pc, C, Y, X)
    M[0, ..., 0] = 0
    M[1, ..., 0, :] = 0
    return F, M.contiguous()


def _grad_batch(case, seed):
    gen = _gen(seed)
    b, H, W = case["batch"], case["H"], case["W"]
    x = torch.randn(b, H, W, case["in_ch"], generator=gen, device=DEV)
    t = torch.randn(b, H, W, case["out_ch"], generator=gen, device=DEV)
    cw = torch.rand(case["out_ch"], generator=gen, device=DEV) / case["out_ch"]
    return x, t, cw


def prepare(case, seed):
    kind = case["kind"]
    if kind in ("solve", "step"):
        d = _desc(case)
        prob = otdyn.Problem(d, DEV)
        prob.set_boundary(*_densities(seed, d.batch, d.C, d.Y, d.X))
        prob.init(otdyn.OT_INIT_COLD)
        if kind == "step":
            prob.step(WARM_ITERS)
        return dict(case=case, prob=prob)
    if kind == "hue":
        probs = _hue_problems(case, seed)
        base = otdyn.ot_dyn_default_desc(1, 1, 1, 2)
        base.bc[0] = otdyn.OT_BC_PERIODIC
        base.tau, base.sigma, base.adapt = 3.0, 0.33, 1
        bt = otdyn.Batch(base, [(n, 1, 1, T) for n, T, _, _ in probs], DEV)
        bt.set_boundary([p[2] for p in probs], [p[3] for p in probs])
        return dict(case=case, bt=bt)
    if kind in ("recolor", "frames"):
        frames = case.get("frames", 1)
        r = othue.HueRenderer(case["W"] * case["H"], case["bins"], DEV, max_frames=frames)
        img = _image(seed, case["H"], case["W"])
        if kind == "frames":
            r.set_source(img)
        return dict(case=case, r=r, img=img, targets=_targets(seed, frames, case["bins"]))
    if kind == "predict":
        f0, f1 = _densities(seed, case["m"], case["C"], case["Y"], case["X"])
        Fc, Mc = _coarse(case, seed)
        out_ch = otnet.warm_channels(case["C"], case["P"])
        in_ch = 2 * case["C"] + out_ch
        params = _net_params(seed, _net_layers(in_ch, out_ch, 32, 4))
        return dict(case=case, f0=f0, f1=f1, Fc=Fc, Mc=Mc, in_ch=in_ch, out_ch=out_ch,
                    net=_net(in_ch, out_ch, case["Y"], case["X"], 32, 4, 32, params))
    x, t, cw = _grad_batch(case, seed)
    layers = _net_layers(case["in_ch"], case["out_ch"], case["base"], case["levels"])
    net = _net(case["in_ch"], case["out_ch"], case["H"], case["W"], case["base"], case["levels"], case["batch"], _net_params(seed, layers))
    return dict(case=case, net=net, x=x, t=t, cw=cw)


def run(state):
    case = state["case"]
    kind = case["kind"]
    if kind == "solve":
        prob = state["prob"]
        prob.init(otdyn.OT_INIT_COLD)
        prob.solve(case["iters"])
        return dict(zip(("F", "Mx", "My", "Mc"), prob.state()))
    if kind == "step":
        state["prob"].step(STEP_ITERS)
        return dict(zip(("F", "Mx", "My", "Mc"), state["prob"].state()))
    if kind == "hue":
        state["bt"].solve(case["iters"], case["chunk"])
        F, M = state["bt"].packed_state()
        return dict(F=F, M=M)
    if kind == "recolor":
        r = state["r"]
        r.set_source(state["img"])
        counts, density = r.histogram()
        return dict(counts=counts, density=density, frame=r.render_frames(state["targets"]))
    if kind == "frames":
        return state["r"].render_frames(state["targets"])
    if kind == "predict":
        return _predict(state)
    loss, grad = state["net"].grad(state["x"], state["t"], state["cw"])
    return dict(loss=loss, grad=grad)


def _predict(s):
    """The warm-start state of a group: as warmstart.evaluate sequences it, the coarse solve given."""
    case = s["case"]
    m, X, Y, C, P, Pc = (case[k] for k in ("m", "X", "Y", "C", "P", "Pc"))
    df, dc = otdyn.ot_dyn_default_desc(X, Y, C, P), otdyn.ot_dyn_default_desc(X // 2, Y // 2, C, Pc)
    stream = torch.cuda.current_stream().cuda_stream
    sl, slc = X * Y * C, X * Y * C // 4
    f32 = dict(dtype=torch.float32, device=DEV)
    c0, c1 = torch.empty(m, C, Y // 2, X // 2, **f32), torch.empty(m, C, Y // 2, X // 2, **f32)
    otnet.ot_warm_restrict(df, m, s["f0"], c0, stream)
    otnet.ot_warm_restrict(df, m, s["f1"], c1, stream)
    Fp, Mp = torch.zeros(m, P + 1, C, Y, X, **f32), torch.zeros(3, m, P, C, Y, X, **f32)
    otnet.ot_warm_prolong(dc, df, m, s["Fc"], (Pc + 1) * slc, s["Mc"][0], s["Mc"][1], s["Mc"][2], Pc * slc, Fp, (P + 1) * sl,
                          Mp[0], Mp[1], Mp[2], P * sl, stream)
    base = torch.empty(m, Y, X, s["out_ch"], **f32)
    otnet.ot_warm_targets(df, m, s["f0"], s["f1"], Fp, (P + 1) * sl, Mp[0], Mp[1], Mp[2], P * sl, None, base, stream)
    x = torch.empty(m, Y, X, s["in_ch"], **f32)
    otnet.ot_warm_inputs(df, m, s["f0"], s["f1"], base, x, stream)
    y = torch.empty(m, Y, X, s["out_ch"], **f32)
    for b0 in range(0, m, 32):
        n = min(32, m - b0)
        otnet.ot_net_forward(s["net"].net, n, x[b0:b0 + n], y[b0:b0 + n])
    F, M = torch.zeros(m, P + 1, C, Y, X, **f32), torch.zeros(3, m, P, C, Y, X, **f32)
    otnet.ot_warm_state(df, m, s["f0"], s["f1"], y, base, F, (P + 1) * sl, M[0], M[1], M[2], P * sl, stream)
    return dict(c0=c0, c1=c1, y=y, F=F, M=M)


def work(case):
    kind = case["kind"]
    if kind in ("solve", "step", "hue"):
        # per iteration the state (x 4, b 4, b_bar 4 words a node) is read and written once
        if kind == "hue":
            nodes = case["count"] * int(np.mean(HUE_BINS) * np.mean(HUE_STEPS))
            logs = 12
        else:
            nodes = case["X"] * case["Y"] * case["C"] * case["P"] * case.get("batch", 1)
            logs = math.log2(max(2, case["X"] * case["Y"] * case["P"]))
        iters = STEP_ITERS if kind == "step" else case["iters"]
        return dict(bytes=96.0 * nodes * iters, flops=(5 * logs + 150) * nodes * iters)
    if kind in ("recolor", "frames"):
        px, f = case["W"] * case["H"], case.get("frames", 1)
        return dict(bytes=3.0 * px * (1 + f), flops=60.0 * px * f)
    if kind == "predict":
        out_ch = otnet.warm_channels(case["C"], case["P"])
        layers, px, m = _net_layers(2 * case["C"] + out_ch, out_ch, 32, 4), case["X"] * case["Y"], case["m"]
        return dict(bytes=4.0 * m * px * (out_ch + out_ch // 8 + 2 * case["C"]), flops=2.0 * m * _macs(layers, px, 4))
    layers = _net_layers(case["in_ch"], case["out_ch"], case["base"], case["levels"])
    px = case["H"] * case["W"]
    nbytes = 4.0 * case["batch"] * px * (case["in_ch"] + case["out_ch"]) + 8.0 * sum(k * k * a * b + b for k, a, b in layers)
    return dict(bytes=nbytes, flops=6.0 * case["batch"] * _macs(layers, px, case["levels"]))


def _macs(layers, px, levels):
    """Multiply-adds of one image of px pixels."""
    at = [l for l in range(levels) for _ in range(2)] + [l for l in range(levels - 2, -1, -1) for _ in range(2)] + [0]
    return sum(k * k * a * b * (px >> (2 * l)) for (k, a, b), l in zip(layers, at))


# ---- the same in float64 --------------------------------------------------------

def _basis(n, periodic, scale):
    """Orthonormal eigenbasis (rows) and eigenvalues of one axis's Laplacian."""
    j = torch.arange(n, device=DEV, dtype=torch.float64)
    if periodic:
        a = 2 * math.pi * torch.remainder(j[:, None] * j[None], n) / n
        T = (torch.cos(a) + torch.sin(a)) / math.sqrt(n)
        lam = 4 * scale ** 2 * torch.sin(math.pi * j / n) ** 2
    else:
        T = math.sqrt(2.0 / n) * torch.cos(math.pi * j[:, None] * (2 * j[None] + 1) / (2 * n))
        T[0] /= math.sqrt(2.0)
        lam = 4 * scale ** 2 * torch.sin(math.pi * j / (2 * n)) ** 2
    return T, lam


class _Exact:
    """Algorithm 1 in float64 on [B, P, C, Y, X] tensors."""

    def __init__(self, X, Y, C, P, f0, f1, perx, perc, tau_sigma, sigma):
        self.dims = {4: (X, perx and X > 1), 3: (Y, False), 2: (C, perc and C > 1)}
        self.P, self.B = P, f0.shape[0]
        self.ts = tau_sigma
        z = lambda k: torch.zeros(self.B, k, C, Y, X, dtype=torch.float64, device=DEV)  # noqa: E731
        self.F = z(P + 1)
        self.F[:, 0], self.F[:, P] = f0.double(), f1.double()
        self.m = {ax: z(P) for ax in self.dims}
        self.b = [z(P) for _ in range(4)]
        self.bb = [z(P) for _ in range(4)]
        self.sigma = torch.full((self.B, 1, 1, 1, 1), sigma, dtype=torch.float64, device=DEV)
        axes = [(ax, n, per) for ax, (n, per) in self.dims.items()] + [(1, P, False)]
        self.T, self.lam = {}, 0
        for ax, n, per in axes:
            self.T[ax], lam = _basis(n, per, float(n))
            shape = [1] * 5
            shape[ax] = n
            self.lam = self.lam + lam.reshape(shape)

    def _wall(self, v, ax):
        if not self.dims[ax][1]:
            v.select(ax, 0).zero_()
        return v

    def _solve(self, r):
        for ax, T in self.T.items():
            if T.shape[0] > 1:
                r = torch.matmul(r.transpose(ax, 4), T.t()).transpose(ax, 4)
        r = torch.where(self.lam > 1e-12, r / self.lam.clamp_min(1e-12), torch.zeros_like(r))
        for ax, T in self.T.items():
            if T.shape[0] > 1:
                r = torch.matmul(r.transpose(ax, 4), T).transpose(ax, 4)
        return r

    def step(self, resid=False):
        old = None
        if resid:
            old = [self.F.clone()] + [v.clone() for v in self.m.values()]
        for q, (ax, m) in enumerate(self.m.items()):
            m -= self.ts * 0.5 * self._wall(torch.roll(self.bb[q], 1, ax) + self.bb[q], ax)
        self.F[:, 1:-1] -= self.ts * 0.5 * (self.bb[3][:, :-1] + self.bb[3][:, 1:])
        r = self.P * (self.F[:, 1:] - self.F[:, :-1])
        for ax, m in self.m.items():
            r += self.dims[ax][0] * (torch.roll(m, -1, ax) - m)
        phi = self._solve(r)
        for ax, m in self.m.items():
            m += self.dims[ax][0] * self._wall(phi - torch.roll(phi, 1, ax), ax)
        self.F[:, 1:-1] += self.P * (phi[:, 1:] - phi[:, :-1])
        k = [0.5 * (m + torch.roll(m, -1, ax)) for ax, m in self.m.items()] + [0.5 * (self.F[:, 1:] + self.F[:, :-1])]
        a = [k[q] + self.b[q] for q in range(4)]
        s, a2 = self.sigma, a[0] ** 2 + a[1] ** 2 + a[2] ** 2
        on = 2 * a[3] + s * a2 > 0
        v = a[3].clamp_min(0) + 0.5 * s * a2
        for _ in range(50):
            w, d = 1 + s * v, v - a[3]
            g, dg = 2 * w * w * d - s * a2, 4 * s * w * d + 2 * w * w
            n = torch.where(on, v - g / dg, v)
            done = bool(((v - n).abs() <= 1e-13 * v.abs()).all())
            v = torch.where(on & (n < v) & (n > 0), n, v)
            if done:
                break
        v = torch.where(on, v, torch.zeros_like(v))
        f = s * v / (1 + s * v)
        z = [f * a[0], f * a[1], f * a[2], v]
        for q in range(4):
            db = k[q] - z[q]
            self.b[q] += db
            self.bb[q] = self.b[q] + db
        if resid:
            n2 = lambda t: sum((u * u).sum(dim=(1, 2, 3, 4)) for u in t)  # noqa: E731
            new = [self.F] + list(self.m.values())
            dual = torch.sqrt(n2([u[:, 1:-1] if i == 0 else u for i, u in enumerate([p - q for p, q in zip(new, old)])])
                              / n2([u[:, 1:-1] if i == 0 else u for i, u in enumerate(new)]))
            return torch.sqrt(n2([k[q] - z[q] for q in range(4)]) / n2(z)), dual
        return None

    def state(self):
        return dict(F=self.F, Mx=self.m[4], My=self.m[3], Mc=self.m[2])


def _exact_hue(case, seed):
    """Groups of one shape side by side, the balancing of sigma at the checks included."""
    probs = _hue_problems(case, seed)
    F, M = [None] * len(probs), [None] * len(probs)
    for n, T in sorted({(p[0], p[1]) for p in probs}):
        ids = [i for i, p in enumerate(probs) if (p[0], p[1]) == (n, T)]
        h = [torch.from_numpy(np.stack([probs[i][q] for i in ids])).to(DEV).reshape(-1, 1, 1, n) for q in (2, 3)]
        e = _Exact(n, 1, 1, T, h[0], h[1], True, False, 3.0 * 0.33, float(np.float32(0.33)))
        changed = 0
        last = torch.zeros(len(ids), dtype=torch.int64, device=DEV)
        for it in range(1, case["iters"] + 1):
            check = it % case["chunk"] == 0
            res = e.step(check)
            if check and changed < 4:
                prim, dual = res
                free = (it - last >= 200) & (torch.maximum(prim, dual) >= 3e-5)
                f = torch.where(free & (dual > 4 * prim), 2.0, torch.where(free & (prim > 4 * dual), 0.5, 1.0)).double()
                last = torch.where(f != 1, it, last)
                f = f.reshape(-1, 1, 1, 1, 1)
                e.sigma = e.sigma / f
                e.b, e.bb = [u * f for u in e.b], [u * f for u in e.bb]
        for j, i in enumerate(ids):
            F[i] = e.F[j].reshape(-1)
            M[i] = torch.cat([e.m[ax][j].reshape(-1) for ax in (4, 3, 2)])
    return dict(F=torch.cat(F), M=torch.cat(M))


def _conv(x, w, b):
    """3x3 (zero padding) or 1x1 convolution of [B, H, W, ci] by w [k, k, ci, co]."""
    if w.shape[0] == 1:
        return torch.matmul(x, w[0, 0]) + b
    H, W = x.shape[1:3]
    p = torch.nn.functional.pad(x, (0, 0, 1, 1, 1, 1))
    return sum(torch.matmul(p[:, i:i + H, j:j + W], w[i, j]) for i in range(3) for j in range(3)) + b


def _net_exact(x, params, layers, levels):
    ws, o = [], 0
    for k, ci, co in layers:
        n = k * k * ci * co
        ws.append((params[o:o + n].reshape(k, k, ci, co), params[o + n:o + n + co]))
        o += n + co
    it, skips = iter(ws), []
    h = x
    for l in range(levels):
        h = torch.relu(_conv(torch.relu(_conv(h, *next(it))), *next(it)))
        if l + 1 < levels:
            skips.append(h)
            B, H, W, c = h.shape
            h = h.reshape(B, H // 2, 2, W // 2, 2, c).mean(dim=(2, 4))
    for l in range(levels - 2, -1, -1):
        h = torch.cat([h.repeat_interleave(2, 1).repeat_interleave(2, 2), skips[l]], dim=-1)
        h = torch.relu(_conv(torch.relu(_conv(h, *next(it))), *next(it)))
    return _conv(h, *next(it))


def _lerp(nf, nc, pos, faces=False):
    """Matrix [nf, nc] of linear interpolation at positions pos (clamped; faces: zero walls at 0 and nc)."""
    W = np.zeros((nf, nc + 1))
    for i, u in enumerate(pos):
        a = int(math.floor(u))
        for j, w in ((a, 1 - (u - a)), (a + 1, u - a)):
            if faces:
                W[i, j] += w if 0 < j < nc else 0.0
            else:
                W[i, min(max(j, 0), nc - 1)] += w
    return torch.from_numpy(W[:, :nc]).to(DEV)


def _exact_predict(case, seed):
    m, X, Y, C, P, Pc = (case[k] for k in ("m", "X", "Y", "C", "P", "Pc"))
    f0, f1 = (d.double() for d in _densities(seed, m, C, Y, X))
    Fc, Mc = (t.double() for t in _coarse(case, seed))
    half = lambda f: f.reshape(m, C, Y // 2, 2, X // 2, 2).mean(dim=(3, 5))  # noqa: E731
    cx = _lerp(X, X // 2, [0.5 * i - 0.25 for i in range(X)])
    cy = _lerp(Y, Y // 2, [0.5 * i - 0.25 for i in range(Y)])
    fx = _lerp(X, X // 2, [0.5 * i for i in range(X)], True)
    fy = _lerp(Y, Y // 2, [0.5 * i for i in range(Y)], True)
    tf = _lerp(P + 1, Pc + 1, [k * Pc / P for k in range(P + 1)])
    tm = _lerp(P, Pc, [(k + 0.5) * Pc / P - 0.5 for k in range(P)])

    def up(v, Wt, Wy, Wx):      # [m, t, C, y, x]
        v = torch.matmul(v, Wx.t())
        v = torch.matmul(Wy, v)
        return torch.matmul(Wt, v.reshape(m, v.shape[1], -1)).reshape(m, Wt.shape[0], C, Y, X)

    Fp = up(Fc, tf, cy, cx)
    Mp = [up(Mc[0], tm, cy, fx), up(Mc[1], tm, fy, cx), up(Mc[2], tm, cy, cx)]
    Mp[0][..., 0] = 0
    Mp[1][..., 0, :] = 0
    t = (torch.arange(1, P, device=DEV, dtype=torch.float64) / P).reshape(1, P - 1, 1, 1, 1)
    lin = (1 - t) * f0[:, None] + t * f1[:, None]
    chan = lambda v: v.permute(0, 3, 4, 1, 2).reshape(m, Y, X, -1)  # noqa: E731
    base = torch.cat([chan(Fp[:, 1:P] - lin)] + [chan(v) for v in Mp], dim=-1)
    x = torch.cat([f0.permute(0, 2, 3, 1), f1.permute(0, 2, 3, 1), base], dim=-1)
    layers = _net_layers(x.shape[-1], base.shape[-1], 32, 4)
    params = _net_params(seed, layers).double()
    y = torch.cat([_net_exact(x[i:i + 16], params, layers, 4) for i in range(0, m, 16)])
    s = (y + base).reshape(m, Y, X, -1)
    back = lambda v, k: v.reshape(m, Y, X, k, C).permute(0, 3, 4, 1, 2)  # noqa: E731
    F = torch.zeros(m, P + 1, C, Y, X, dtype=torch.float64, device=DEV)
    F[:, 1:P] = lin + back(s[..., :C * (P - 1)], P - 1)
    M, o = [], C * (P - 1)
    for q in range(3):
        M.append(back(s[..., o + q * C * P:o + (q + 1) * C * P], P).clone())
    M[0][..., 0] = 0
    M[1][..., 0, :] = 0
    return dict(c0=half(f0), c1=half(f1), y=y, F=F, M=torch.stack(M))


def exact(case, seed):
    kind = case["kind"]
    if kind in ("solve", "step"):
        d = _desc(case)
        f0, f1 = _densities(seed, d.batch, d.C, d.Y, d.X)
        e = _Exact(d.X, d.Y, d.C, d.P, f0, f1, case.get("perx", False), True, float(np.float32(d.tau * d.sigma)),
                   float(np.float32(d.sigma)))
        for _ in range(case["iters"] if kind == "solve" else WARM_ITERS + STEP_ITERS):
            e.step()
        return e.state()
    if kind == "hue":
        return _exact_hue(case, seed)
    if kind == "predict":
        return _exact_predict(case, seed)
    if kind == "grad":
        x, t, cw = _grad_batch(case, seed)
        layers = _net_layers(case["in_ch"], case["out_ch"], case["base"], case["levels"])
        params = _net_params(seed, layers).double().requires_grad_(True)
        npix, loss = x.shape[0] * x.shape[1] * x.shape[2], 0.0
        for i in range(0, x.shape[0], 8):
            y = _net_exact(x[i:i + 8].double(), params, layers, case["levels"])
            part = (cw.double() * (y - t[i:i + 8].double()) ** 2).sum() / npix
            part.backward()
            loss += float(part)
        return dict(loss=loss, grad=params.grad)
    if kind == "recolor":       # the density of the source; counts and bytes are whole numbers
        rgb = _image(seed, case["H"], case["W"]).reshape(-1, 3).cpu().numpy().astype(np.int32)
        hi, lo = rgb.max(1), rgb.min(1)
        r, g, b = rgb.T
        rs, gs = hi == r, (hi != r) & (hi == g)
        # the bin of a hue on a bin's edge is that of its float32 value, each step rounded once
        f = np.float32
        q = np.where(rs, g - b, np.where(gs, b - r, r - g)).astype(f) / np.maximum(hi - lo, 1).astype(f)
        h6 = np.where(rs, np.where(q < 0, q + f(6), q), np.where(gs, q + f(2), q + f(4)))
        h = np.where(hi > lo, h6, f(0)) / f(6)
        h = np.where(h >= 1, h - f(1), h)
        n = case["bins"]
        bins = np.minimum(np.floor(h * f(n)).astype(np.int64), n - 1)
        return dict(counts=None, density=np.bincount(bins, minlength=n) * (n / h.size), frame=None)
    return None          # frames: bytes
