"""The work a user has this framework do, as measurable cases.

The two halves of the framework are the thermal lattice Boltzmann solver
(single cavities and batches of them) and the warm-start network trained on
its snapshots.  A case is a dict of plain values; `kind` says which public
entry points one pass goes through:

  cavity   lbm.Cavity: step(steps), then the wall Nusselt numbers, the
           diagnostics and the fields, as a run that watches its flow does
  batch    lbm.Batch of ragged cavities: step(steps), the Nusselt numbers of
           all of them, the fields of each
  layer    one 3x3 convolution layer of the network, forward and backward
           (output, data gradient, weight and bias gradient)
  predict  the network's forward pass, prediction in FP32
  gradient forward, masked loss, backward: loss and every gradient

`exact` computes the same in 64 bits with plain torch: the moment-space
collisions by matrix products with the bases of Section 2.2 of the paper, the
streaming by shifted copies, the network by shifted matrix products.
"""
import math

import numpy as np
import torch

from paper_2211_03160_amd import lbm, nn
from paper_2211_03160_amd import workloads as W

MOST_ROLL_NODES = 8_000_000  # larger cavities start from conduction + noise


# ------------------------------------------------------------------- the cases
def listed():
    return [
        # the smallest cell of the warm-start workflow and of first runs:
        # watched every 50 steps, bound by launches and latency
        dict(name="rb2d_65_fp32", kind="cavity", nx=65, ny=65, nz=1, side=False, lateral=False, storage="fp32",
             ra=3e4, pr=0.71, steps=50),
        # the 129^2 validation cell, FP64 storage
        dict(name="rb2d_129_fp64", kind="cavity", nx=129, ny=129, nz=1, side=False, lateral=False, storage="fp64",
             ra=1e5, pr=0.71, steps=100),
        # the cell of the README's example
        dict(name="rb2d_1025_fp32", kind="cavity", nx=1025, ny=1025, nz=1, side=False, lateral=False, storage="fp32",
             ra=1e7, pr=0.71, steps=100),
        # the paper's side-heated cavity, ragged, 16-bit storage
        dict(name="sh2d_1537x2049_fp16", kind="cavity", nx=1537, ny=2049, nz=1, side=True, lateral=False,
             storage="fp16", ra=1e7, pr=0.71, steps=100),
        # the headline cell
        dict(name="rb2d_8193_fp32", kind="cavity", nx=8193, ny=8193, nz=1, side=False, lateral=False, storage="fp32",
             ra=1e8, pr=0.71, steps=40),
        # the small 3D cell of the precision study
        dict(name="rb3d_49_fp32", kind="cavity", nx=49, ny=49, nz=49, side=False, lateral=False, storage="fp32",
             ra=1e5, pr=0.71, steps=40),
        # an ordinary 3D cell, three different sides, FP16 flow with FP32 heat
        dict(name="rb3d_257x193x129_mixed", kind="cavity", nx=257, ny=193, nz=129, side=False, lateral=False,
             storage="mixed", ra=1e6, pr=0.71, steps=40),
        # the 3D benchmark cell
        dict(name="rb3d_385_fp32", kind="cavity", nx=385, ny=385, nz=385, side=False, lateral=False, storage="fp32",
             ra=1e7, pr=0.71, steps=20),
        # the batched sweep (heights and aspect ratios of the benchmark's)
        dict(name="batch16_fp32", kind="batch", count=16, most=1025, storage="fp32", sweep=1234, steps=60),
        # a decoder layer of the 257^2 warm-start network: its widest input
        dict(name="layer_16x136x136_96_32", kind="layer", n=16, h=136, w=136, cin=96, cout=32),
        # predictions for the held-out cavities of the 65^2 warm start
        dict(name="predict_8x34x34", kind="predict", n=8, h=34, w=34, levels=2),
        # one gradient of the 257^2 warm-start training (batch 16, 129 coarse
        # nodes padded to 136)
        dict(name="gradient_16x136x136", kind="gradient", n=16, h=136, w=136, levels=4),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["2d", "2d", "2d", "3d", "3d", "batch", "layer", "predict", "gradient"])
    storage = rng.choice(["fp32", "fp32", "fp64", "fp16", "bf16", "mixed"])
    if kind == "2d":
        nx, ny = _log(rng, 33, 4097), _log(rng, 33, 4097)
        steps = max(4, min(_log(rng, 20, 200), 1_500_000_000 // (nx * ny)))
        return dict(kind="cavity", nx=nx, ny=ny, nz=1, side=rng.random() < 0.3, lateral=rng.random() < 0.3,
                    storage=storage, ra=10.0 ** rng.uniform(4, 8), pr=rng.uniform(0.7, 7.0), steps=steps)
    if kind == "3d":
        nx, ny, nz = _log(rng, 17, 300), _log(rng, 17, 300), _log(rng, 17, 300)
        steps = max(4, min(_log(rng, 10, 60), 250_000_000 // (nx * ny * nz)))
        return dict(kind="cavity", nx=nx, ny=ny, nz=nz, side=rng.random() < 0.3, lateral=rng.random() < 0.3,
                    storage=storage, ra=10.0 ** rng.uniform(4, 7), pr=rng.uniform(0.7, 7.0), steps=steps)
    if kind == "batch":
        return dict(kind="batch", count=rng.randint(2, 20), most=rng.choice([129, 257, 513, 1025]), storage=storage,
                    sweep=rng.randint(1, 1 << 30), steps=_log(rng, 20, 60))
    if kind == "layer":
        ch = [16, 32, 64, 96, 128, 192, 256, 384]
        cin, cout = rng.choice(ch), rng.choice(ch[:5] + [256])
        h, w = _log(rng, 10, 140), _log(rng, 10, 140)
        n = max(1, min(rng.randint(1, 16), int(3e10 / (h * w * cin * cout * 18))))
        return dict(kind="layer", n=n, h=h, w=w, cin=cin, cout=cout)
    levels = rng.randint(2, 4)
    q = 2 ** (levels - 1)
    h, w = q * max(2, _log(rng, 24, 136) // q), q * max(2, _log(rng, 24, 136) // q)
    return dict(kind=kind, n=rng.randint(1, 12), h=h, w=w, levels=levels)


# ------------------------------------------------------------- solver inputs
def _cfg(c):
    dim = 3 if c["nz"] > 1 else 2
    n = (c["nx"], c["ny"], c["nz"])[:dim]
    if c["side"]:
        return W.side_heated(dim, n, ra=c["ra"], pr=c["pr"], storage=c["storage"])
    return W.rayleigh_benard(dim, n, ra=c["ra"], pr=c["pr"], storage=c["storage"],
                             lateral=W.PERIODIC if c["lateral"] else W.ADIABATIC)


def _batch(c):
    heights = [h for h in (129, 257, 513, 1025) if h <= c["most"]]
    cfgs, _ = W.batched_sweep(c["count"], seed=c["sweep"], storage=c["storage"], heights=heights)
    return cfgs


def _rolls(cfg, seed):
    """A convective state to start from (u [dim][N], T [N]): one large roll of
    a seeded strength, the temperature it carries, and noise."""
    dim, (nx, ny, nz) = cfg["dim"], cfg["n"]
    r = np.random.default_rng(seed)
    amp, heat = r.uniform(0.03, 0.06), r.uniform(0.05, 0.15)
    X = (np.arange(nx) + 0.5) / nx
    Y = (np.arange(ny) + 0.5) / ny
    Z = (np.arange(nz) + 0.5) / nz
    V = Y if dim == 2 else Z  # the upward coordinate
    sx, cx = np.sin(np.pi * X) ** 2, np.sin(2 * np.pi * X)
    sv, cv = np.sin(np.pi * V) ** 2, np.sin(2 * np.pi * V)
    if dim == 2:
        u = np.stack([amp * cv[:, None] * sx[None, :], -amp * sv[:, None] * cx[None, :]])
        across = sv[:, None] * cx[None, :]
        shape = (ny, nx)
    else:
        mid = np.sin(np.pi * Y) ** 2
        u = np.stack([amp * cv[:, None, None] * mid[None, :, None] * sx[None, None, :],
                      0.2 * amp * sv[:, None, None] * np.sin(2 * np.pi * Y)[None, :, None] * sx[None, None, :],
                      -amp * sv[:, None, None] * mid[None, :, None] * cx[None, None, :]])
        across = sv[:, None, None] * mid[None, :, None] * cx[None, None, :]
        shape = (nz, ny, nx)
    hot_x = cfg["bc"][0] == W.DIRICHLET
    base = 1.0 - X if hot_x else (1.0 - V).reshape((-1,) + (1,) * (dim - 1))
    T = base - heat * across + W.NOISE * (2.0 * r.random(shape) - 1.0)
    return u.reshape(dim, -1), np.ascontiguousarray(np.broadcast_to(T, shape)).ravel()


def _nodes(cfg):
    return cfg["n"][0] * cfg["n"][1] * cfg["n"][2]


# ----------------------------------------------------------- network inputs
CHANS = (32, 64, 128, 256)


def _unet_shapes(levels, cin=16, cout=16):
    ch, shapes, prev = CHANS[:levels], [], cin
    for lvl in range(levels):
        shapes += [(prev, ch[lvl]), (ch[lvl], ch[lvl])]
        prev = ch[lvl]
    for lvl in range(levels - 2, -1, -1):
        shapes += [(prev + ch[lvl], ch[lvl]), (ch[lvl], ch[lvl])]
        prev = ch[lvl]
    return shapes + [(prev, cout)]


def _bf(x):
    return x.to(torch.bfloat16).to(torch.float32)


def _gen(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    return g


def _layer_inputs(c, seed):
    """FP32 tensors that hold BF16 values: activations (a ReLU's output),
    weights [tap][cout][cin], output gradient; and the FP32 bias."""
    g = _gen(seed)
    x = torch.randn(c["n"], c["h"], c["w"], c["cin"], generator=g, device="cuda").clamp_min_(0)
    w = torch.randn(9, c["cout"], c["cin"], generator=g, device="cuda") * math.sqrt(2.0 / (9 * c["cin"]))
    b = 0.1 * torch.randn(c["cout"], generator=g, device="cuda")
    dy = 1e-3 * torch.randn(c["n"], c["h"], c["w"], c["cout"], generator=g, device="cuda")
    return _bf(x), _bf(w), b, _bf(dy)


def _net_inputs(c, seed):
    """Input planes as the warm start makes them (conduction profile, log Ra,
    Pr, aspect, inside mask, zeros), targets and mask, weights and biases."""
    g = _gen(seed)
    n, h, w = c["n"], c["h"], c["w"]
    inside_h, inside_w = h - h // 20, w - w // 20
    x = torch.zeros(n, h, w, 16, device="cuda")
    v = (torch.arange(inside_h, device="cuda") + 0.5) / inside_h
    x[:, :inside_h, :inside_w, 0] = (0.5 - v)[None, :, None]
    for k in (1, 2, 3):
        x[:, :inside_h, :inside_w, k] = (2 * torch.rand(n, generator=g, device="cuda") - 1)[:, None, None]
    x[:, :inside_h, :inside_w, 4] = 1.0
    t = torch.zeros(n, h, w, 3, device="cuda")
    m = torch.zeros(n, h, w, 3, device="cuda")
    m[:, :inside_h, :inside_w] = 1.0
    phase = 6.28 * torch.rand(n, 1, 1, 3, generator=g, device="cuda")
    u = torch.arange(inside_w, device="cuda") / inside_w
    t[:, :inside_h, :inside_w] = 0.5 * torch.sin(6.28 * u[None, None, :, None] + phase) * \
        torch.sin(3.14 * v)[None, :, None, None]
    ws, bs = [], []
    for ci, co in _unet_shapes(c["levels"]):
        ws.append(_bf(torch.randn(9, co, ci, generator=g, device="cuda") * math.sqrt(2.0 / (9 * ci))))
        bs.append(0.02 * torch.randn(co, generator=g, device="cuda"))
    return _bf(x), t, m, ws, bs


# -------------------------------------------------------------------- prepare
def prepare(case, seed):
    c = case
    if c["kind"] == "cavity":
        cfg = _cfg(c)
        cav = lbm.Cavity(cfg)
        if _nodes(cfg) <= MOST_ROLL_NODES:
            cav.init_fields(None, *_rolls(cfg, seed))
        else:
            cav.init(seed, W.NOISE)
        return dict(case=c, cavity=cav)
    if c["kind"] == "batch":
        cfgs = _batch(c)
        b = lbm.Batch(cfgs)
        b.init([seed + k for k in range(len(cfgs))], [W.NOISE] * len(cfgs))
        for k, cfg in enumerate(cfgs):
            b.init_fields(k, None, *_rolls(cfg, seed + k))
        return dict(case=c, batch=b, views=[b.cavity(k) for k in range(len(cfgs))])
    if c["kind"] == "layer":
        x, w, b, dy = _layer_inputs(c, seed)
        gw = torch.empty_like(w)
        gb = torch.empty_like(b)
        return dict(case=c, x=nn.to_bf16(x), w=nn.to_bf16(w), b=b, dy=nn.to_bf16(dy), gw=gw, gb=gb)
    x, t, m, ws, bs = _net_inputs(c, seed)
    net = nn.UNet(chans=CHANS[: c["levels"]], seed=1)
    net.set_weights([w.cpu().numpy() for w in ws], [b.cpu().numpy() for b in bs])
    return dict(case=c, net=net, x=nn.to_bf16(x), t=t, m=m)


# ------------------------------------------------------------------------ run
def run(state):
    s = state
    c = s["case"]
    if c["kind"] == "cavity":
        cav = s["cavity"]
        cav.step(c["steps"])
        nu = cav.nusselt()
        d = cav.diagnostics()
        rho, u, T = cav.fields_device()
        return dict(nu=list(nu), mass=d["mass"], energy=d["energy"], umax=d["umax"], nu_vol=d["nu_vol"], re=d["re"],
                    nonfinite=d["nonfinite"], rho=rho, u=u, T=T)
    if c["kind"] == "batch":
        b = s["batch"]
        b.step(c["steps"])
        hot, cold = b.nusselt()
        return dict(hot=hot, cold=cold, fields=[list(v.fields_device()) for v in s["views"]])
    if c["kind"] == "layer":
        y = nn.conv3x3(s["x"], s["w"], s["b"], c["cout"], True)
        dz = nn.relu_backward(y, s["dy"])
        nn.conv3x3_wgrad(s["x"], dz, c["cout"], s["gw"], s["gb"])
        dx = nn.conv3x3(dz, nn.conv3x3_flip(s["w"], c["cin"], c["cout"]), None, c["cin"], False)
        return dict(y=y.view(torch.bfloat16), dx=dx.view(torch.bfloat16), gw=s["gw"], gb=s["gb"])
    net = s["net"]
    y, tape = net.forward(s["x"])
    if c["kind"] == "predict":
        return dict(y=nn.to_f32(y))
    loss, dy = nn.mse(y, s["t"], s["m"])
    net.backward(tape, dy)
    return dict(loss=loss, y=y.view(torch.bfloat16), gw=[lay["gw"] for lay in net.layers],
                gb=[lay["gb"] for lay in net.layers])


# ----------------------------------------------------------------------- work
def _cavity_work(cfg, steps):
    dim, n = cfg["dim"], _nodes(cfg)
    qf, qg = (9, 5) if dim == 2 else (19, 7)
    ef = {"fp32": 4, "fp64": 8}.get(cfg["storage"], 2)
    eg = {"fp32": 4, "fp64": 8, "mixed": 4}.get(cfg["storage"], 2)
    # the state in, the state out, the fields; 148 and 330 operations are
    # what the moment-space collisions of the two lattices take per update
    return n * (2 * (qf * ef + qg * eg) + 8 * (2 + dim)), n * steps * (148 if dim == 2 else 330)


def _unet_flops(c, backward):
    total, lv = 0.0, c["levels"]
    res = [v for v in range(lv) for _ in range(2)] + [v for v in range(lv - 2, -1, -1) for _ in range(2)] + [0]
    for k, ((ci, co), v) in enumerate(zip(_unet_shapes(lv), res)):
        mac = c["n"] * (c["h"] >> v) * (c["w"] >> v) * 9 * ci * co
        total += 2 * mac * ((3 if k else 2) if backward else 1)
    return total


def work(case):
    c = case
    if c["kind"] == "cavity":
        b, f = _cavity_work(_cfg(c), c["steps"])
        return dict(bytes=b, flops=f)
    if c["kind"] == "batch":
        both = [_cavity_work(cfg, c["steps"]) for cfg in _batch(c)]
        return dict(bytes=sum(v[0] for v in both), flops=sum(v[1] for v in both))
    if c["kind"] == "layer":
        p, ci, co = c["n"] * c["h"] * c["w"], c["cin"], c["cout"]
        return dict(bytes=2 * p * (2 * ci + 2 * co) + 9 * ci * co * 6, flops=3 * 2.0 * p * 9 * ci * co)
    weights = sum(9 * ci * co for ci, co in _unet_shapes(c["levels"]))
    p = c["n"] * c["h"] * c["w"]
    back = c["kind"] == "gradient"
    return dict(bytes=p * (32 + (32 + 24 if back else 64)) + weights * (6 if back else 2), flops=_unet_flops(c, back))


# ---------------------------------------------------- the solver in 64 bits
def _lattice(dim):
    """(e flow, w flow, M, rate names), (e heat, N, rate names), a_T."""
    if dim == 2:
        ef = [(0, 0), (1, 0), (0, 1), (-1, 0), (0, -1), (1, 1), (-1, 1), (-1, -1), (1, -1)]
        wf = [4 / 9] + [1 / 9] * 4 + [1 / 36] * 4

        def row(x, y):
            s = x * x + y * y
            return [1, 3 * s - 4, (9 * s * s - 21 * s + 8) / 2, x, (3 * s - 5) * x, y, (3 * s - 5) * y,
                    x * x - y * y, x * y]

        kf = ["0", "nu", "nu", "0", "q", "0", "q", "nu", "nu"]
        eg = ef[:5]

        def rowg(x, y):
            s = x * x + y * y
            return [1, x, y, 5 * s - 4, x * x - y * y]

        kg = ["0", "j", "j", "1", "1"]
        return (ef, wf, [row(*e) for e in ef], kf), (eg, [rowg(*e) for e in eg], kg), -1.5
    ax = [(1, 0, 0), (0, 1, 0), (0, 0, 1)]
    ed = [(1, 1, 0), (1, -1, 0), (1, 0, 1), (1, 0, -1), (0, 1, 1), (0, 1, -1)]
    neg = lambda e: tuple(-v for v in e)  # noqa: E731
    ef = [(0, 0, 0)] + [p for e in ax + ed for p in (e, neg(e))]
    wf = [1 / 3] + [1 / 18] * 6 + [1 / 36] * 12

    def row3(x, y, z):
        s = x * x + y * y + z * z
        return [1, 19 * s - 30, (21 * s * s - 53 * s + 24) / 2, x, (5 * s - 9) * x, y, (5 * s - 9) * y, z,
                (5 * s - 9) * z, 3 * x * x - s, (3 * s - 5) * (3 * x * x - s), y * y - z * z,
                (3 * s - 5) * (y * y - z * z), x * y, y * z, x * z, (y * y - z * z) * x, (z * z - x * x) * y,
                (x * x - y * y) * z]

    kf = ["0", "nu", "nu", "0", "q", "0", "q", "0", "q", "nu", "nu", "nu", "nu", "nu", "nu", "nu", "q", "q", "q"]
    eg = ef[:7]

    def rowg3(x, y, z):
        s = x * x + y * y + z * z
        return [1, x, y, z, 7 * s - 6, 3 * x * x - s, y * y - z * z]

    kg = ["0", "j", "j", "j", "1", "1", "1"]
    return (ef, wf, [row3(*e) for e in ef], kf), (eg, [rowg3(*e) for e in eg], kg), -0.75


def _noise(n, seed):
    """2 s - 1 per node, s the top 53 bits of SplitMix64 of seed xor SplitMix64(node)."""
    def wrap(v):
        v &= (1 << 64) - 1
        return v - (1 << 64) if v >> 63 else v

    def mix(x):
        z = x + wrap(0x9E3779B97F4A7C15)
        z = (z ^ ((z >> 30) & ((1 << 34) - 1))) * wrap(0xBF58476D1CE4E5B9)
        z = (z ^ ((z >> 27) & ((1 << 37) - 1))) * wrap(0x94D049BB133111EB)
        return z ^ ((z >> 31) & ((1 << 33) - 1))

    idx = torch.arange(n, dtype=torch.int64, device="cuda")
    r = (mix(mix(idx) ^ wrap(seed)) >> 11) & ((1 << 53) - 1)
    return 2.0 * (r.double() * 2.0 ** -53) - 1.0


class _Solver:
    """The discrete step of Section 2.2 in FP64: moments, both collisions in
    moment space, pull streaming with half-way bounce-back and
    anti-bounce-back, and the wall heat flux."""

    def __init__(self, cfg):
        D = dict(dtype=torch.float64, device="cuda")
        self.cfg, self.dim = cfg, cfg["dim"]
        dim = self.dim
        (self.ef, wf, M, kf), (self.eg, Mg, kg), at = _lattice(dim)
        self.n = cfg["n"][:dim]
        H, U, dT = self.n[-1], cfg["u_ff"], cfg["t_hot"] - cfg["t_cold"]
        self.H, self.dT = H, dT
        self.nu = U * H * math.sqrt(cfg["pr"] / cfg["ra"])
        self.alpha = U * H / math.sqrt(cfg["pr"] * cfg["ra"])
        self.gb, self.T0 = U * U / (dT * H), 0.5 * (cfg["t_hot"] + cfg["t_cold"])
        s_nu = 1.0 / (3 * self.nu + 0.5)
        moving = (4 + at) / 20 if dim == 2 else (6 + at) / 42
        rates = {"0": 0.0, "nu": s_nu, "q": 8 * (2 - s_nu) / (8 - s_nu), "1": 1.0,
                 "j": 1.0 / (self.alpha / (2 * moving) + 0.5)}
        self.omega, self.at = 2 * moving, at
        self.e = torch.tensor(self.ef, **D)
        self.w = torch.tensor(wf, **D)
        self.M, self.Mg = torch.tensor(M, **D).T.contiguous(), torch.tensor(Mg, **D).T.contiguous()
        self.Mi, self.Mgi = torch.linalg.inv(self.M), torch.linalg.inv(self.Mg)
        self.S, self.Sg = torch.tensor([[rates[k]] for k in kf], **D), torch.tensor([[rates[k]] for k in kg], **D)
        self.eg_t = torch.tensor(self.eg, **D)
        # node arrays are [..., y, x]: axis a of a velocity is dimension -1 - a
        self.shape = tuple(reversed(self.n))

    def feq(self, rho, u):
        eu = self.e @ u
        return self.w[:, None] * rho * (1 + 3 * eu + 4.5 * eu * eu - 1.5 * (u * u).sum(0))

    def geq(self, T, u):
        zero = torch.zeros_like(T)
        rows = [T] + [u[a] * T for a in range(self.dim)] + [self.at * T] + [zero] * (len(self.eg) - self.dim - 2)
        return torch.stack(rows)

    def start(self, rho, u, T):
        parts = [(self.feq(rho[k], u[:, k]), self.Mgi @ self.geq(T[k], u[:, k])) for k in self.chunks(len(T))]
        self.f, self.g = (torch.cat(p, 1) for p in zip(*parts))

    @staticmethod
    def chunks(n, size=1 << 22):
        return [slice(a, min(a + size, n)) for a in range(0, n, size)]

    def moments(self, f, g):
        rho, T = f.sum(0), g.sum(0)
        F = rho * self.gb * (T - self.T0)
        j = self.e.T @ f
        j[-1] += 0.5 * F
        return rho, j / rho, T, F

    def collide(self):
        for k in self.chunks(self.f.shape[1]):
            f, g = self.f[:, k].contiguous(), self.g[:, k].contiguous()
            rho, u, T, F = self.moments(f, g)
            eu = self.e @ u
            src = self.w[:, None] * F * (3 * (self.e[:, -1:] - u[-1]) + 9 * eu * self.e[:, -1:])
            d = -self.S * (self.M @ (f - self.feq(rho, u))) + (1 - 0.5 * self.S) * (self.M @ src)
            dg = -self.Sg * (self.Mg @ g - self.geq(T, u))
            self.f[:, k] = f + self.Mi @ d
            self.g[:, k] = g + self.Mgi @ dg

    def stream(self):
        flux = [0.0] * 6
        f, g = self.f.view((-1,) + self.shape), self.g.view((-1,) + self.shape)
        bc, tw = self.cfg["bc"], self.cfg["t_wall"]
        out = []
        for pops, es, heat in ((f, self.ef, False), (g, self.eg, True)):
            new = torch.empty_like(pops)
            for i, e in enumerate(es):
                o = es.index(tuple(-v for v in e))
                new[i] = torch.roll(pops[i], shifts=tuple(e), dims=tuple(-1 - a for a in range(self.dim)))
                for a in range(self.dim):
                    face = 2 * a + (0 if e[a] > 0 else 1)
                    if e[a] == 0 or bc[face] == W.PERIODIC:
                        continue
                    at = [slice(None)] * self.dim
                    at[self.dim - 1 - a] = 0 if e[a] > 0 else self.n[a] - 1
                    own = pops[o][tuple(at)]
                    if heat and bc[face] == W.DIRICHLET:
                        new[i][tuple(at)] = self.omega * tw[face] - own
                        flux[face] = float((self.omega * tw[face] - 2 * own).sum())
                    else:
                        new[i][tuple(at)] = own
            out.append(new.view(len(es), -1))
        self.f, self.g = out
        return flux

    def steps(self, n):
        fluxes = []
        for _ in range(n):
            self.collide()
            fluxes.append(self.stream())
        mean = [0.5 * (a + b) for a, b in zip(fluxes[-1], fluxes[-2])]
        nodes = math.prod(self.n)
        nu = []
        for sign, hot in ((1.0, True), (-1.0, False)):
            num = area = 0.0
            for face in range(2 * self.dim):
                tw = self.cfg["t_wall"][face]
                if self.cfg["bc"][face] == W.DIRICHLET and tw != self.T0 and (tw > self.T0) == hot:
                    num += sign * self.n[face // 2] * mean[face]
                    area += nodes / self.n[face // 2]
            nu.append(num / (self.alpha * self.dT) / area)
        parts = [self.moments(self.f[:, k].contiguous(), self.g[:, k].contiguous())[:3]
                 for k in self.chunks(self.f.shape[1])]
        rho, u, T = (torch.cat(p, -1) for p in zip(*parts))
        return nu, rho, u, T

    def watch(self, n):
        nu, rho, u, T = self.steps(n)
        uu = (u * u).sum(0)
        return dict(nu=nu, mass=float(rho.sum()), energy=float(T.sum()), umax=float(uu.max().sqrt()),
                    nu_vol=float(1 + self.H * (u[-1] * (T - self.T0)).mean() / (self.alpha * self.dT)),
                    re=float(uu.mean().sqrt() * self.H / self.nu), nonfinite=None, rho=rho, u=u.reshape(-1), T=T)


def _started(cfg, seed):
    s = _Solver(cfg)
    n = _nodes(cfg)
    D = dict(dtype=torch.float64, device="cuda")
    rho = torch.ones(n, **D)
    if n <= MOST_ROLL_NODES:
        u, T = _rolls(cfg, seed)
        s.start(rho, torch.from_numpy(u).cuda(), torch.from_numpy(T).cuda())
        return s
    ax = 0 if cfg["bc"][0] == W.DIRICHLET else s.dim - 1
    lo, hi = cfg["t_wall"][2 * ax], cfg["t_wall"][2 * ax + 1]
    k = (torch.arange(s.n[ax], **D) + 0.5) * (hi - lo) / s.n[ax] + lo
    T = k.reshape([-1 if s.dim - 1 - d == ax else 1 for d in range(s.dim)]).expand(s.shape).reshape(-1)
    s.start(rho, torch.zeros(s.dim, n, **D), T + W.NOISE * _noise(n, seed))
    return s


# --------------------------------------------------- the network in 64 bits
def _conv(x, w):
    """3x3 convolution, zero padding: x [n][h][w][ci], w [tap][co][ci]."""
    n, h, wd, ci = x.shape
    p = torch.nn.functional.pad(x, (0, 0, 1, 1, 1, 1))
    y = 0
    for t in range(9):
        i, j = t // 3, t % 3
        y = y + p[:, i:i + h, j:j + wd].reshape(-1, ci) @ w[t].T
    return y.view(n, h, wd, -1)


def _unet(x, ws, bs, levels):
    k, skips, h = 0, [], x
    for lvl in range(levels):
        if lvl:
            n, a, b, c = h.shape
            h = h.view(n, a // 2, 2, b // 2, 2, c).mean((2, 4))
        for _ in range(2):
            h, k = torch.relu(_conv(h, ws[k]) + bs[k]), k + 1
        skips.append(h)
    for lvl in range(levels - 2, -1, -1):
        h = torch.cat([h.repeat_interleave(2, 1).repeat_interleave(2, 2), skips[lvl]], -1)
        for _ in range(2):
            h, k = torch.relu(_conv(h, ws[k]) + bs[k]), k + 1
    return _conv(h, ws[k]) + bs[k]


def exact(case, seed):
    c = case
    if c["kind"] == "cavity":
        return _started(_cfg(c), seed).watch(c["steps"])
    if c["kind"] == "batch":
        hot, cold, fields = [], [], []
        for k, cfg in enumerate(_batch(c)):
            nu, rho, u, T = _started(cfg, seed + k).steps(c["steps"])
            hot.append(nu[0])
            cold.append(nu[1])
            fields.append([rho, u.reshape(-1), T])
        return dict(hot=np.array(hot), cold=np.array(cold), fields=fields)
    if c["kind"] == "layer":
        x, w, b, dy = (v.double() for v in _layer_inputs(c, seed))
        x.requires_grad_(), w.requires_grad_(), b.requires_grad_()
        y = torch.relu(_conv(x, w) + b)
        y.backward(dy)
        return dict(y=y.detach(), dx=x.grad, gw=w.grad, gb=b.grad)
    x, t, m, ws, bs = _net_inputs(c, seed)
    ws = [w.double().requires_grad_() for w in ws]
    bs = [b.double().requires_grad_() for b in bs]
    y = _unet(x.double(), ws, bs, c["levels"])
    if c["kind"] == "predict":
        return dict(y=y.detach())
    loss = (((y[..., :3] - t) * m) ** 2).sum() / m.double().sum()
    loss.backward()
    return dict(loss=loss.detach().reshape(1), y=y.detach(), gw=[w.grad for w in ws], gb=[b.grad for b in bs])
