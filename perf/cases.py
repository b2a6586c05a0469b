"""Workloads that stand for what this framework is used for, each as a state a
program holds (`prepare`) and one pass over it (`run`):

cavity    one cavity advanced by a monitoring interval (lbmx.Cavity.step), its
          Nusselt numbers and map and its fields read back: the body of every
          steady-state run;
batch     a set of uneven cavities advanced together (lbmx.Batch), their Nu and
          their fields resampled to 64^3: the data-set generation;
start     a cavity initialised from other cavities or from predicted fields
          (grid sequencing, extrapolated start, warm start);
train     one optimiser step of the warm-start U-Net;
predict   the U-Net's prediction of a case's fields;
conv      one of the U-Net's 3x3x3 convolution layers, forward and backward;
upcat     a decoder layer reading its upsampled-and-concatenated input in place.

`exact` gives the same outputs in 64-bit arithmetic from plain torch.
"""
import math
import os

import numpy as np
import torch

from paper_1511_04633_amd import inputs, lbmx, unet

WEIGHTS = os.path.join(os.path.dirname(os.path.abspath(unet.__file__)), "weights", "unet64.npz")
# (input channels, output channels) of the network's layers at its resolutions;
# decoder layers as (upsampled, skip, output).
LAYERS = ((16, 16), (16, 32), (32, 32), (32, 64), (64, 64), (64, 96), (96, 96))
UPCAT = ((96, 64, 64), (64, 32, 32), (32, 16, 16))
STORAGES = ("f32", "f32", "f32", "f64", "f16_f32", "f16_i16", "f16")


def listed():
    return [
        # the smallest grid run (16^3, Ra 1e3), where a step costs one launch
        dict(name="cavity_16_f32", kind="cavity", n=16, wall_type=1, ra=1e3, storage="f32", steps=1000),
        # the paper's 50^3 grid in FP64: validation runs
        dict(name="cavity_50_f64", kind="cavity", n=50, wall_type=2, ra=1e4, storage="f64", steps=500),
        # the coarse level of a grid-sequenced 128^3 run
        dict(name="cavity_64_f32", kind="cavity", n=64, wall_type=3, ra=1e5, storage="f32", steps=1000),
        # the 16-bit storage that keeps the Nu target
        dict(name="cavity_96_f16_i16", kind="cavity", n=96, wall_type=2, ra=3e5, storage="f16_i16", steps=500),
        # the time-to-steady grid
        dict(name="cavity_128_f32", kind="cavity", n=128, wall_type=1, ra=1e5, storage="f32", steps=1000),
        # the benchmark grid
        dict(name="cavity_256_f32", kind="cavity", n=256, wall_type=1, ra=1e6, storage="f32", steps=1000),
        # 16 uneven cavities of the data set, one monitoring interval
        dict(name="batch_16_f32", kind="batch", count=16, batch_seed=1511, storage="f32", steps=500),
        # grid sequencing: a 192^3 cavity started from a 96^3 one
        dict(name="start_96_192_f32", kind="start", how="cavity", m=96, n=192, storage="f32"),
        # one training step at the training batch and size
        dict(name="train_4x64", kind="train", B=4, m=64),
        # the warm start's inference
        dict(name="predict_1x64", kind="predict", B=1, m=64),
        # the full-resolution encoder layer
        dict(name="conv_16_16_64", kind="conv", B=4, D=64, H=64, W=64, ci=16, co=16),
        # the deepest decoder layer: many channels on a small grid
        dict(name="upcat_96_64_64_16", kind="upcat", B=4, D=16, H=16, W=16, cu=96, cs=64, co=64),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(("cavity", "cavity", "cavity", "batch", "start", "train", "predict", "conv", "conv", "upcat"))
    if kind == "cavity":
        n = _log_int(rng, 12, 240)
        most = 4.5 if n < 32 else 6.0
        storage = rng.choice(STORAGES)
        steps = max(20, min(1000, int(6e9 / n ** 3 * (0.5 if storage == "f64" else 1.0))))
        return dict(kind=kind, n=n, wall_type=rng.randint(1, 3), ra=10.0 ** rng.uniform(3.0, most),
                    storage=storage, steps=rng.randint(max(1, steps // 2), steps))
    if kind == "batch":
        return dict(kind=kind, count=rng.randint(2, 16), batch_seed=rng.randint(1, 10 ** 6),
                    storage=rng.choice(("f32", "f32", "f16_i16")), steps=rng.randint(100, 500))
    if kind == "start":
        n = _log_int(rng, 24, 200)
        return dict(kind=kind, how=rng.choice(("cavity", "two", "fields")), m=max(16, n // 2), n=n,
                    storage=rng.choice(("f32", "f32", "f16_f32", "f64")))
    if kind == "train":
        return dict(kind=kind, B=rng.randint(1, 6), m=rng.choice((16, 32, 48, 64)))
    if kind == "predict":
        return dict(kind=kind, B=rng.randint(1, 4), m=rng.choice((16, 24, 32, 48, 64, 80)))
    B = rng.randint(1, 4)
    if kind == "conv":
        ci, co = rng.choice(LAYERS)
        return dict(kind=kind, B=B, D=_log_int(rng, 6, 72), H=_log_int(rng, 6, 72), W=_log_int(rng, 6, 72),
                    ci=ci, co=co)
    cu, cs, co = rng.choice(UPCAT)
    return dict(kind=kind, B=B, D=2 * _log_int(rng, 4, 32), H=2 * _log_int(rng, 4, 32),
                W=2 * _log_int(rng, 4, 32), cu=cu, cs=cs, co=co)


# ------------------------------------------------------------------- inputs
def _gen(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed))
    return g


def _smooth_fields(m, seed):
    """u, v, w, theta (FP32 [m, m, m], z y x) like a convecting cavity's:
    velocities a few per cent in lattice units that vanish at the walls, theta
    the conduction profile with a smooth disturbance."""
    amp = 2.0 * inputs.uniform01(seed, 64).reshape(4, 16) - 1.0
    ax = (torch.arange(m, device="cuda", dtype=torch.float64) + 0.5) / m
    z, y, x = torch.meshgrid(ax, ax, ax, indexing="ij")
    wall = torch.sin(math.pi * x) * torch.sin(math.pi * y) * torch.sin(math.pi * z)
    out = []
    for k in range(4):
        s = torch.zeros_like(wall)
        for q in range(4):
            a, b, c = 1 + q % 3, 1 + (q + k) % 3, 1 + (q + 2 * k) % 2
            s = s + amp[k, q] * torch.cos(a * math.pi * x + 3.0 * amp[k, 4 + q]) * \
                torch.cos(b * math.pi * y) * torch.cos(c * math.pi * z + amp[k, 8 + q])
        out.append(0.01 * wall * s if k < 3 else 0.5 - y + 0.1 * wall * s)
    return [t.float().contiguous() for t in out]


def _cavity(case, n, seed, src=48):
    cav = lbmx.Cavity(n=n, wall_type=case.get("wall_type", 1), ra=case.get("ra", 1e5),
                      storage=case["storage"])
    f = _smooth_fields(src, seed)
    torch.cuda.synchronize()
    cav.init_fields(*f)
    return cav


def _bf(t):
    return t.to(torch.bfloat16).contiguous()


def _layer(case, seed):
    """Tensors of one layer: activations as after SiLU, weights of the
    initialisation's scale, a small output gradient, the pre-activation of the
    layer before."""
    g = _gen(seed)
    B, D, H, W, co = (case[k] for k in ("B", "D", "H", "W", "co"))
    rn = lambda *s: torch.randn(s, generator=g, device="cuda")  # noqa: E731
    act = lambda *s: _bf(torch.nn.functional.silu(rn(*s)))      # noqa: E731
    up = case["kind"] == "upcat"
    ci = case["cu"] + case["cs"] if up else case["ci"]
    t = {"w": _bf(rn(co, 27, ci) * math.sqrt(2.0 / (27 * ci))), "b": 0.1 * rn(co),
         "gz": _bf(1e-3 * rn(B, D, H, W, co))}
    if up:
        t["low"] = act(B, D // 2, H // 2, W // 2, case["cu"])
        t["skip"] = act(B, D, H, W, case["cs"])
    else:
        t["x"] = act(B, D, H, W, ci)
        t["zprev"] = _bf(rn(B, D, H, W, ci))
    return t


def _net_inputs(case, seed):
    r = np.random.default_rng(seed)
    B = case["B"]
    return r.uniform(3.0, 6.0, B), r.integers(1, 4, B)


def _load_net(m):
    net = unet.UNet(seed=0, m=m)
    z = np.load(WEIGHTS, allow_pickle=False)
    net.load_state({k: z[k] for k in z.files})
    return net


def _target(case, seed):
    V = case["m"] ** 3
    f = [torch.stack(_smooth_fields(case["m"], seed + 31 * b)).reshape(4, V) for b in range(case["B"])]
    scale = torch.tensor([50.0, 50.0, 50.0, 3.0], device="cuda")
    return (torch.stack(f) * scale[:, None]).transpose(1, 2).contiguous()


def _moments(seed):
    """Adam moments as in the middle of a training run (per layer the weights',
    then the biases')."""
    g = _gen(seed + 1)
    out = []
    for ci, co, _ in _net_layers(64):
        for shape in ((co, 27, ci), (co,)):
            sd = 1e-3 * torch.rand(shape, generator=g, device="cuda") + 1e-3
            out.append((sd * torch.randn(shape, generator=g, device="cuda"), sd * sd))
    return out


STEP = 2000  # optimiser steps taken before the timed one
LR = 5e-4


# ------------------------------------------------------------------ prepare
def prepare(case, seed):
    kind = case["kind"]
    if kind == "cavity":
        return {"case": case, "cav": _cavity(case, case["n"], seed)}
    if kind == "batch":
        cases = inputs.batch_cases(case["batch_seed"], case["count"])
        b = lbmx.Batch(cases, storage=case["storage"])
        b.autotune()
        for k, c in enumerate(cases):
            n = c["n"]
            y = (np.arange(n) + 0.5) / n
            th = np.broadcast_to((0.5 - y)[None, :, None], (n, n, n)).reshape(-1)
            b.init_rest(k, th + inputs.theta_noise(n, seed + k, 0.05))
        return {"case": case, "batch": b}
    if kind == "start":
        s = {"case": case, "dst": lbmx.Cavity(n=case["n"], wall_type=1, ra=1e5, storage=case["storage"])}
        if case["how"] == "fields":
            s["fields"] = _smooth_fields(64, seed)
        else:
            s["a"] = _cavity(case, case["m"], seed)
            if case["how"] == "two":
                s["b"] = _cavity(case, max(8, case["m"] // 2), seed + 1)
        torch.cuda.synchronize()
        return s
    if kind in ("train", "predict"):
        net = _load_net(case["m"])
        lr, wt = _net_inputs(case, seed)
        s = {"case": case, "net": net, "cond": unet.cond_tensor(lr, wt), "log10_ra": lr, "wall_type": wt}
        if kind == "train":
            s["target"] = _target(case, seed)
            s["partial"] = torch.zeros(1024, dtype=torch.float64, device="cuda")
            mom = iter(_moments(seed))
            for c in net.convs():
                for m, v in ((c.mw, c.vw), (c.mb, c.vb)):
                    a, b = next(mom)
                    m.copy_(a)
                    v.copy_(b)
            net.step_count = STEP
        return s
    t = _layer(case, seed)
    ci, co = t["w"].shape[2], t["w"].shape[0]
    t["wflip"] = torch.empty((ci, 27, co), dtype=torch.bfloat16, device="cuda")
    unet.call("lbmx_nn_conv3d_flip", unet.P(t["w"]), unet.P(t["wflip"]), ci, co, unet.stream_ptr())
    t["gw"] = torch.zeros((co, 27, ci), device="cuda")
    t["gb"] = torch.zeros(co, device="cuda")
    return {"case": case, "t": t}


# ---------------------------------------------------------------------- run
def _read(cav):
    nu = cav.nusselt(with_map=True)
    rho, ux, uy, uz, th = cav.read_macro()
    return {"nu": [nu["nu3d"], nu["nu2d"], nu["numax"]], "map": nu["map"], "rho": rho, "u": ux, "v": uy,
            "w": uz, "theta": th}


def run(state):
    case = state["case"]
    kind = case["kind"]
    if kind == "cavity":
        state["cav"].step(case["steps"])
        return _read(state["cav"])
    if kind == "batch":
        b = state["batch"]
        b.step(case["steps"])
        nu = [b.nusselt(k) for k in range(len(b))]
        return {"nu": np.array([[v["nu3d"], v["nu2d"], v["numax"]] for v in nu]),
                "fields": [b.resample(k, 64) for k in range(len(b))]}
    if kind == "start":
        d = state["dst"]
        if case["how"] == "cavity":
            d.init_from(state["a"])
        elif case["how"] == "two":
            d.init_from_two(state["a"], 1.25, state["b"], -0.25)
        else:
            d.init_fields(*state["fields"])
        return _read(d)
    if kind == "predict":
        if case["B"] == 1:
            return unet.predict_fields(state["net"], float(state["log10_ra"][0]), int(state["wall_type"][0]))
        return state["net"].forward(state["cond"], case["B"])
    if kind == "train":
        net = state["net"]
        grad, count = net.forward_loss(state["cond"], case["B"], state["target"], state["partial"])
        net.backward(grad)
        net.adam(LR)
        return {"loss": (state["partial"].sum() / count).float(),
                "w": [c.w for c in net.convs()], "b": [c.b for c in net.convs()]}
    t, s, P = state["t"], unet.stream_ptr(), unet.P
    B, D, H, W, co = (case[k] for k in ("B", "D", "H", "W", "co"))
    e = lambda c: torch.empty((B, D, H, W, c), dtype=torch.bfloat16, device="cuda")  # noqa: E731
    z, a = e(co), e(co)
    t["gw"].zero_()
    t["gb"].zero_()
    if kind == "conv":
        ci = case["ci"]
        unet.call("lbmx_nn_conv3d_fwd_ep", P(t["x"]), P(t["w"]), P(t["b"]), P(z), P(a), None, None, 0,
                  B, D, H, W, ci, co, s)
        unet.call("lbmx_nn_conv3d_wgrad", P(t["x"]), P(t["gz"]), P(t["gw"]), P(t["gb"]), B, D, H, W, ci,
                  co, s)
        gx = e(ci)
        unet.call("lbmx_nn_conv3d_fwd_ep", P(t["gz"]), P(t["wflip"]), None, P(gx), None, P(t["zprev"]),
                  None, 0, B, D, H, W, co, ci, s)
        return {"z": z, "a": a, "gw": t["gw"], "gb": t["gb"], "gx": gx}
    cu, cs = case["cu"], case["cs"]
    unet.call("lbmx_nn_conv3d_fwd_upcat", P(t["low"]), P(t["skip"]), P(t["w"]), P(t["b"]), P(z), P(a), B,
              D, H, W, cu, cs, co, s)
    unet.call("lbmx_nn_conv3d_wgrad_upcat", P(t["low"]), P(t["skip"]), P(t["gz"]), P(t["gw"]), P(t["gb"]),
              B, D, H, W, cu, cs, co, s)
    gu, gs = e(cu), e(cs)
    unet.call("lbmx_nn_conv3d_fwd_ep", P(t["gz"]), P(t["wflip"]), None, P(gu), None, None, P(gs), cu, B, D,
              H, W, co, cu + cs, s)
    return {"z": z, "a": a, "gw": t["gw"], "gb": t["gb"], "gu": gu, "gs": gs}


# --------------------------------------------------------------------- work
NODE_FLOPS = 420.0  # additions and multiplications of one node update in pair-sum form


def _pop_bytes(storage):
    return lbmx.bytes_per_cell(storage) / 2.0


def _net_layers(m):
    c = (16, 32, 64, 96)
    return [(16, c[0], m), (c[0], c[0], m), (c[0], c[1], m // 2), (c[1], c[1], m // 2),
            (c[1], c[2], m // 4), (c[2], c[2], m // 4), (c[2], c[3], m // 8), (c[3], c[3], m // 8),
            (c[3] + c[2], c[2], m // 4), (c[2], c[2], m // 4), (c[2] + c[1], c[1], m // 2),
            (c[1], c[1], m // 2), (c[1] + c[0], c[0], m), (c[0], c[0], m), (c[0], 16, m)]


def work(case):
    """A pass's state or tensors read once and its results written once (for
    the steps of a cavity: the state in and out once, and the fields), and the
    arithmetic of the method."""
    kind = case["kind"]
    if kind == "cavity":
        v = float(case["n"]) ** 3
        return {"bytes": v * (2.0 * _pop_bytes(case["storage"]) + 40.0),
                "flops": v * NODE_FLOPS * case["steps"]}
    if kind == "batch":
        v = float(sum(c["n"] ** 3 for c in inputs.batch_cases(case["batch_seed"], case["count"])))
        return {"bytes": v * 2.0 * _pop_bytes(case["storage"]) + case["count"] * 16.0 * 64 ** 3,
                "flops": v * NODE_FLOPS * case["steps"]}
    if kind == "start":
        v, p = float(case["n"]) ** 3, _pop_bytes(case["storage"])
        src = {"cavity": p * case["m"] ** 3, "two": p * (case["m"] ** 3 + max(8, case["m"] // 2) ** 3),
               "fields": 16.0 * 64 ** 3}[case["how"]]
        return {"bytes": src + v * (p + 40.0), "flops": v * 500.0}
    if kind in ("train", "predict"):
        B, m = case["B"], case["m"]
        layers = _net_layers(m)
        par = sum(27.0 * ci * co + co for ci, co, _ in layers)
        mac = sum(27.0 * ci * co * r ** 3 * B for ci, co, r in layers)
        if kind == "predict":
            return {"bytes": 2.0 * par + 4.0 * B * m ** 3 * (4 if B == 1 else 16), "flops": 2.0 * mac}
        first = 27.0 * layers[0][0] * layers[0][1] * m ** 3 * B  # no data gradient of the first layer
        return {"bytes": 24.0 * par + 16.0 * B * m ** 3, "flops": 2.0 * (3.0 * mac - first)}
    v = float(case["B"] * case["D"] * case["H"] * case["W"])
    co = case["co"]
    if kind == "conv":
        ci = case["ci"]
        # x, output gradient and gate in; z, a and the data gradient out
        return {"bytes": 2.0 * v * (3 * ci + 3 * co) + 8.0 * 27 * ci * co, "flops": 6.0 * 27 * ci * co * v}
    cu, cs = case["cu"], case["cs"]
    ci = cu + cs
    return {"bytes": 2.0 * v * (cu / 8.0 + cs + ci + 3 * co) + 8.0 * 27 * ci * co,
            "flops": 6.0 * 27 * ci * co * v}


# -------------------------------------------------------------------- exact
E19 = [(0, 0, 0), (1, 0, 0), (-1, 0, 0), (0, 1, 0), (0, -1, 0), (0, 0, 1), (0, 0, -1), (1, 1, 0), (-1, 1, 0),
       (1, -1, 0), (-1, -1, 0), (1, 0, 1), (-1, 0, 1), (1, 0, -1), (-1, 0, -1), (0, 1, 1), (0, -1, 1),
       (0, 1, -1), (0, -1, -1)]
E7 = E19[:7]
W19 = [1 / 3] + [1 / 18] * 6 + [1 / 36] * 12
W7 = [1 / 4] + [1 / 8] * 6


def _moment_rows():
    """The moment polynomials of Eqs. (21)-(22) on the D3Q19 velocities."""
    rows = []
    for x, y, z in E19:
        s = x * x + y * y + z * z
        rows.append([1, 19 * s - 30, (21 * s * s - 53 * s + 24) / 2, x, (5 * s - 9) * x, y, (5 * s - 9) * y, z,
                     (5 * s - 9) * z, 3 * x * x - s, (3 * s - 5) * (3 * x * x - s), y * y - z * z,
                     (3 * s - 5) * (y * y - z * z), x * y, y * z, x * z, (y * y - z * z) * x,
                     (z * z - x * x) * y, (x * x - y * y) * z])
    return torch.tensor(rows, dtype=torch.float64, device="cuda").T.contiguous()


class _Exact:
    """The double-MRT cavity in 64 bits: dense moment matrices, collision, then
    streaming with half-way bounce-back and the thermal wall rules."""

    def __init__(self, n, wall_type, ra, ma=0.1, pr=0.71):
        self.n, self.wt = n, wall_type
        self.u_c = ma * math.sqrt(1 / 3)
        nu = self.u_c * n * math.sqrt(pr / ra)
        self.gb = self.u_c ** 2 / n
        sn, tau = 1 / (3 * nu + 0.5), 0.5 + 4 * nu / pr
        S = [1.0, 1.19, 1.4, 1.0, 1.2, 1.0, 1.2, 1.0, 1.2, sn, 1.4, sn, 1.4, sn, sn, sn, 1.98, 1.98, 1.98]
        M = _moment_rows()
        self.M = M
        self.MS = torch.linalg.inv(M) @ torch.diag(torch.tensor(S, dtype=torch.float64, device="cuda"))
        N = torch.tensor([[1] * 7, [e[0] for e in E7], [e[1] for e in E7], [e[2] for e in E7],
                          [6] + [-1] * 6, [0, 2, 2, -1, -1, -1, -1], [0, 0, 0, 1, 1, -1, -1]],
                         dtype=torch.float64, device="cuda")
        Q = torch.diag(1 / torch.tensor([1.0, tau, tau, tau, 1, 1, 1], dtype=torch.float64, device="cuda"))
        self.N, self.NQ = N, torch.linalg.inv(N) @ Q

    def set_fields(self, rho, u, th):
        """Equilibrium state of fields [n, n, n] (z, y, x)."""
        uu = sum(c * c for c in u)
        eu = lambda e: sum(k * c for k, c in zip(e, u) if k) + 0 * uu  # noqa: E731
        self.f = torch.stack([w * ((rho - 1) + rho * (3 * eu(e) + 4.5 * eu(e) ** 2 - 1.5 * uu)) + w
                              for e, w in zip(E19, W19)])
        self.g = torch.stack([w * th * (1 + 4 * eu(e)) for e, w in zip(E7, W7)])

    def macro(self):
        rho = self.f.sum(0)
        j = [sum(e[k] * self.f[i] for i, e in enumerate(E19) if e[k]) for k in range(3)]
        return rho, [c / rho for c in j], self.g.sum(0)

    def _stream(self, p, E, wall):
        """Pull: out_i(x) = p_i(x - e_i) inside, wall(i, opposite, slab) outside."""
        n, out = self.n, torch.empty_like(p)
        for i, e in enumerate(E):
            opp = E.index(tuple(-k for k in e))
            to, fr = [], []
            for k in (2, 1, 0):  # tensor axes z, y, x
                to.append(slice(max(e[k], 0), n + min(e[k], 0)))
                fr.append(slice(max(-e[k], 0), n + min(-e[k], 0)))
            out[i][tuple(to)] = p[i][tuple(fr)]
            for k in range(3):
                if e[k]:
                    at = [slice(None)] * 3
                    at[2 - k] = 0 if e[k] > 0 else n - 1
                    out[i][tuple(at)] = wall(i, e, k, p[opp][tuple(at)])
        return out

    def step(self):
        n = self.n
        rho, u, th = self.macro()
        j = [c * rho for c in u]
        jx, jy, jz = j
        jj = jx * jx + jy * jy + jz * jz
        o = torch.zeros_like(rho)
        p1, p2 = 2 * jx * jx - jy * jy - jz * jz, jy * jy - jz * jz
        meq = torch.stack([rho, -11 * rho + 19 * jj, 3 * rho - 5.5 * jj, jx, -2 / 3 * jx, jy, -2 / 3 * jy, jz,
                           -2 / 3 * jz, p1, -0.5 * p1, p2, -0.5 * p2, jx * jy, jy * jz, jx * jz, o, o, o])
        m = (self.M @ self.f.reshape(19, -1)).reshape(19, n, n, n)
        f = self.f - (self.MS @ (m - meq).reshape(19, -1)).reshape(19, n, n, n)
        G = self.gb * th
        uu = sum(c * c for c in u)
        for i, (e, w) in enumerate(zip(E19, W19)):
            eu = sum(k * c for k, c in zip(e, u) if k) + o
            f[i] += 3 * G * (e[2] - u[2]) * rho * w * (1 + 3 * eu + 4.5 * eu * eu - 1.5 * uu)
        neq = torch.stack([th, u[0] * th, u[1] * th, u[2] * th, 0.75 * th, o, o])
        k = (self.N @ self.g.reshape(7, -1)).reshape(7, n, n, n)
        g = self.g - (self.NQ @ (k - neq).reshape(7, -1)).reshape(7, n, n, n)
        ylin = 0.5 - (torch.arange(n, device="cuda", dtype=torch.float64) + 0.5) / n

        def twall(i, e, k, s):
            if k == 1:
                return -s + 2 * W7[i] * (0.5 if e[1] > 0 else -0.5)
            if (k == 0 and self.wt == 1) or (k == 2 and self.wt != 2):
                return s
            return -s + 2 * W7[i] * (ylin[None, :] if k == 0 else ylin[:, None])

        self.f = self._stream(f, E19, lambda i, e, k, s: s)
        self.g = self._stream(g, E7, twall)

    def read(self):
        rho, u, th = self.macro()
        n = self.n
        m = -n * (9 * th[:, 0, :] - th[:, 1, :] - 8 * 0.5) / 3
        line = m[:, n // 2] if n % 2 else 0.5 * (m[:, n // 2 - 1] + m[:, n // 2])
        return {"nu": [float(m.mean()), float(line.mean()), float(m.max())], "map": m.cpu().numpy(),
                **{k: v.cpu().numpy() for k, v in zip(("rho", "u", "v", "w", "theta"), (rho, *u, th))}}


def _resample(a, n):
    """Trilinear, node-centred, clamped at the outermost nodes."""
    m = a.shape[0]
    p = ((torch.arange(n, device="cuda", dtype=torch.float64) + 0.5) * m / n - 0.5).clamp(0, m - 1)
    i = p.floor().clamp(max=max(m - 2, 0)).long()
    fr = p - i
    i1 = (i + 1).clamp(max=m - 1)
    a = a.double()
    for ax in range(3):
        s = [1, 1, 1]
        s[ax] = n
        t = fr.reshape(s)
        a = a.index_select(ax, i) * (1 - t) + a.index_select(ax, i1) * t
    return a


def _start(n, wall_type, ra, fields):
    x = _Exact(n, wall_type, ra)
    r = [_resample(f, n) for f in fields]
    x.set_fields(torch.ones_like(r[0]), r[:3], r[3])
    return x


def _silu_grad(z):
    s = torch.sigmoid(z)
    return s * (1 + z * (1 - s))


class _Conv64(torch.autograd.Function):
    """3x3x3 convolution of channel-last x with w [co][27][ci], zero padding."""

    @staticmethod
    def _taps(x):
        B, D, H, W, C = x.shape
        p = torch.nn.functional.pad(x, (0, 0, 1, 1, 1, 1, 1, 1))
        for t in range(27):
            dz, dy, dx = t // 9, t // 3 % 3, t % 3
            yield t, p[:, dz:dz + D, dy:dy + H, dx:dx + W].reshape(-1, C)

    @staticmethod
    def forward(ctx, x, w):
        ctx.save_for_backward(x, w)
        out = 0
        for t, xs in _Conv64._taps(x):
            out = out + xs @ w[:, t].T
        return out.reshape(*x.shape[:4], w.shape[0])

    @staticmethod
    def backward(ctx, g):
        x, w = ctx.saved_tensors
        g2 = g.reshape(-1, g.shape[-1])
        gw = torch.stack([g2.T @ xs for _, xs in _Conv64._taps(x)], 1)
        gx = 0
        for t, gs in _Conv64._taps(g):
            gx = gx + gs @ w[:, 26 - t]
        return gx.reshape(x.shape), gw


def _up(x):
    return x.repeat_interleave(2, 1).repeat_interleave(2, 2).repeat_interleave(2, 3)


def _net64(case, log10_ra, wall_type):
    """The network in 64 bits from its BF16 weights; returns (prediction,
    parameters as FP64 leaves: weights, biases)."""
    z = np.load(WEIGHTS, allow_pickle=False)
    m, B = case["m"], case["B"]
    w = [torch.tensor(z["w%d" % k], device="cuda").bfloat16().double().requires_grad_() for k in range(15)]
    b = [torch.tensor(z["b%d" % k], device="cuda").double().requires_grad_() for k in range(15)]
    ax = (2.0 * torch.arange(m, device="cuda", dtype=torch.float64) + 1.0) / m - 1.0
    ch = [torch.zeros(B, m, m, m, dtype=torch.float64, device="cuda") for _ in range(16)]
    for q in range(B):
        ch[0][q] = (log10_ra[q] - 4.5) / 1.5
        ch[int(wall_type[q])][q] = 1.0
    ch[4] = ch[4] + ax[None, None, None, :]
    ch[5] = ch[5] + ax[None, None, :, None]
    ch[6] = ch[6] + ax[None, :, None, None]
    h, k, skips = torch.stack(ch, -1).bfloat16().double(), 0, []
    act = torch.nn.functional.silu

    def block(h, k):
        for q in (k, k + 1):
            h = act(_Conv64.apply(h, w[q]) + b[q])
        return h

    for lvl in range(4):
        h = block(h, 2 * lvl)
        if lvl < 3:
            skips.append(h)
            h = h.reshape(B, h.shape[1] // 2, 2, h.shape[2] // 2, 2, h.shape[3] // 2, 2, -1).mean((2, 4, 6))
    for lvl in range(3):
        h = block(torch.cat([_up(h), skips.pop()], -1), 8 + 2 * lvl)
    return (_Conv64.apply(h, w[14]) + b[14]).reshape(B, m ** 3, 16), w, b


def exact(case, seed):
    kind = case["kind"]
    if kind == "cavity":
        if case["n"] ** 3 * case["steps"] > 1.2e9:
            return None
        x = _start(case["n"], case["wall_type"], case["ra"], _smooth_fields(48, seed))
        for _ in range(case["steps"]):
            x.step()
        return x.read()
    if kind == "start":
        n, how = case["n"], case["how"]
        if how == "fields":
            return _start(n, 1, 1e5, _smooth_fields(64, seed)).read()
        rho, u, th = _start(case["m"], 1, 1e5, _smooth_fields(48, seed)).macro()
        f = [_resample(t, n) for t in (rho - 1, *u, th)]
        if how == "two":
            rho, u, th = _start(max(8, case["m"] // 2), 1, 1e5, _smooth_fields(48, seed + 1)).macro()
            f = [1.25 * a - 0.25 * _resample(t, n) for a, t in zip(f, (rho - 1, *u, th))]
        x = _Exact(n, 1, 1e5)
        x.set_fields(1 + f[0], f[1:4], f[4])
        return x.read()
    if kind == "predict":
        lr, wt = _net_inputs(case, seed)
        with torch.no_grad():
            pred = _net64(case, lr, wt)[0]
        if case["B"] > 1:
            return pred
        scale = torch.tensor(np.load(WEIGHTS, allow_pickle=False)["scale"], device="cuda").double()
        return (pred[0, :, :4] * scale).T.contiguous()
    if kind == "train":
        lr, wt = _net_inputs(case, seed)
        pred, w, b = _net64(case, lr, wt)
        loss = (pred[:, :, :4] - _target(case, seed).double()).square().mean()
        loss.backward()
        z = np.load(WEIGHTS, allow_pickle=False)
        mom = iter(_moments(seed))
        out = {"loss": loss.detach(), "w": [], "b": []}
        for k in range(15):
            for name, p in (("w", w[k]), ("b", b[k])):
                m, v = (t.double() for t in next(mom))
                g = p.grad
                m, v = 0.9 * m + 0.1 * g, 0.999 * v + 0.001 * g * g
                m, v = m / (1 - 0.9 ** (STEP + 1)), v / (1 - 0.999 ** (STEP + 1))
                old = torch.tensor(z["%s%d" % (name, k)], device="cuda").double()
                out[name].append(old - LR * m / (v.sqrt() + 1e-8))
        return out
    if kind == "batch":
        return None
    t = {k: v.double() for k, v in _layer(case, seed).items()}
    x = torch.cat([_up(t["low"]), t["skip"]], -1) if kind == "upcat" else t["x"]
    x, w = x.requires_grad_(), t["w"].requires_grad_()
    y = _Conv64.apply(x, w)
    y.backward(t["gz"])
    z = y.detach() + t["b"]
    out = {"z": z, "a": torch.nn.functional.silu(z), "gw": w.grad, "gb": t["gz"].sum((0, 1, 2, 3))}
    if kind == "conv":
        out["gx"] = x.grad * _silu_grad(t["zprev"])
    else:
        out["gu"], out["gs"] = x.grad[..., :case["cu"]], x.grad[..., case["cu"]:]
    return out
