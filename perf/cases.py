"""Performance cases: what a user of this framework has it do, with the exact
answers in 64 bits.

Three families.  ``solve``: one topology-optimization iteration of a single
FDTD context (set the density, forward solve, adjoint solve, gradient), 2D
TMz, 2D TEz and 3D, FP32 and FP64, with the full history or checkpoints.
``batch``: the same for uneven 2D instances advanced together.  ``design``:
the work between two solves (open-close filter, its transpose, statistics,
one MMA step).  ``unet`` and ``layer``: the surrogate network's training step
and inference, and one 3x3 convolution layer forward and backward.
"""
import math

import numpy as np
import torch

import fdtd_workloads as W
import paper_2203_01462_amd as P
from paper_2203_01462_amd import design, nn

C0, MU0 = 299792458.0, 4.0e-7 * math.pi
EPS0 = 1.0 / (MU0 * C0 * C0)
EXACT_STEPS = {"tmz": 2.0e9, "te": 2.0e9, "3d": 6.0e8}  # node-steps beyond which exact() takes too long


def listed():
    return [
        # the small 2D case of the benchmark, where launches and latency count
        dict(name="tmz_200_f64", kind="solve", mode="tmz", nx=200, ny=200, nz=1, prec=64, steps=2000, pml=20, box=60,
             boxz=1, gap=1, ckpt=0, t0=4.0, freqs=8),
        # the grid of the surrogate-guided design runs (128 x 128 design box)
        dict(name="tmz_512_f32", kind="solve", mode="tmz", nx=512, ny=512, nz=1, prec=32, steps=2500, pml=16, box=128,
             boxz=1, gap=3, ckpt=0, t0=3.0, freqs=8),
        # an odd, non-square grid with damping, checkpointed (history that must not grow with the steps)
        dict(name="tmz_333x517_f32_ckpt", kind="solve", mode="tmz", nx=333, ny=517, nz=1, prec=32, steps=1500, pml=13,
             box=77, boxz=1, gap=3, ckpt=250, t0=2.5, freqs=5),
        # the large 2D benchmark grid, until the pulse is over the gap
        dict(name="tmz_2048_f32", kind="solve", mode="tmz", nx=2048, ny=2048, nz=1, prec=32, steps=5000, pml=32,
             box=512, boxz=1, gap=5, ckpt=0, t0=3.0, freqs=16),
        # in-plane polarization (one density per edge), a paper-sized design and a larger one
        dict(name="te_384_f32", kind="solve", mode="te", nx=384, ny=384, nz=1, prec=32, steps=2400, pml=16, box=96,
             boxz=1, gap=6, ckpt=0, t0=3.0, freqs=16),
        dict(name="te_1024_f32", kind="solve", mode="te", nx=1024, ny=1024, nz=1, prec=32, steps=1600, pml=32, box=256,
             boxz=1, gap=5, ckpt=0, t0=2.0, freqs=16),
        # 3D: a medium FP64 grid, and the first steps of the 256^3 benchmark
        dict(name="yee3d_80_f64", kind="solve", mode="3d", nx=80, ny=80, nz=80, prec=64, steps=600, pml=6, box=20,
             boxz=10, gap=2, ckpt=0, t0=2.0, freqs=8),
        dict(name="yee3d_256_f32", kind="solve", mode="3d", nx=256, ny=256, nz=256, prec=32, steps=500, pml=16,
             box=128, boxz=32, gap=4, ckpt=0, t0=2.0, freqs=16),
        # uneven instances together (a data-generation batch of the surrogate, a parameter scan)
        dict(name="batch_16", kind="batch", count=16, steps=1000, prec=32, sides="128,256,512,1024", config=0),
        # between two solves of a design loop on the 512^2 workload
        dict(name="design_128", kind="design", nx=128, ny=128, nz=1, prec=32, radius=2.5, alpha=1.0),
        # the surrogate: a training step at the benchmark's batch
        dict(name="unet_train_128_b32", kind="unet", side=128, batch=32, train=True),
        # one convolution layer on ragged images and channel counts
        dict(name="layer_ragged", kind="layer", n=4, cin=48, cout=80, h=50, w=75),
    ]


def _between(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["tmz", "tmz", "tmz", "te", "3d", "3d", "batch", "design", "unet", "layer", "layer"])
    if kind in ("tmz", "te"):
        nx = _between(rng, 96, 1600)
        ny = max(96, min(1600, int(nx * rng.uniform(0.6, 1.6))))
        prec = rng.choice([32, 32, 64])
        pml = rng.randint(6, max(8, min(32, min(nx, ny) // 10)))
        box = rng.randint(12, min(nx, ny) // 3)
        steps = int(max(200, min(2500, 3.0e9 / (nx * ny * (prec // 32)))))
        return dict(kind="solve", mode=kind, nx=nx, ny=ny, nz=1, prec=prec, steps=steps + rng.randint(0, 40), pml=pml,
                    box=box, boxz=1, gap=rng.randint(1, 6), ckpt=rng.choice([0, 0, steps // 5]) if kind == "tmz" else 0,
                    t0=rng.uniform(1.5, 2.5), freqs=rng.randint(1, 16))
    if kind == "3d":
        nx, ny, nz = (_between(rng, 48, 160) for _ in range(3))
        prec = rng.choice([32, 32, 64])
        box = rng.randint(8, min(nx, ny) // 3)
        steps = int(max(100, min(600, 4.0e8 / (nx * ny * nz * (prec // 32)))))
        return dict(kind="solve", mode="3d", nx=nx, ny=ny, nz=nz, prec=prec, steps=steps + rng.randint(0, 20),
                    pml=rng.randint(5, 10), box=box, boxz=rng.randint(4, 12), gap=rng.randint(1, 3),
                    ckpt=rng.choice([0, 0, 60]), t0=1.5, freqs=rng.randint(1, 16))
    if kind == "batch":
        return dict(kind="batch", count=rng.randint(3, 16), steps=rng.randint(300, 900), prec=rng.choice([32, 32, 64]),
                    sides=rng.choice(["128,256", "96,160,320", "128,256,512", "128,256,512,1024"]),
                    config=rng.randint(1, 99))
    if kind == "design":
        if rng.random() < 0.3:
            return dict(kind="design", nx=rng.randint(20, 128), ny=rng.randint(20, 128), nz=rng.randint(4, 32),
                        prec=rng.choice([32, 64]), radius=rng.choice([1.5, 2.5, 3.2]), alpha=rng.choice([0.05, 0.3, 1.0, 64.0]))
        return dict(kind="design", nx=_between(rng, 40, 512), ny=_between(rng, 40, 512), nz=1, prec=rng.choice([32, 64]),
                    radius=rng.choice([1.5, 2.5, 4.0, 7.5]), alpha=rng.choice([0.05, 0.3, 1.0, 64.0]))
    if kind == "unet":
        train = rng.random() < 0.5
        return dict(kind="unet", side=8 * rng.randint(6, 16), batch=_between(rng, 1, 32), train=train)
    return dict(kind="layer", n=_between(rng, 1, 32), cin=_between(rng, 3, 256), cout=_between(rng, 1, 256),
                h=_between(rng, 12, 96), w=_between(rng, 12, 96))


# ---------------------------------------------------------------- workloads

def _workload(c):
    """The workload description of a ``solve`` case."""
    n = (c["nx"], c["ny"], c["nz"])
    three = c["mode"] == "3d"
    bz = c["boxz"] if three else 1
    box = (c["box"], c["box"], bz)
    gap = (c["gap"], c["gap"], c["gap"] if three else 1)
    lo = tuple((a - b) // 2 if k < 2 or three else 0 for k, (a, b) in enumerate(zip(n, box)))
    glo = tuple((a - b) // 2 if k < 2 or three else 0 for k, (a, b) in enumerate(zip(n, gap)))
    base = {"tmz": W.medium2d, "te": W.medium_te, "3d": W.medium3d}[c["mode"]]()
    return W.with_(base, name="case", precision=c["prec"], n=n, n_steps=c["steps"], dx=2e-9, pml_cells=c["pml"],
                   tfsf_margin=3 if three else 5, t0_over_tau=c["t0"], design_lo=lo, design_n=box, gap_lo=glo,
                   gap_n=gap, lambda_lo=500e-9, lambda_hi=1000e-9, n_freq=c["freqs"], gamma_mult=4.0)


def _batch_workloads(c):
    sides = tuple(int(s) for s in c["sides"].split(","))
    return [W.with_(w, precision=c["prec"]) for w in W.c4(count=c["count"], n_steps=c["steps"], seed=c["config"], sides=sides)]


def _dtype(c):
    return torch.float32 if c["prec"] == 32 else torch.float64


def _rho(w, seed, dtype):
    return torch.from_numpy(W.seeded_rho(w, seed)).to(dtype)


def _design_inputs(c, seed):
    g = torch.Generator().manual_seed(seed)
    shape = (c["nz"], c["ny"], c["nx"]) if c["nz"] > 1 else (c["ny"], c["nx"])
    dt = _dtype(c)
    x = torch.rand(shape, generator=g, dtype=torch.float64)
    grad = torch.randn(shape, generator=g, dtype=torch.float64) * 1e-2
    return x.to(dt), grad.to(dt)


def _unet_inputs(c, seed):
    g = torch.Generator().manual_seed(seed)
    b, s = c["batch"], c["side"]
    return torch.rand(b, s, s, generator=g), torch.randn(b, generator=g), torch.randn(b, s, s, generator=g)


def _layer_inputs(c, seed):
    """Channel-major activations, weights [cout][3][3][cin], the gradient of
    the output, all BF16; bias FP32."""
    g = torch.Generator().manual_seed(seed)
    n, ci, co, h, w = c["n"], c["cin"], c["cout"], c["h"], c["w"]
    bf = torch.bfloat16
    x = torch.relu(torch.randn(ci, n, h, w, generator=g)).to(bf)
    wt = (torch.randn(co, 3, 3, ci, generator=g) * math.sqrt(2.0 / (9 * ci))).to(bf)
    dz = torch.randn(co, n, h, w, generator=g).to(bf)
    return x, wt, torch.randn(co, generator=g), dz


# ---------------------------------------------------------------- the cases

def prepare(case, seed):
    k = case["kind"]
    if k == "solve":
        w = _workload(case)
        stream = torch.cuda.Stream()
        ctx = P.FDTD(w, stream=stream.cuda_stream, ckpt_every=case["ckpt"])
        with torch.cuda.stream(stream):
            rho = _rho(w, seed, _dtype(case)).cuda()
            grad = torch.empty_like(rho)
        stream.synchronize()
        return dict(kind=k, ctx=ctx, stream=stream, rho=rho, grad=grad)
    if k == "batch":
        ws = _batch_workloads(case)
        stream = torch.cuda.Stream()
        b = P.Batch(ws, stream=stream.cuda_stream)
        with torch.cuda.stream(stream):
            rhos = [_rho(w, seed * 1000 + i, _dtype(case)).cuda() for i, w in enumerate(ws)]
            grads = [torch.empty_like(r) for r in rhos]
        stream.synchronize()
        return dict(kind=k, batch=b, stream=stream, rhos=rhos, grads=grads)
    if k == "design":
        stream = torch.cuda.Stream()
        with torch.cuda.stream(stream):
            x, g = (t.cuda() for t in _design_inputs(case, seed))
            filt = design.Filter(tuple(x.shape), case["radius"], x.dtype)
            mma = design.MMA(x.numel(), x.dtype)
            bufs = [torch.empty_like(x) for _ in range(3)]
        stream.synchronize()
        return dict(kind=k, stream=stream, x=x, g=g, filt=filt, mma=mma, bufs=bufs, alpha=case["alpha"])
    if k == "unet":
        net = nn.UNet(case["side"], case["batch"], seed=7)
        return dict(kind=k, net=net, train=case["train"], inputs=[t.cuda() for t in _unet_inputs(case, seed)])
    x, wt, bias, dz = _layer_inputs(case, seed)
    s = dict(case, x=x.cuda().view(torch.int16), wt=wt.cuda().view(torch.int16), bias=bias.cuda(),
             dz=dz.cuda().view(torch.int16))
    n, ci, co, h, w = (case[v] for v in ("n", "cin", "cout", "h", "w"))
    s.update(a=torch.empty(co, n, h, w, dtype=torch.int16, device="cuda"),
             dza=torch.empty(ci, n, h, w, dtype=torch.int16, device="cuda"),
             wrot=torch.empty(ci * co * 9, dtype=torch.int16, device="cuda"),
             dw=torch.empty(co, 3, 3, ci, device="cuda"), db=torch.empty(co, device="cuda"),
             work=torch.empty(max(nn.wgrad_work(n, ci, co, h, w), 1), device="cuda"))
    return s


def run(s):
    k = s["kind"]
    if k == "solve":
        ctx = s["ctx"]
        ctx.set_density(s["rho"])
        F = ctx.forward()
        ctx.adjoint()
        return {"F": F, "grad": ctx.gradient(s["grad"])}
    if k == "batch":
        b = s["batch"]
        for i, r in enumerate(s["rhos"]):
            b.set_density(i, r)
        F = b.forward()
        b.adjoint()
        return {"F": F, "grad": [b.gradient(i, g) for i, g in enumerate(s["grads"])]}
    if k == "design":
        with torch.cuda.stream(s["stream"]):
            x, g, (rf, gv, xn) = s["x"], s["g"], s["bufs"]
            s["filt"].apply(x, s["alpha"], out=rf)
            s["filt"].transpose(g, out=gv)
            zeta, kkt = design.stats(rf, gv)
            rho0 = s["mma"].begin(x, -1.0, gv)
            approx, dist = s["mma"].solve(rho0, xn)
        return {"filtered": rf, "gradient": gv, "xnew": xn, "scalars": [zeta, kkt, rho0, approx, dist]}
    if k == "unet":
        net, (rho, Ft, St) = s["net"], s["inputs"]
        F, S = net.forward(rho)
        if not s["train"]:
            return {"F": F, "S": S}
        net.backward(*net.loss_grad(Ft, St))
        # a whole training step; at rate 0, as in the first step of a warm-up,
        # the weights stay and a pass can be repeated
        net.step(0.0)
        return {"F": F, "S": S, "loss": net.loss, "grad": net.g}
    n, ci, co, h, w = (s[v] for v in ("n", "cin", "cout", "h", "w"))
    nn.conv3x3(s["x"], s["wt"], s["bias"], n, ci, co, h, w, a=s["a"])
    nn.conv3x3_wgrad(s["x"], s["dz"], s["dw"], s["db"], s["work"], n, ci, co, h, w)
    nn.conv3x3_dgrad_relu(s["dz"], s["wt"], s["wrot"], s["x"], s["dza"], n, ci, co, h, w)
    return {"a": s["a"].view(torch.bfloat16), "dza": s["dza"].view(torch.bfloat16), "dw": s["dw"], "db": s["db"]}


def _solve_work(w):
    """Updates of every node in every step of both solves; densities and
    gradients, and the forward field on the design edges, written by the
    forward solve and read by the adjoint."""
    esz = w["precision"] // 8
    cells = w["n"][0] * w["n"][1] * (w["n"][2] if w["dims"] == 3 else 1)
    nd = int(np.prod(W.design_shape(w)))
    comps = 3 if w["dims"] == 3 else 1
    return dict(flops=cells * w["n_steps"] * 2 * (36 if w["dims"] == 3 else 10),
                bytes=2 * nd * esz + 2 * w["n_steps"] * nd * comps * esz)


def work(case):
    k = case["kind"]
    if k == "solve":
        return _solve_work(_workload(case))
    if k == "batch":
        ws = [_solve_work(w) for w in _batch_workloads(case)]
        return {q: sum(v[q] for v in ws) for q in ("flops", "bytes")}
    if k == "design":
        n, esz, r = case["nx"] * case["ny"] * case["nz"], case["prec"] // 8, case["radius"]
        taps = math.pi * r * r if case["nz"] == 1 else 4 / 3 * math.pi * r ** 3
        return dict(bytes=5 * n * esz, flops=n * (8 * 2 * taps + 60))
    if k == "unet":
        s, b = case["side"], case["batch"]
        plan = nn.layer_plan()
        macs = sum(ci * 9 * co * (s >> l) ** 2 for ci, co, l in plan) * b
        params = sum(ci * 9 * co + co for ci, co, _ in plan) + 257
        if not case["train"]:
            return dict(flops=2 * macs, bytes=2 * 4 * b * s * s + 2 * params)
        return dict(flops=6 * macs, bytes=3 * 4 * b * s * s + params * (2 + 2 + 8 * 4))
    n, ci, co, hw = case["n"], case["cin"], case["cout"], case["h"] * case["w"]
    return dict(flops=3 * 2 * n * ci * 9 * co * hw, bytes=2 * (2 * n * ci * hw + 2 * n * co * hw) + ci * co * 9 * 6)


# ---------------------------------------------------------------- 64 bits

def _device():
    return "cuda" if torch.cuda.is_available() else "cpu"


def _grade(w, dt, n, half):
    """(b, a, 1/kappa) of the absorber at the n positions of one axis."""
    P_, x = w["pml_cells"], np.arange(n) + (0.5 if half else 0.0)
    d = np.maximum(np.maximum(P_ - x, x - (n - 1 - P_)) / P_, 0.0) if P_ else np.zeros(n)
    return _grade_depth(w, dt, d)


def _grade_depth(w, dt, d):
    m, eta = w["pml_order"], math.sqrt(MU0 / (EPS0 * w["eps_s"]))
    sig = w["pml_sigma_scale"] * 0.8 * (m + 1) / (eta * w["dx"]) * d ** m
    kap, alp = 1 + (w["pml_kappa_max"] - 1) * d ** m, w["pml_alpha_max"] * (1 - d)
    b = np.where(d > 0, np.exp(-(sig / kap + alp) * dt / EPS0), 1.0)
    with np.errstate(invalid="ignore"):
        a = np.where(sig > 0, sig * (b - 1) / (sig * kap + kap * kap * alp), 0.0)
    return b, a, np.where(d > 0, 1 / kap, 1.0)


def _wave(w, t):
    fl, fh = C0 / w["lambda_hi"], C0 / w["lambda_lo"]
    tau = math.sqrt(math.log(2.0)) / (math.pi * 0.5 * (fh - fl))
    t = t - w["t0_over_tau"] * tau
    return w["amplitude"] * np.sin(math.pi * (fl + fh) * t) * np.exp(-(t / tau) ** 2)


def _line(w, dt, g, L):
    """The one-dimensional incident wave: E at the nodes, H between them."""
    n1, N, ch, ce = L + 21, w["n_steps"], dt / (MU0 * w["dx"]), dt / (EPS0 * w["eps_s"] * w["dx"])
    pos = np.arange(n1) - (n1 - 21.0)
    be, ae, ke = _grade_depth(w, dt, np.maximum(pos / 20, 0))
    bh, ah, kh = (v[:-1] for v in _grade_depth(w, dt, np.maximum((pos + 0.5) / 20, 0)))
    e, h, pe, ph = np.zeros(n1), np.zeros(n1 - 1), np.zeros(n1), np.zeros(n1 - 1)
    E, H = np.zeros((N + 1, L)), np.zeros((N, L))
    e[0] = g[0]
    E[0] = e[:L]
    for n in range(N):
        d = e[1:] - e[:-1]
        ph = bh * ph + ah * d
        h = h - ch * (d * kh + ph)
        H[n] = h[:L]
        d = h[1:] - h[:-1]
        pe[1:-1] = be[1:-1] * pe[1:-1] + ae[1:-1] * d
        e[1:-1] -= ce * (d * ke[1:-1] + pe[1:-1])
        e[0], e[-1] = g[n + 1], 0.0
        E[n + 1] = e[:L]
    return E, H


class _Yee:
    """The discrete problem in plain torch: full-size arrays [z][y][x] per
    field component, one step as a differentiable function of the density."""

    def __init__(self, w):
        self.w, three, te = w, w["dims"] == 3, W.is_te(w)
        nx, ny, nz = w["n"] if three else (*w["n"][:2], 1)
        self.n, self.shape, dev = (nx, ny, nz), (nz, ny, nx), _device()
        self.Ec, self.Hc = ((0, 1, 2), (0, 1, 2)) if three else ((0, 1), (2,)) if te else ((2,), (0, 1))
        self.axes = (0, 1, 2) if three else (0, 1)
        pol, prop = (0, 2) if three else (0, 1) if te else (2, 1)
        dt = self.dt = w["courant"] * w["dx"] / C0
        f64 = dict(dtype=torch.float64, device=dev)
        idx = [torch.arange(self.n[a], device=dev).reshape([-1 if 2 - a == d else 1 for d in range(3)]) for a in range(3)]

        def box(lo, hi):  # nodes lo[a] <= x <= hi[a] on the active axes
            m = torch.ones(self.shape, dtype=torch.bool, device=dev)
            for a in self.axes:
                m = m & (idx[a] >= lo[a]) & (idx[a] <= hi[a])
            return m

        self.vE = {c: box([0 if a == c else 1 for a in range(3)], [v - 2 for v in self.n]).double() for c in self.Ec}
        self.vH = {c: box([1 if a == c else 0 for a in range(3)], [v - 2 for v in self.n]).double() for c in self.Hc}
        self.tab = {}
        for a in self.axes:
            for kind in (0, 1):
                self.tab[a, kind] = [torch.tensor(v, **f64).reshape([-1 if 2 - a == d else 1 for d in range(3)])
                                     for v in _grade(w, dt, self.n[a], kind == 1)]
        # curl terms: (component, axis of the difference, other component, sign)
        self.curlE = [(a, b, c, s) for a in self.Hc for b, c, s in (((a + 1) % 3, (a + 2) % 3, 1), ((a + 2) % 3, (a + 1) % 3, -1))
                      if c in self.Ec and b in self.axes]
        self.curlH = [(a, b, c, s) for a in self.Ec for b, c, s in (((a + 1) % 3, (a + 2) % 3, 1), ((a + 2) % 3, (a + 1) % 3, -1))
                      if c in self.Hc and b in self.axes]
        # total-field box and the incident wave
        lo = [w["pml_cells"] + w["tfsf_margin"]] * 3
        hi = [v - 1 - lo[0] for v in self.n]
        self.g = _wave(w, np.arange(w["n_steps"] + 2) * dt)
        self.ref, L = lo[prop] - 2, hi[prop] - lo[prop] + 5
        self.einc, self.hinc = (torch.tensor(v, **f64) for v in _line(w, dt, self.g, L))
        self.pol, self.mag, self.prop = pol, 3 - pol - prop, prop
        self.msign = 1.0 if (self.mag + 1) % 3 == prop else -1.0
        tE = box(lo, [hi[a] - (a == pol) for a in range(3)]).double()
        tH = {c: box(lo, [hi[a] - (a != c) for a in range(3)]).double() for c in self.Hc}
        tEc = {c: box(lo, [hi[a] - (a == c) for a in range(3)]).double() for c in self.Ec}
        self.line_at = (idx[prop] - self.ref).clamp(0, L - 1)
        # scattered H beside total E, total E beside scattered H
        self.cH = {(a, b): ((1 - tH[a]), tE) for a, b, c, _ in self.curlE if c == pol}
        self.cE = {(a, b): (tEc[a], 1 - tH[self.mag]) for a, b, c, _ in self.curlH if c == self.mag}
        # design edges, gap edges
        d0, dn, g0, gn = w["design_lo"], w["design_n"], w["gap_lo"], w["gap_n"]
        ext = (lambda c, n0: [n0[a] + (1 if te and a != c else 0) for a in range(3)])
        self.gap = {c: box(g0, [g0[a] + e - 1 for a, e in enumerate(ext(c, gn))]) for c in self.Ec}
        inside = {c: box(d0, [d0[a] + e - 1 for a, e in enumerate(ext(c, dn))]) for c in self.Ec}
        self.des, self.rho_at, off = {}, {}, 0
        for c in self.Ec:
            k = torch.zeros(self.shape, dtype=torch.long, device=dev)
            cnt = int(inside[c].sum())
            k[inside[c]] = torch.arange(off, off + cnt, device=dev)
            if te:
                off += cnt
            self.des[c], self.rho_at[c] = inside[c] & ~self.gap[c], k
        self.gap_at = {c: torch.nonzero(self.gap[c].reshape(-1)).reshape(-1) for c in self.Ec}
        # objective weights and phasors
        fl, fh, K = C0 / w["lambda_hi"], C0 / w["lambda_lo"], w["n_freq"]
        f = np.array([0.5 * (fl + fh)]) if K == 1 else fl + (fh - fl) * np.arange(K) / (K - 1)
        n = np.arange(1, w["n_steps"] + 1)
        ph = np.exp(-2j * np.pi * f[:, None] * n * dt) * dt
        wk = 1.0 / np.abs(ph @ self.g[1:w["n_steps"] + 1]) ** 2
        self.ph = [torch.tensor(v, **f64) for v in (ph.real, ph.imag)]
        self.wk = torch.tensor(wk, **f64)

    def coefficients(self, rho):
        w, dt = self.w, self.dt
        psi, gam = w["omega_p"] ** 2, w["gamma_mult"] * w["gamma_p"]
        psis, den, r = w["psi_s_ratio"] * psi, 1 + gam * dt / 2, rho.reshape(-1)
        beta = EPS0 * (psis + (psi - psis) * r) * dt / 2 / den
        bs = beta * dt + w["sigma_max"] * dt * r * (1 - r)
        inv = 2 / (2 * EPS0 * (w["eps_s"] + (w["eps_inf"] - w["eps_s"]) * r) + bs)
        self.kpm1, dthJ = -gam * dt / den, dt * 0.5 * (1 + (1 - gam * dt / 2) / den)
        out = {}
        zero = torch.zeros((), dtype=torch.float64, device=rho.device)
        for c in self.Ec:
            m, k = self.des[c], self.rho_at[c]
            ce = dt / (EPS0 * w["dx"]) / torch.where(self.gap[c], zero + w["eps_g"], zero + w["eps_s"])
            out[c] = [torch.where(m, (inv * dt / w["dx"])[k], ce) * self.vE[c], torch.where(m, (inv * dthJ)[k], zero),
                      torch.where(m, (inv * bs)[k], zero), torch.where(m, beta[k], zero)]
        return out

    def start(self):
        def z():
            return torch.zeros(self.shape, dtype=torch.float64, device=_device())
        names = [("E", c) for c in self.Ec] + [("H", c) for c in self.Hc] + [("J", c) for c in self.Ec]
        names += [("pH", a, b) for a, b, _, _ in self.curlE] + [("pE", a, b) for a, b, _, _ in self.curlH]
        return {k: z() for k in names}

    def _diff(self, v, axis, back):
        d = 2 - axis
        pad = torch.zeros_like(v.narrow(d, 0, 1))
        return torch.diff(v, dim=d, prepend=pad) if back else torch.diff(v, dim=d, append=pad)

    def step(self, s, co, n):
        s = dict(s)
        ch = self.dt / (MU0 * self.w["dx"])
        einc, hinc = self.einc[n][self.line_at], self.msign * self.hinc[n][self.line_at]
        new = {c: s["H", c] for c in self.Hc}
        for kind, terms, corr, src in ((1, self.curlE, self.cH, einc), (0, self.curlH, self.cE, hinc)):
            if kind == 0:
                curl = {c: 0.0 for c in self.Ec}
            for a, b, c, sign in terms:
                bb, aa, ik = self.tab[b, kind]
                key = ("pH" if kind else "pE", a, b)
                d = self._diff(s["E" if kind else "H", c], b, kind == 0)
                s[key] = (bb * s[key] + aa * d) * (self.vH[a] if kind else self.vE[a])
                t = d * ik + s[key]
                if (a, b) in corr and c == (self.pol if kind else self.mag):
                    m, m2 = corr[a, b]
                    t = t + (-1.0 if kind else 1.0) * m * self._diff(m2 * src, b, kind == 0)
                if kind:
                    new[a] = new[a] - sign * ch * t
                else:
                    curl[a] = curl[a] + sign * t
            if kind:
                for c in self.Hc:
                    s["H", c] = new[c] * self.vH[c]
        mon = []
        for c in self.Ec:
            c1, c2, c3, beta = co[c]
            e0, J = s["E", c], s["J", c]
            e1 = e0 + (c1 * curl[c] - c2 * J - c3 * e0)
            s["E", c], s["J", c] = e1, J + (self.kpm1 * J + beta * (e0 + e1))
            mon.append(e1.reshape(-1)[self.gap_at[c]])
        return s, torch.cat(mon)

    def solve(self, rho, seg=32):
        """(F, dF/drho): the forward solve, then the segments backwards."""
        N = self.w["n_steps"]
        rho = rho.to(_device()).double().requires_grad_(True)
        with torch.no_grad():
            co, s, saved, mon = self.coefficients(rho), self.start(), [], []
            for n in range(N):
                if n % seg == 0:
                    saved.append(s)
                s, m = self.step(s, co, n)
                mon.append(m)
        series = torch.stack(mon).requires_grad_(True)
        F = (self.wk[:, None] * ((self.ph[0] @ series) ** 2 + (self.ph[1] @ series) ** 2)).sum()
        gm = torch.autograd.grad(F, series)[0]
        gs, grad = {k: torch.zeros_like(v) for k, v in s.items()}, torch.zeros_like(rho)
        for q in range(len(saved) - 1, -1, -1):
            s0 = {k: v.detach().requires_grad_(True) for k, v in saved.pop().items()}
            co, s, tot = self.coefficients(rho), s0, 0.0
            for n in range(q * seg, min(N, (q + 1) * seg)):
                s, m = self.step(s, co, n)
                tot = tot + (m * gm[n]).sum()
            tot = tot + sum((v * gs[k]).sum() for k, v in s.items())
            got = torch.autograd.grad(tot, [rho, *s0.values()], allow_unused=True)
            grad += got[0]
            gs = {k: v if v is not None else torch.zeros_like(s0[k]) for k, v in zip(s0, got[1:])}
        return float(F.detach()), grad.detach()


def _filter64(x, r, alpha):
    """The open-close filter as a differentiable function."""
    three = x.dim() == 3
    x = x if three else x[None]
    R = int(math.ceil(r))
    taps = [(a, b, c, r - math.sqrt(a * a + b * b + c * c)) for a in range(-R if three else 0, (R if three else 0) + 1)
            for b in range(-R, R + 1) for c in range(-R, R + 1)]
    taps = [t for t in taps if t[3] > 0]

    def total(v):
        p = torch.nn.functional.pad(v, (R, R, R, R, R, R))
        s = torch.zeros_like(v)
        for a, b, c, wt in taps:
            s = s + wt * p[R + a:R + a + v.shape[0], R + b:R + b + v.shape[1], R + c:R + c + v.shape[2]]
        return s

    norm = total(torch.ones_like(x))
    for dual in (False, True, True, False):
        u = 1 - x if dual else x
        e = norm / total(1 / (u + alpha)) - alpha
        x = (1 - e if dual else e).clamp(0.0, 1.0)
    return x if three else x[0]


def _design64(c, x, g):
    x, g = x.to(_device()).double().requires_grad_(True), g.to(_device()).double()
    rf = _filter64(x, c["radius"], c["alpha"])
    gv = torch.autograd.grad((rf * g).sum(), x)[0]
    x, rf = x.detach(), rf.detach()
    zeta = float((4 * rf * (1 - rf)).mean())
    kkt = float((rf - (rf - gv).clamp(0, 1)).norm())
    rho0 = max(1e-6, 0.1 * float(gv.abs().mean()))
    L, U = x - 0.5, x + 0.5
    p = (U - x) ** 2 * (1.001 * gv.clamp(min=0) + 0.001 * (-gv).clamp(min=0) + rho0)
    q = (x - L) ** 2 * (0.001 * gv.clamp(min=0) + 1.001 * (-gv).clamp(min=0) + rho0)
    lo = torch.maximum((L + 0.1 * (x - L)).clamp(min=0.0), x - 0.5)
    hi = torch.minimum((U - 0.1 * (U - x)).clamp(max=1.0), x + 0.5)
    xn = (p.sqrt() * L + q.sqrt() * U) / (p.sqrt() + q.sqrt())
    xn = torch.minimum(torch.maximum(xn, lo), hi)
    approx = -1.0 + float((p / (U - xn) - p / (U - x) + q / (xn - L) - q / (x - L)).sum())
    dist = float(((U - L) * (xn - x) ** 2 / ((U - xn) * (xn - L))).sum())
    return {"filtered": rf, "gradient": gv, "xnew": xn, "scalars": [zeta, kkt, rho0, approx, dist]}


def _bf(t):
    return t.to(torch.bfloat16).double()


class _Store(torch.autograd.Function):
    """A value stored as BF16 (its gradient passes unrounded)."""

    @staticmethod
    def forward(ctx, x):
        return _bf(x)

    @staticmethod
    def backward(ctx, g):
        return g


class _Act(torch.autograd.Function):
    """BF16 ReLU output; the gradient before the ReLU is stored as BF16 too."""

    @staticmethod
    def forward(ctx, z):
        a = _bf(z.clamp(min=0))
        ctx.save_for_backward(a)
        return a

    @staticmethod
    def backward(ctx, g):
        return _bf(g * (ctx.saved_tensors[0] > 0))


class _Head(torch.autograd.Function):
    @staticmethod
    def forward(ctx, z):
        return z

    @staticmethod
    def backward(ctx, g):
        return _bf(g)


def _conv64(x, wt, bias):
    """x [c][n][h][w], wt [cout][3][3][cin]."""
    p = torch.nn.functional.pad(x, (1, 1, 1, 1))
    h, w = x.shape[2:]
    z = 0.0
    for ky in range(3):
        for kx in range(3):
            v = p[:, :, ky:ky + h, kx:kx + w].reshape(x.shape[0], -1)
            z = z + wt[:, ky, kx, :] @ v
    return z.reshape(-1, *x.shape[1:]) + (0.0 if bias is None else bias[:, None, None, None])


def _unet64(c, inputs):
    dev, s, n = _device(), c["side"], c["batch"]
    rho, Ft, St = (t.to(dev).double() for t in inputs)
    plan, ch = nn.layer_plan(), nn.CHANNELS
    offs, o = [], 0
    g = torch.Generator().manual_seed(7)
    for ci, co, _ in plan:
        o = (o + 7) // 8 * 8
        offs.append(o)
        o += co * ci * 9 + co
    p = torch.zeros(o + ch[-1] + 1, dtype=torch.float32)
    for (ci, co, _), ow in zip(plan, offs):
        p[ow:ow + co * ci * 9] = torch.randn(co * ci * 9, generator=g) * math.sqrt(2.0 / (ci * 9))
    p[o:o + ch[-1]] = torch.randn(ch[-1], generator=g) / math.sqrt(ch[-1])
    p[offs[-1]:offs[-1] + ch[0] * 9] *= 0.1
    p = p.to(dev).double().requires_grad_(True)
    pb, k = _Store.apply(p), [0]

    def conv(x, act=True):
        i = k[0]
        ci, co, _ = plan[i]
        k[0] += 1
        m = co * ci * 9
        z = _conv64(x, pb[offs[i]:offs[i] + m].reshape(co, 3, 3, ci), p[offs[i] + m:offs[i] + m + co])
        return _Act.apply(z) if act else _Head.apply(z)

    def up(x):
        return x.repeat_interleave(2, 2).repeat_interleave(2, 3)

    x, skips = _bf(rho).reshape(1, n, s, s), []
    for lvl in range(len(ch)):
        x = conv(conv(x))
        if lvl < len(ch) - 1:
            skips.append(x)
            x = _Store.apply(0.25 * x.reshape(ch[lvl], n, x.shape[2] // 2, 2, -1, 2).sum(dim=(3, 5)))
    F = (x.mean(dim=(2, 3)) * p[o:o + ch[-1], None]).sum(0) + p[-1]
    for lvl in range(len(ch) - 2, -1, -1):
        x = conv(conv(torch.cat([up(x), skips[lvl]])))
    S = conv(x, act=False).reshape(n, s, s)
    if not c["train"]:
        return {"F": F.detach(), "S": S.detach()}
    lF, lS = ((F - Ft) ** 2).sum(), ((S - St) ** 2).sum()
    grad = torch.autograd.grad(lF / n + lS / (n * s * s), p)[0]
    return {"F": F.detach(), "S": S.detach(), "loss": torch.stack([lF, lS]).detach(), "grad": grad}


def exact(case, seed):
    k = case["kind"]
    if k == "solve":
        w = _workload(case)
        if case["nx"] * case["ny"] * case["nz"] * case["steps"] > EXACT_STEPS[case["mode"]]:
            return None
        rho = _rho(w, seed, _dtype(case))
        F, grad = _Yee(w).solve(rho)
        return {"F": F, "grad": grad.reshape(rho.shape)}
    if k == "batch":
        ws = _batch_workloads(case)
        if len(ws) * case["steps"] > 4000:
            return None
        got = [_Yee(w).solve(_rho(w, seed * 1000 + i, _dtype(case))) for i, w in enumerate(ws)]
        return {"F": np.array([v[0] for v in got]), "grad": [v[1].reshape(W.design_shape(w)) for v, w in zip(got, ws)]}
    if k == "design":
        return _design64(case, *_design_inputs(case, seed))
    if k == "unet":
        return _unet64(case, _unet_inputs(case, seed))
    x, wt, bias, dz = (t.to(_device()).double() for t in _layer_inputs(case, seed))
    x.requires_grad_(True)
    wt.requires_grad_(True)
    z = _conv64(x, wt, bias)
    dx, dw = torch.autograd.grad(z, [x, wt], dz)
    return {"a": z.detach().clamp(min=0), "dza": dx * (x.detach() > 0), "dw": dw, "db": dz.sum(dim=(1, 2, 3))}
