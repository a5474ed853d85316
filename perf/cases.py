"""The work that users of this library have it do, as a list of timed cases.

Each case is one pass through the public Python entry points (Sim, Mlp,
filter_subsample, closure_samples, spectra) the way a run, a training set or a
monitoring loop calls them.  `listed()` holds the cases, `draw()` gives more of
the same ranges, `prepare()` makes what a program has in hand before the call,
`run()` is one pass, `work()` what the pass cannot do without and `exact()` the
same result in 64-bit torch arithmetic written independently of the library.
"""

from __future__ import annotations

import math

import torch

from paper_1705_09807_amd import learned as G
from paper_1705_09807_amd.sim import Sim

DEV = "cuda:0"
F64 = torch.float64


# ---------------------------------------------------------------------------
# Cases
# ---------------------------------------------------------------------------
def _steps(name, nx, ny, dtype, steps, delta, schedule="fused", closure="analytic", mag="d2q5", stencil="iso9",
           nu=2e-4, ghost=1.6, every=1):
    c = dict(kind="steps", nx=nx, ny=ny, dtype=dtype, steps=steps, delta=float(delta), schedule=schedule,
             closure=closure, mag=mag, stencil=stencil, nu=nu, ghost=ghost, every=every)
    return dict(c, name=name) if name else c


def listed():
    return [
        # the smallest run in use: the 64^2 parity jet, sampled every 10 steps (launches and latency)
        _steps("les_64_fp64", 64, 64, "fp64", 10, 2.0, nu=1e-3, ghost=0.0),
        # the LES half of the headline workload, 50 steps between two looks at the fields
        _steps("les_1024_fp32", 1024, 1024, "fp32", 50, 4.0),
        # the DNS half of the headline workload
        _steps("dns_4096_fp32", 4096, 4096, "fp32", 10, 0.0),
        # the throughput configuration: 16-bit storage at a grid far beyond the caches (the largest case)
        _steps("les_8192_bf16", 8192, 8192, "bf16", 10, 4.0),
        # the paper's own study: 1024^2 LES in FP64 with a single relaxation time
        _steps("jet_1024_fp64", 1024, 1024, "fp64", 20, 2.0, nu=1e-3, ghost=0.0),
        # the paper's own model choices (D2Q9 vector distribution, closure with density gradients) on a ragged grid
        _steps("paper_model_1500x1001_fp64", 1500, 1001, "fp64", 7, 2.0, closure="full", mag="d2q9", nu=1e-3,
               ghost=0.0),
        # memory-limited runs: one population buffer updated in place, gradients lagging one step
        _steps("inplace_4096_fp32", 4096, 4096, "fp32", 10, 4.0, schedule="aa_lagged"),
        # LES with the learned closure, the network evaluated every step
        _steps("learned_1024_fp16", 1024, 1024, "fp16", 10, 4.0, closure="learned"),
        # monitoring of a DNS: diagnostics and energy spectra of one snapshot
        dict(kind="monitor", name="monitor_4096", n=4096, dtype="fp32"),
        # one snapshot of training data: filter and subsample a DNS, closure samples of every coarse cell
        dict(kind="samples", name="samples_4096_by_4", nx=4096, ny=4096, factor=4, delta=16.0, stencil="iso9"),
        # one optimiser step of the closure network at the default batch
        dict(kind="train", name="train_4096", rows=262144, batch=4096),
        # normalisation of a training set and the network's a-priori check on all its rows
        dict(kind="apriori", name="apriori_1m", rows=1048576),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["steps"] * 7 + ["learned"] * 2 + ["monitor", "samples", "train", "apriori"])
    if kind == "steps":
        nx, ny = _log(rng, 40, 4096), _log(rng, 40, 4096)
        steps = max(1, min(rng.randint(1, 30), 150_000_000 // (nx * ny)))
        schedule = rng.choice(["fused"] * 4 + ["aa", "aa_lagged"])
        delta = rng.choice([0.0, 0.0, 2.0, 4.0])
        dtype = rng.choice(["fp64", "fp32", "fp32", "fp16", "bf16"])
        closure = mag = None
        stencil = rng.choice(["iso9", "iso9", "central5", "local_iso9"])
        if schedule == "aa_lagged" and stencil.startswith("local"):
            stencil = "iso9"
        if schedule == "fused" and not stencil.startswith("local"):
            closure = rng.choice(["analytic", "analytic", "full"])
            mag = rng.choice(["d2q5", "d2q5", "d2q9"]) if dtype in ("fp64", "fp32") else None
        return _steps(None, nx, ny, dtype, steps, delta, schedule=schedule, closure=closure or "analytic",
                      mag=mag or "d2q5", stencil=stencil, nu=1e-3)
    if kind == "learned":
        nx, ny = _log(rng, 100, 2048), _log(rng, 100, 2048)
        return _steps(None, nx, ny, rng.choice(["fp32", "fp16", "bf16"]), rng.randint(2, 16), 4.0, closure="learned",
                      every=rng.choice([1, 1, 4, 16]), nu=1e-3)
    if kind == "monitor":
        return dict(kind="monitor", n=2 ** rng.randint(6, 12), dtype=rng.choice(["fp64", "fp32", "fp16"]))
    if kind == "samples":
        f = rng.choice([2, 4, 8])
        return dict(kind="samples", nx=f * _log(rng, 40, 4096 // f), ny=f * _log(rng, 40, 4096 // f), factor=f,
                    delta=rng.choice([3.0, 4.0]) * f, stencil=rng.choice(["iso9", "central5"]))
    if kind == "train":
        return dict(kind="train", rows=_log(rng, 20000, 500000), batch=_log(rng, 200, 16384))
    return dict(kind="apriori", rows=_log(rng, 2000, 1000000))


# ---------------------------------------------------------------------------
# Inputs
# ---------------------------------------------------------------------------
def _gen(seed):
    return torch.Generator(device=DEV).manual_seed(int(seed) * 7919 + 17)


def _fields(nx, ny, seed):
    """[5, ny, nx] rho, m_x, m_y, B_x, B_y of a developing magnetized double shear layer: tanh layers, streamwise
    modes with seeded amplitudes and phases, weak acoustic and magnetic waves, white noise, a mean drift."""
    g = _gen(seed)
    p = torch.rand(32, generator=g, device=DEV, dtype=F64).tolist()
    y = torch.arange(ny, device=DEV, dtype=F64)[:, None] / ny
    x = torch.arange(nx, device=DEV, dtype=F64)[None, :] / nx
    tau, u0, d = 2 * math.pi, 0.05, 1.0 / 40.0
    ux = u0 * (torch.tanh((y - 0.25) / d) - torch.tanh((y - 0.75) / d) - 1.0) + 0.004
    env = torch.exp(-((y - 0.25) / (2 * d)) ** 2) + torch.exp(-((y - 0.75) / (2 * d)) ** 2)
    uy = 0.002 + 0 * (x + y)
    for k in range(5):
        uy = uy + u0 * 0.05 * (0.5 + p[k]) * torch.sin(tau * ((k + 2) * x + p[5 + k])) * env
    rho = 1.0 + 0.004 * torch.cos(tau * (2 * x + p[10])) * torch.sin(tau * (y + p[11]))
    bx = 0.01 + 0.003 * torch.sin(tau * (3 * y + p[12])) + 0.002 * torch.cos(tau * (x + 2 * y + p[13]))
    by = 0.001 + 0.003 * torch.sin(tau * (2 * x + p[14])) - 0.001 * torch.cos(tau * (x + 2 * y + p[13]))
    m = torch.stack([rho, rho * ux, rho * uy, bx + 0 * x, by + 0 * y])
    m[1:] += 2e-4 * (2 * torch.rand(4, ny, nx, generator=g, device=DEV, dtype=F64) - 1)
    return m


def _weights(seed):
    """(w1 [63, 64], b1, w2, b2, w3, b3) FP32: Glorot-sized weights and small biases."""
    g = _gen(seed + 101)

    def u(i, o):
        return ((torch.rand(i, o, generator=g, device=DEV, dtype=F64) * 2 - 1) * math.sqrt(6.0 / (i + o))).float()

    def b(o):
        return ((torch.rand(o, generator=g, device=DEV, dtype=F64) * 2 - 1) * 0.1).float()

    return u(63, 64), b(64), u(64, 64), b(64), u(64, 4), b(4)


NORM = dict(shift=[1.0, 0.0, 0.0, 0.01, 0.0, 0.0, 0.0], scale=[150.0, 22.0, 300.0, 220.0, 220.0, 900.0, 900.0],
            out_scale=[2e-6, 2e-6, 2e-6, 1e-6])


def _mlp(seed):
    return G.Mlp(G.flat_params(*[w.cpu() for w in _weights(seed)]), device=DEV)


def _rows(n, seed):
    """Feature rows [n, 64] and targets [n, 4] with the fields' means and spreads, a few rows out of range."""
    g = _gen(seed + 202)
    mean = torch.tensor(NORM["shift"], device=DEV, dtype=F64).repeat_interleave(9)
    dev = 1.0 / torch.tensor(NORM["scale"], device=DEV, dtype=F64).repeat_interleave(9)
    x = torch.zeros(n, 64, device=DEV, dtype=torch.float32)
    z = torch.randn(n, 63, generator=g, device=DEV, dtype=torch.float32)
    c = torch.randn(n, 7, generator=g, device=DEV, dtype=torch.float32).repeat_interleave(9, dim=1)
    x[:, :63] = ((0.9 * c + 0.4 * z).double() * dev + mean).float()
    x[::997, 20] = 5.0
    t = 2e-6 * torch.randn(n, 4, generator=g, device=DEV, dtype=torch.float32)
    t[:, 0] += (3e-6 * c[:, 9] * c[:, 18]).float()
    return x, t


def prepare(case, seed):
    k = case["kind"]
    if k == "steps":
        s = Sim(nx=case["nx"], ny=case["ny"], nu=case["nu"], eta=case["nu"], delta=case["delta"], s5=case["ghost"],
                s6=case["ghost"], s7=case["ghost"], s8=case["ghost"], grad_stencil=case["stencil"],
                dtype=case["dtype"], schedule=case["schedule"], b_ref=(0.01, 0.0), closure=case["closure"],
                mag_lattice=case["mag"], device=DEV)
        s.init_from_moments(_fields(case["nx"], case["ny"], seed))
        torch.cuda.synchronize()
        s._keep = None  # the initial fields are not needed any more
        if case["closure"] == "learned":
            mlp = _mlp(seed)
            mlp.set_norm(**NORM)
            s.set_closure_mlp(mlp.pack())
            s.set_correction_interval(case["every"])
        return dict(case=case, sim=s)
    if k == "monitor":
        s = Sim(nx=case["n"], ny=case["n"], nu=1e-3, eta=1e-3, dtype=case["dtype"], b_ref=(0.01, 0.0), device=DEV)
        s.init_from_moments(_fields(case["n"], case["n"], seed))
        torch.cuda.synchronize()
        s._keep = None
        return dict(case=case, sim=s)
    if k == "samples":
        return dict(case=case, mom=_fields(case["nx"], case["ny"], seed))
    mlp = _mlp(seed)
    x, t = _rows(case["rows"], seed)
    st = dict(case=case, mlp=mlp, x=x, t=t)
    if k == "train":
        mlp.set_norm(**NORM)
        st["idx"] = torch.randint(0, case["rows"], (case["batch"],), generator=_gen(seed + 303), device=DEV,
                                  dtype=torch.int32)
    return st


def run(state):
    case = state["case"]
    k = case["kind"]
    if k == "steps":
        s = state["sim"]
        s.step(case["steps"])
        m = s.moments()
        # a snapshot keeps the digits that the storage type carries
        return m if case["dtype"] == "fp64" else m.float()
    if k == "monitor":
        s = state["sim"]
        d = s.diagnostics()
        m = s.moments()
        ek, em, ekx = G.spectra(m)
        return dict(diag=d, mom=m, ek=ek, em=em, ekx=ekx)
    if k == "samples":
        c = G.filter_subsample(state["mom"], case["factor"], case["delta"])
        x, t = G.closure_samples(c, case["delta"] / case["factor"], case["stencil"])
        return dict(coarse=c, x=x, t=t)
    mlp = state["mlp"]
    if k == "train":
        loss = mlp.train_step(state["x"], state["t"], state["idx"], 2e-3)
        return dict(loss=loss, params=mlp.params, m=mlp.m, v=mlp.v)
    mlp.fit_norm(state["x"], state["t"])
    y, ood = mlp.forward(state["x"])
    return dict(norm=mlp.norm, y=y, ood=ood)


# ---------------------------------------------------------------------------
# What a pass cannot do without
# ---------------------------------------------------------------------------
SIZE = {"fp64": 8, "fp32": 4, "fp16": 2, "bf16": 2}
MLP_FLOPS = 2 * (63 * 64 + 64 * 64 + 64 * 4)


def work(case):
    """Bytes: each input once, each output once (for a run of several steps: the state once in and once out, and the
    snapshot); flops: the collision (and closure) of every cell and step, the network, the transforms, the taps."""
    k = case["kind"]
    if k == "steps":
        n = case["nx"] * case["ny"]
        pops = 9 + 2 * (9 if case["mag"] == "d2q9" else 5)
        flops = (230 if pops == 19 else 300) + (110 if case["delta"] else 0)
        evals = -(-case["steps"] // case["every"]) if case["closure"] == "learned" else 0
        b = n * (2 * pops * SIZE[case["dtype"]] + 5 * (8 if case["dtype"] == "fp64" else 4))
        return dict(bytes=b, flops=n * (case["steps"] * flops + evals * MLP_FLOPS))
    if k == "monitor":
        n = case["n"]
        return dict(bytes=n * n * (19 * SIZE[case["dtype"]] + 40),
                    flops=n * n * (80.0 + 2 * (5 * 2 * math.log2(n) + 10)))
    if k == "samples":
        n, f = case["nx"] * case["ny"], case["factor"]
        taps = 2 * math.ceil(5 * case["delta"] / math.sqrt(12)) + 1
        return dict(bytes=n * 40 + n // (f * f) * (96 + 272), flops=n * (20 + 24 * taps / f + 24 * taps / (f * f)))
    if k == "train":
        return dict(bytes=case["batch"] * (256 + 16 + 4) + 8580 * 24, flops=case["batch"] * 3.0 * MLP_FLOPS)
    return dict(bytes=case["rows"] * (256 + 16 + 16 + 4), flops=case["rows"] * (MLP_FLOPS + 40.0))


# ---------------------------------------------------------------------------
# The same in 64 bits
# ---------------------------------------------------------------------------
CX = [0, 1, 0, -1, 0, 1, -1, -1, 1]
CY = [0, 0, 1, 0, -1, 1, 1, -1, -1]
W9 = [4 / 9] + [1 / 9] * 4 + [1 / 36] * 4
W5 = [1 / 3] + [1 / 6] * 4


def _sh(a, dx, dy):
    """a at (x + dx, y + dy)."""
    return torch.roll(a, (-dy, -dx), (-2, -1))


def _grad(a, stencil):
    if stencil.endswith("iso9"):
        d = _sh(a, 1, 1) - _sh(a, -1, -1)
        e = _sh(a, 1, -1) - _sh(a, -1, 1)
        return ((_sh(a, 1, 0) - _sh(a, -1, 0)) / 3 + (d + e) / 12, (_sh(a, 0, 1) - _sh(a, 0, -1)) / 3 + (d - e) / 12)
    return (_sh(a, 1, 0) - _sh(a, -1, 0)) / 2, (_sh(a, 0, 1) - _sh(a, 0, -1)) / 2


def _moments(f, gx, gy):
    return [sum(f), sum(CX[i] * f[i] for i in range(9) if CX[i]), sum(CY[i] * f[i] for i in range(9) if CY[i]),
            sum(gx), sum(gy)]


def _closure(gm, gb, pb, ir, k2):
    """tau_xy, tau_xx - tau_yy, tau_xx + tau_yy, eps of the gradients of m and B (pb: those of the induction product)."""
    kr = k2 * ir
    pxx, pyy = kr * (gm[0][0] ** 2 + gm[0][1] ** 2), kr * (gm[1][0] ** 2 + gm[1][1] ** 2)
    pxy = kr * (gm[0][0] * gm[1][0] + gm[0][1] * gm[1][1])
    qxx, qyy = k2 * (gb[0][0] ** 2 + gb[0][1] ** 2), k2 * (gb[1][0] ** 2 + gb[1][1] ** 2)
    qxy = k2 * (gb[0][0] * gb[1][0] + gb[0][1] * gb[1][1])
    eps = kr * (gm[0][0] * pb[1][0] + gm[0][1] * pb[1][1] - gm[1][0] * pb[0][0] - gm[1][1] * pb[0][1])
    return pxy - qxy, (pxx - pyy) - (qxx - qyy), pxx + pyy, eps


def _bf(a):
    return a.to(torch.bfloat16).to(F64)


def _network(z, w):
    """y of normalised inputs z [n, 63]: bfloat16 operands, exact products and sums."""
    w1, b1, w2, b2, w3, b3 = [v.double() for v in w]
    h = torch.relu(_bf(z) @ _bf(w1) + b1)
    h2 = torch.relu(_bf(h) @ _bf(w2) + b2)
    return _bf(h2) @ _bf(w3) + b3, h, h2


def _learned_terms(m, w):
    ux, uy = m[1] / m[0], m[2] / m[0]
    om = (_sh(uy, 1, 0) - _sh(uy, -1, 0) - _sh(ux, 0, 1) + _sh(ux, 0, -1)) / 2
    jz = (_sh(m[4], 1, 0) - _sh(m[4], -1, 0) - _sh(m[3], 0, 1) + _sh(m[3], 0, -1)) / 2
    z = []
    for k, a in enumerate([m[0], ux, uy, m[3], m[4], om, jz]):
        a = (a - float(torch.tensor(NORM["shift"][k]))) * float(torch.tensor(NORM["scale"][k]))
        z += [_sh(a, dx, dy).reshape(-1) for dy in (-1, 0, 1) for dx in (-1, 0, 1)]
    z = torch.stack(z, 1)
    y, _, _ = _network(z, w)
    y = y * torch.tensor(NORM["out_scale"], device=DEV).double()
    y = torch.where((z.abs() > 6).any(1, keepdim=True), torch.zeros_like(y), y)
    return [y[:, o].reshape(m[0].shape) for o in range(4)]


def _exact_steps(case, seed):
    if case["nx"] * case["ny"] * case["steps"] > 700_000_000:
        return None
    qg = 9 if case["mag"] == "d2q9" else 5
    wg = W9 if qg == 9 else W5
    s3 = 2.0 / (6.0 * case["nu"] + 1.0)
    sg = case["ghost"] if case["ghost"] > 0 else s3
    k2 = case["delta"] ** 2 / 12.0
    w = _weights(seed) if case["closure"] == "learned" else None
    m = list(_fields(case["nx"], case["ny"], seed))
    ux, uy, bx, by = m[1] / m[0], m[2] / m[0], m[3], m[4]
    f, gx, gy = [], [], []
    for i in range(9):
        cu, cb = CX[i] * ux + CY[i] * uy, CX[i] * bx + CY[i] * by
        f.append(W9[i] * m[0] * (1 + 3 * cu + 4.5 * cu ** 2 - 1.5 * (ux ** 2 + uy ** 2))
                 + 4.5 * W9[i] * (0.5 * (bx ** 2 + by ** 2) * (CX[i] ** 2 + CY[i] ** 2) - cb ** 2))
        if i < qg:
            gx.append(wg[i] * (bx + 3 * (cu * bx - cb * ux)))
            gy.append(wg[i] * (by + 3 * (cu * by - cb * uy)))
    del m, ux, uy, bx, by
    prev = corr = None
    for t in range(case["steps"]):
        m = _moments(f, gx, gy)
        ir = 1.0 / m[0]
        txy = td = ts = eps = 0.0
        if k2:
            src = prev if (case["schedule"] == "aa_lagged" and prev is not None) else m
            if case["stencil"].startswith("local"):
                wm = _grad(m[2], case["stencil"])[0] - _grad(m[1], case["stencil"])[1]
                e3 = m[1] * m[2] * ir - m[3] * m[4]
                e4 = (m[1] ** 2 - m[2] ** 2) * ir - (m[3] ** 2 - m[4] ** 2)
                sxy = -1.5 * s3 * ((f[5] - f[6] + f[7] - f[8]) - e3)
                sxx = -0.75 * s3 * ((f[1] + f[3] - f[2] - f[4]) - e4)
                e = (m[1] * m[4] - m[2] * m[3]) * ir
                gm = [(sxx, sxy - 0.5 * wm), (sxy + 0.5 * wm, -sxx)]
                gb = [(-3 * s3 * (gx[1] - gx[3]), -3 * s3 * (gx[2] - gx[4] + e)),
                      (-3 * s3 * (gy[1] - gy[3] - e), -3 * s3 * (gy[2] - gy[4]))]
                pb = gb
            else:
                gm = [_grad(src[k], case["stencil"]) for k in (1, 2)]
                gb = [_grad(src[k], case["stencil"]) for k in (3, 4)]
                pb = gb
                if case["closure"] == "full":
                    gr = [v * ir for v in _grad(m[0], case["stencil"])]
                    gm = [tuple(gm[k][b] - m[1 + k] * gr[b] for b in (0, 1)) for k in (0, 1)]
                    pb = [tuple(gb[k][b] - m[3 + k] * gr[b] for b in (0, 1)) for k in (0, 1)]
            txy, td, ts, eps = _closure(gm, gb, pb, ir, k2)
        if w is not None:
            if corr is None or t % case["every"] == 0:
                corr = _learned_terms(m, w)
            txy, td, ts, eps = txy + corr[1], td + corr[0] - corr[2], ts + corr[0] + corr[2], eps + corr[3]
        prev = m
        rho, mx, my, bx, by = m
        a = f[1] + f[2] + f[3] + f[4]
        b = f[5] + f[6] + f[7] + f[8]
        q = -3 * ((mx ** 2 + my ** 2) * ir + ts)
        d3 = s3 / 4 * ((f[5] - f[6] + f[7] - f[8]) - (mx * my * ir - bx * by + txy))
        d4 = s3 / 4 * ((f[1] - f[2] + f[3] - f[4]) - ((mx ** 2 - my ** 2) * ir - (bx ** 2 - by ** 2) + td))
        d5 = sg / 12 * ((2 * (f[3] - f[1]) + f[5] - f[6] - f[7] + f[8]) + mx)
        d6 = sg / 12 * ((2 * (f[4] - f[2]) + f[5] + f[6] - f[7] - f[8]) + my)
        d7 = sg / 180 * ((4 * f[0] - 5 * a + 4 * b) - q)
        d8 = sg / 20 * ((4 * f[0] - b) - (5.0 / 3.0 * rho + q))
        new = []
        for i in range(9):
            cx, cy = CX[i], CY[i]
            r = (cx * cy * d3 + (cx * cx - cy * cy) * d4 + (3 * cx * cy * cy - 2 * cx) * d5
                 + (3 * cy * cx * cx - 2 * cy) * d6 + (4 - 9 * (cx * cx + cy * cy - 2 * cx * cx * cy * cy)) * d7
                 + (4 - 4 * (cx * cx + cy * cy) + 3 * cx * cx * cy * cy) * d8)
            new.append(_sh(f[i] - r, -cx, -cy))
        f = new
        E = (mx * by - my * bx) * ir + eps
        for i in range(qg):
            gx[i] = _sh(gx[i] - s3 * (gx[i] - wg[i] * (bx - 3 * CY[i] * E)), -CX[i], -CY[i])
            gy[i] = _sh(gy[i] - s3 * (gy[i] - wg[i] * (by + 3 * CX[i] * E)), -CX[i], -CY[i])
    return torch.stack(_moments(f, gx, gy))


def _exact_monitor(case, seed):
    n = case["n"]
    m = list(_fields(n, n, seed))
    ux, uy = m[1] / m[0], m[2] / m[0]
    cd = lambda a, dx, dy: (_sh(a, dx, dy) - _sh(a, -dx, -dy)) / 2  # noqa: E731
    om, jz = cd(uy, 1, 0) - cd(ux, 0, 1), cd(m[4], 1, 0) - cd(m[3], 0, 1)
    dv = cd(m[3], 1, 0) + cd(m[4], 0, 1)
    diag = dict(t=None, nonfinite=None, mass=m[0].sum(), mom_x=m[1].sum(), mom_y=m[2].sum(), bsum_x=m[3].sum(),
                bsum_y=m[4].sum(), e_kin=((m[1] ** 2 + m[2] ** 2) / (2 * m[0])).mean(),
                e_mag=((m[3] ** 2 + m[4] ** 2) / 2).mean(), enstrophy=(om ** 2 / 2).mean(), j2=(jz ** 2).mean(),
                divb_max=dv.abs().max(), divb_rms=(dv ** 2).mean().sqrt())
    diag = {k: None if v is None else float(v) for k, v in diag.items()}
    kk = torch.fft.fftfreq(n, 1.0 / n, device=DEV, dtype=F64).round()
    k2 = (kk[:, None] ** 2 + kk[None, :] ** 2)
    b = torch.floor(torch.sqrt(k2) + 0.5).long().reshape(-1)
    nb = int(math.floor(math.sqrt(2.0) * (n // 2) + 0.5)) + 1
    power = lambda p, q: sum((torch.fft.fft2(a) / (n * n)).abs() ** 2 for a in (p, q)) / 2  # noqa: E731
    pu, pb = power(ux, uy), power(m[3], m[4])
    z = torch.zeros(nb, device=DEV, dtype=F64)
    ekx = torch.zeros(n // 2 + 1, device=DEV, dtype=F64).index_add(0, kk.abs().long(), pu.sum(0))
    return dict(diag=diag, mom=torch.stack(m), ek=z.index_add(0, b, pu.reshape(-1)), em=z.index_add(0, b, pb.reshape(-1)), ekx=ekx)


def _exact_samples(case, seed):
    m = list(_fields(case["nx"], case["ny"], seed))
    f, delta = case["factor"], case["delta"]
    r = math.ceil(5 * (delta / math.sqrt(12.0)))
    tap = [math.exp(-(i * i) / (2 * delta * delta / 12.0)) for i in range(-r, r + 1)]
    tot = math.fsum(tap)
    out = []
    prods = [lambda: m[0], lambda: m[1], lambda: m[2], lambda: m[3], lambda: m[4], lambda: m[1] * m[1] / m[0],
             lambda: m[1] * m[2] / m[0], lambda: m[2] * m[2] / m[0], lambda: m[3] * m[3], lambda: m[3] * m[4],
             lambda: m[4] * m[4], lambda: (m[1] * m[4] - m[2] * m[3]) / m[0]]
    for p in prods:
        a = p()
        s = sum(tap[i + r] / tot * torch.roll(a, -i, 1)[:, ::f] for i in range(-r, r + 1))
        out.append(sum(tap[i + r] / tot * torch.roll(s, -i, 0)[::f] for i in range(-r, r + 1)))
    c = torch.stack(out)
    rho, mx, my, bx, by = c[:5]
    ux, uy = mx / rho, my / rho
    om = (_sh(uy, 1, 0) - _sh(uy, -1, 0)) / 2 - (_sh(ux, 0, 1) - _sh(ux, 0, -1)) / 2
    jz = (_sh(by, 1, 0) - _sh(by, -1, 0)) / 2 - (_sh(bx, 0, 1) - _sh(bx, 0, -1)) / 2
    x = torch.zeros(rho.numel(), 64, device=DEV, dtype=F64)
    for k, a in enumerate([rho, ux, uy, bx, by, om, jz]):
        for dy in (-1, 0, 1):
            for dx in (-1, 0, 1):
                x[:, k * 9 + (dy + 1) * 3 + dx + 1] = _sh(a, dx, dy).reshape(-1)
    gm, gb = [_grad(v, case["stencil"]) for v in (mx, my)], [_grad(v, case["stencil"]) for v in (bx, by)]
    txy, td, ts, eps = _closure(gm, gb, gb, 1 / rho, (delta / f) ** 2 / 12.0)
    rxx, rxy, ryy = c[5] - mx * mx / rho, c[6] - mx * my / rho, c[7] - my * my / rho
    qxx, qxy, qyy = c[8] - bx * bx, c[9] - bx * by, c[10] - by * by
    t = torch.stack([rxx + (qyy - qxx) / 2 - (ts + td) / 2, rxy - qxy - txy, ryy + (qxx - qyy) / 2 - (ts - td) / 2,
                     c[11] - (mx * by - my * bx) / rho - eps], -1)
    return dict(coarse=c, x=x, t=t.reshape(-1, 4))


def _norm64(shift, scale, out):
    n = torch.zeros(32, device=DEV, dtype=F64)
    n[:7], n[8:15], n[15], n[16:20] = shift, scale, 1.0, out
    return n.float().double()


def _exact_train(case, seed):
    x, t = _rows(case["rows"], seed)
    idx = torch.randint(0, case["rows"], (case["batch"],), generator=_gen(seed + 303), device=DEV, dtype=torch.int32)
    x, t = x[idx.long()].double(), t[idx.long()].double()
    w = _weights(seed)
    w1, b1, w2, b2, w3, b3 = [v.double() for v in w]
    nm = _norm64(*[torch.tensor(NORM[k], device=DEV, dtype=F64) for k in ("shift", "scale", "out_scale")])
    z = (x[:, :63] - nm[:7].repeat_interleave(9)) * nm[8:15].repeat_interleave(9)
    y, h1, h2 = _network(z, w)
    r = y - t / nm[16:20]
    d3 = r * (2.0 / r.numel())
    d2 = (d3 @ _bf(w3).T) * (h2 > 0)
    d1 = (d2 @ _bf(w2).T) * (h1 > 0)
    g1 = torch.cat([_bf(z).T @ d1, torch.zeros(1, 64, device=DEV, dtype=F64)])
    g = torch.cat([v.reshape(-1) for v in (g1, d1.sum(0), _bf(h1).T @ d2, d2.sum(0), _bf(h2).T @ d3, d3.sum(0))])
    p = torch.cat([v.reshape(-1) for v in (torch.cat([w1, torch.zeros(1, 64, device=DEV, dtype=F64)]), b1, w2, b2, w3,
                                           b3)])
    return dict(loss=(r ** 2).mean().reshape(1), params=p - 2e-3 * g / (g.abs() + 1e-8), m=0.1 * g, v=0.001 * g * g)


def _exact_apriori(case, seed):
    x, t = _rows(case["rows"], seed)
    c = x[:, 4:63:9].double()
    out = (t.double() ** 2).mean(0).sqrt()
    nm = _norm64(c.mean(0), 1.0 / c.std(0, unbiased=False), out)
    z = (x[:, :63].double() - nm[:7].repeat_interleave(9)) * nm[8:15].repeat_interleave(9)
    return dict(norm=nm, y=_network(z, _weights(seed))[0], ood=None)


def exact(case, seed):
    return {"steps": _exact_steps, "monitor": _exact_monitor, "samples": _exact_samples, "train": _exact_train,
            "apriori": _exact_apriori}[case["kind"]](case, seed)
