"""The workloads the library's speed is measured on.

Every case is work that a user of the filter has it do, through the package's
public calls, on synthetic maps of the structure the library is made for
(periodic 2' pixels; signal, 1/f noise, row stripes, inhomogeneous white noise,
disc masks).  The kinds:

  solve      Context.solve on one map: the three-level, merged or augmented
             chain, float32 or float64, with or without a mask, on a fixed
             cooling schedule, or cooled adaptively to the residual target
  noalloc    solve_noalloc: the call of serving loops, no context kept
  refined    solve_refined: float32 sweeps refined by float64 residuals
  batch      solve_batch on many maps of one or several shapes
  train      WarmNet.train_step, one optimiser step of the learned warm start
  predict    WarmNet.predict, the warm start itself

listed() names the cases, draw(rng) gives more of the same ranges, prepare()
makes what a program holds before the call, run() is one call, work() what one
call cannot do without, exact() the result in 64 bits from plain torch.
"""

from __future__ import annotations

import math

import numpy as np
import torch

import paper_1704_00865_amd as wf
from paper_1704_00865_amd import nn

ARCMIN = math.pi / (180.0 * 60.0)
DPIX = 2.0 * ARCMIN
OMEGA = DPIX * DPIX
# transform lengths with built kernels (float64 up to 2048)
LENGTHS = (64, 128, 256, 384, 512, 768, 1024, 1536, 2048, 4096)
TUNED = (256, 768, 1536, 2048)  # float32 lengths built in every tiling


def listed():
    return [
        # the smallest map: a single patch filtered on demand; launches and
        # latency are all of it
        dict(name="solve_64_f32", kind="solve", ny=64, nx=64, prec="f32", chain="three",
             mask=True, sweeps=100, every=16),
        # a serving loop's call: small map, double precision, no context
        dict(name="noalloc_256_f64", kind="noalloc", ny=256, nx=256, prec="f64", chain="three",
             mask=True, sweeps=100, every=16),
        # the ordinary time-to-solution run: 512^2, double precision, cooled
        # adaptively until the residual is 1e-6 (lambda^0.97 from 1e4)
        dict(name="solve_512_f64_to_1e-6", kind="adaptive", ny=512, nx=512, prec="f64",
             chain="augmented", mask=False, sweeps=20000, every=16),
        # a rectangular map with a factor 3 in its sides, the two-level merged
        # chain, a budget that is not a whole number of residual checks
        dict(name="solve_768x1536_f32_merged", kind="solve", ny=768, nx=1536, prec="f32",
             chain="merged", mask=True, sweeps=100, every=8),
        # the benchmark's map and schedule, in the autotuned tiling
        dict(name="solve_2048_f32", kind="solve", ny=2048, nx=2048, prec="f32", chain="three",
             mask=True, sweeps=500, every=16),
        # the same map in double precision with the augmented chain (the
        # chain of the time-to-solution runs)
        dict(name="solve_2048_f64_augmented", kind="solve", ny=2048, nx=2048, prec="f64",
             chain="augmented", mask=True, sweeps=200, every=16),
        # the fastest route to a converged double-precision field
        dict(name="refined_512", kind="refined", ny=512, nx=512, prec="f64", chain="augmented",
             mask=False, sweeps=240, corr=160, rounds=5, every=8),
        # the largest single map
        dict(name="solve_4096_f32", kind="solve", ny=4096, nx=4096, prec="f32", chain="three",
             mask=True, sweeps=100, every=16),
        # the survey batch: 16 maps each of three sizes in one call
        dict(name="batch_uneven_f32", kind="batch", sizes="256,768,1536", per=16, prec="f32",
             chain="three", mask=False, sweeps=100, every=16, tune=True),
        # training targets of the warm start: equal masked maps, augmented
        # chain, whose chain field is the output
        dict(name="batch_1024_f32_augmented", kind="batch", sizes="1024", per=16, prec="f32",
             chain="augmented", mask=True, sweeps=100, every=16, tune=False),
        # one step of training the warm start
        dict(name="train_256", kind="train", ny=256, nx=256, n=16),
        # the warm start of four full-size maps
        dict(name="predict_1024", kind="predict", ny=1024, nx=1024, n=4),
    ]


def draw(rng):
    kind = rng.choice(("solve", "solve", "solve", "noalloc", "adaptive", "refined", "batch",
                       "batch", "train", "predict"))
    every = rng.choice((8, 16))
    if kind == "solve":
        prec = rng.choice(("f32", "f32", "f64"))
        top = 2048 if prec == "f64" else 4096
        # sides within a factor 4 of each other
        ny = rng.choice([n for n in LENGTHS if n <= top])
        nx = rng.choice([n for n in LENGTHS if n <= top and ny <= 4 * n and n <= 4 * ny])
        cost = ny * nx * (2 if prec == "f64" else 1)
        most = min(500, int(2048 * 2048 * 400 / cost))
        return dict(kind=kind, ny=ny, nx=nx, prec=prec,
                    chain=rng.choice(("three", "merged", "augmented")),
                    mask=rng.random() < 0.6, sweeps=rng.randint(48, max(49, most)), every=every)
    if kind == "noalloc":
        n = rng.choice((64, 128, 256, 384, 512))
        m = rng.choice([k for k in (64, 128, 256, 384, 512) if n <= 4 * k and k <= 4 * n])
        return dict(kind=kind, ny=n, nx=m, prec=rng.choice(("f32", "f64")),
                    chain=rng.choice(("three", "augmented")), mask=rng.random() < 0.5,
                    sweeps=rng.randint(48, 300), every=every)
    if kind == "adaptive":
        n = rng.choice((64, 128, 256, 384, 512))
        return dict(kind=kind, ny=n, nx=n, prec="f64", chain="augmented", mask=False,
                    sweeps=20000, every=every)
    if kind == "refined":
        n = rng.choice((128, 256, 384, 512, 768, 1024))
        return dict(kind=kind, ny=n, nx=n, prec="f64", chain="augmented", mask=False,
                    sweeps=rng.randint(220, 300), corr=rng.randint(150, 200), rounds=5,
                    every=every)
    if kind == "batch":
        sizes = rng.sample((128, 256, 384, 512, 768, 1024), rng.randint(1, 3))
        return dict(kind=kind, sizes=",".join(str(n) for n in sorted(sizes)),
                    per=rng.randint(3, 12), prec=rng.choice(("f32", "f32", "f64")),
                    chain=rng.choice(("three", "augmented")), mask=rng.random() < 0.5,
                    sweeps=rng.randint(48, 160), every=every, tune=False)
    n = rng.choice((64, 128, 256, 512))
    if kind == "train":
        return dict(kind=kind, ny=n, nx=rng.choice((64, 128, 256)),
                    n=rng.randint(1, 2 * 256 // n + 1))
    return dict(kind=kind, ny=n, nx=rng.choice((64, 128, 256, 512)),
                n=rng.randint(1, 4 * 512 // n + 3))


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------
def _device():
    return torch.device("cuda" if torch.cuda.is_available() else "cpu")


def _round(x):
    """float32-representable values in float64: both precisions and exact()
    then solve the same problem."""
    return x.to(torch.float32).to(torch.float64)


def _disc_mask(seed, ny, nx, frac):
    """1 = observed: periodic discs of radius 5 to 20 pixels over frac."""
    rng = np.random.default_rng([seed, 9])
    mask = np.ones((ny, nx), np.uint8)
    target, left = int(frac * ny * nx), 0
    for _ in range(1 << 20):
        r, cy, cx = int(rng.integers(5, 21)), int(rng.integers(ny)), int(rng.integers(nx))
        o = np.arange(-r, r + 1)
        at = np.ix_((cy + o) % ny, (cx + o) % nx)
        disc = o[:, None] ** 2 + o[None, :] ** 2 <= r * r
        left += int((mask[at][disc] != 0).sum())
        mask[at] = np.where(disc, 0, mask[at])
        if left >= target:
            return mask
    return mask


def _problem(seed, ny, nx, masked, level=10.0):
    """One map and its covariances, float64 tensors of float32 values."""
    dev = _device()
    g = torch.Generator(device=dev).manual_seed(int(seed) * 7919 + ny * 31 + nx)
    f8 = dict(dtype=torch.float64, device=dev)
    ly = 2 * math.pi * torch.fft.fftfreq(ny, d=DPIX, **f8)
    lx = 2 * math.pi * torch.fft.rfftfreq(nx, d=DPIX, **f8)
    ell = torch.hypot(ly[:, None], lx[None, :])
    ell = ell.clamp_min(2 * math.pi / (max(ny, nx) * DPIX))

    def noise(*shape):
        return torch.randn(*shape, generator=g, **f8)

    def field(var):
        return torch.fft.irfft2(var.sqrt() * torch.fft.rfft2(noise(ny, nx), norm="ortho"),
                                s=(ny, nx), norm="ortho")

    s_k = _round(2 * math.pi * 2500.0 * ell**-2 * torch.exp(-(ell / 1500.0) ** 2) / OMEGA)
    p_oof = _round((level * ARCMIN) ** 2 / OMEGA * (1 + (1000.0 / ell) ** 3))
    lyr = ly.abs().clamp_min(2 * math.pi / (ny * DPIX))
    shape = 1 + (1000.0 / lyr) ** 2
    p_st = _round(level**2 * ny / shape.sum() * shape)
    stripes = torch.fft.ifft(p_st.sqrt() * torch.fft.fft(noise(ny), norm="ortho"),
                             norm="ortho").real
    fy = torch.fft.fftfreq(ny, **f8)[:, None]
    fx = torch.fft.rfftfreq(nx, **f8)[None, :]
    z = torch.fft.irfft2(torch.fft.rfft2(noise(ny, nx)) *
                         torch.exp(-2 * math.pi**2 * 64.0 * (fx**2 + fy**2)), s=(ny, nx))
    z = (z - z.mean()) / z.std()
    n_pix = _round((level * torch.exp(0.5 * z)) ** 2)
    s = field(s_k)
    d = _round(s + field(p_oof) + stripes[:, None] + n_pix.sqrt() * noise(ny, nx))
    mask = torch.from_numpy(_disc_mask(seed, ny, nx, 0.1)).to(dev) if masked else None
    return dict(d=d, s_k=s_k, n_pix=n_pix, p_oof=p_oof, p_stripe=p_st, mask=mask), s


def _cast(p, prec):
    dt = torch.float32 if prec == "f32" else torch.float64
    return {k: v if v is None or v.dtype == torch.uint8 else v.to(dt).contiguous()
            for k, v in p.items()}


def _ramp(sweeps, lam0=1.0e4, cool=0.8):
    """The fixed cooling schedule: lambda_k = lam0^(1 - k/n) for the first
    n = 0.8 sweeps, then 1."""
    n = max(1, int(cool * sweeps))
    return [lam0 ** (1 - k / n) if k < n else 1.0 for k in range(sweeps)]


def _schedule(case):
    if case["kind"] == "adaptive":
        return wf.Schedule(lambda0=1.0e4, shrink=0.97, rtol=1e-6, max_sweeps=case["sweeps"],
                           monitor_every=case["every"], chain=case["chain"])
    return wf.Schedule(lambdas=_ramp(case["sweeps"]), rtol=0.0, max_sweeps=case["sweeps"],
                       monitor_every=case["every"], chain=case["chain"],
                       chain_field=case["kind"] == "batch" and case["chain"] == "augmented")


def _batch_maps(case, seed):
    """Seed, side and noise level of each map of a batch."""
    out = []
    for n in (int(x) for x in case["sizes"].split(",")):
        for i in range(case["per"]):
            level = float(np.random.default_rng([seed, n, i]).uniform(5.0, 30.0))
            out.append((seed * 1009 + 97 * i, n, level))
    return out


def _net_params(seed):
    """He weights with a non-zero output layer: a network in mid-training."""
    p = nn.init_params(seed)
    ci, co, w0, _ = nn.layer_offsets()[-1]
    w = np.zeros((9 * ci, co), np.float32)
    w[:, 0] = np.random.default_rng([seed, 3]).standard_normal(9 * ci) * 0.05
    p[w0:w0 + w.size] = w.ravel()
    return p


def _net_maps(case, seed):
    made = [_problem(seed * 1009 + i, case["ny"], case["nx"], True) for i in range(case["n"])]
    maps = {k: torch.stack([p[k] for p, _ in made]) for k in ("d", "n_pix", "mask")}
    maps["s"] = _round(torch.stack([s for _, s in made]))
    return maps


LR = 1.0e-3


def prepare(case, seed):
    kind = case["kind"]
    if kind in ("solve", "adaptive", "noalloc"):
        p = _cast(_problem(seed, case["ny"], case["nx"], case["mask"])[0], case["prec"])
        state = dict(kind=kind, p=p, schedule=_schedule(case))
        if kind != "noalloc":
            state["ctx"] = wf.Context(case["ny"], case["nx"], case["prec"])
            if case["prec"] == "f32" and case["ny"] in TUNED and case["nx"] in TUNED:
                state["ctx"].autotune(**p)  # as a program that filters many such maps does
        return state
    if kind == "refined":
        p = _cast(_problem(seed, case["ny"], case["nx"], False)[0], "f64")

        def sched(n, lam0):
            return wf.Schedule(lambdas=_ramp(n, lam0), rtol=0.0, max_sweeps=n,
                               monitor_every=case["every"], chain=case["chain"])
        return dict(kind=kind, p=p, c32=wf.Context(case["ny"], case["nx"], "f32"),
                    c64=wf.Context(case["ny"], case["nx"], "f64"),
                    first=sched(case["sweeps"], 1.0e4), corr=sched(case["corr"], 300.0),
                    rounds=case["rounds"])
    if kind == "batch":
        maps = [_cast(_problem(s, n, n, case["mask"], lv)[0], case["prec"])
                for s, n, lv in _batch_maps(case, seed)]
        ctxs = [wf.Context(*m["d"].shape, case["prec"]) for m in maps]
        outs = [torch.empty_like(m["d"]) for m in maps]
        if case["tune"]:
            wf.autotune_batch(ctxs, maps, outs=outs)
        return dict(kind=kind, maps=maps, ctxs=ctxs, outs=outs, schedule=_schedule(case))
    maps = _cast(_net_maps(case, seed), "f32")
    net = nn.WarmNet(case["ny"], case["nx"], batch_max=case["n"])
    net.set_params(_net_params(seed))
    return dict(kind=kind, net=net, maps=maps)


def run(state):
    kind = state["kind"]
    if kind in ("solve", "adaptive"):
        s, rep, _ = state["ctx"].solve(**state["p"], schedule=state["schedule"])
        return {"s": s, "sweeps": rep["sweeps"]}
    if kind == "noalloc":
        s, rep, _ = wf.solve_noalloc(**state["p"], schedule=state["schedule"])
        return {"s": s, "sweeps": rep["sweeps"]}
    if kind == "refined":
        s, rep, _ = wf.solve_refined(state["c32"], state["c64"], **state["p"],
                                     first=state["first"], corr=state["corr"],
                                     max_rounds=state["rounds"], rtol=0.0)
        return {"s": s, "sweeps": rep["sweeps"]}
    if kind == "batch":
        outs, _ = wf.solve_batch(state["ctxs"], state["maps"], schedule=state["schedule"],
                                 outs=state["outs"])
        return outs
    m = state["maps"]
    if kind == "train":
        loss = state["net"].train_step(m["d"], m["n_pix"], m["mask"], m["s"], LR)
        return {"loss": loss, "params": state["net"].get_params()}
    return state["net"].predict(m["d"], m["n_pix"], m["mask"])


# ---------------------------------------------------------------------------
# work and exact values
# ---------------------------------------------------------------------------
def _solve_work(ny, nx, sweeps, prec, masked):
    """Inputs read once, the map written once; two real 2-D transforms of
    2.5 N log2 N operations and about 25 per pixel of updates a sweep."""
    e, n, m = (4 if prec == "f32" else 8), ny * nx, ny * (nx // 2 + 1)
    return {"bytes": e * (3 * n + 2 * m + ny) + (n if masked else 0),
            "flops": sweeps * n * (5.0 * math.log2(n) + 25.0)}


def work(case):
    kind = case["kind"]
    if kind in ("solve", "noalloc"):
        return _solve_work(case["ny"], case["nx"], case["sweeps"], case["prec"], case["mask"])
    if kind == "adaptive":  # about five thousand sweeps reach the target
        return _solve_work(case["ny"], case["nx"], 5000, case["prec"], case["mask"])
    if kind == "refined":
        return _solve_work(case["ny"], case["nx"], case["sweeps"] + case["rounds"] * case["corr"],
                           "f64", False)
    if kind == "batch":
        each = [_solve_work(int(n), int(n), case["sweeps"], case["prec"], case["mask"])
                for n in case["sizes"].split(",")]
        return {k: case["per"] * sum(w[k] for w in each) for k in ("bytes", "flops")}
    pix = case["n"] * case["ny"] * case["nx"]
    flops = 0.0
    for i, ((ci, co), lev) in enumerate(zip(nn.layer_shapes(), LEVELS)):
        ci, co = (4 if i == 0 else ci), (1 if i == len(LEVELS) - 1 else co)
        passes = 1 if kind == "predict" else (2 if i == 0 else 3)
        flops += passes * 18.0 * ci * co * (pix >> (2 * lev))
    return {"bytes": pix * (13 if kind == "predict" else 13) +
            4 * (1 if kind == "predict" else 6) * nn.layer_offsets()[-1][3], "flops": flops}


def _exact_solve(p, chain, lambdas=None, adaptive=None, chain_field=False):
    """The messenger iteration in float64 from its equations: the field after
    the schedule's sweeps.  adaptive: (every, max_sweeps, shrink, rtol)."""
    d, s, npix = p["d"], p["s_k"], p["n_pix"]
    ny, nx = d.shape
    obs = torch.ones_like(d, dtype=torch.bool) if p["mask"] is None else p["mask"] != 0
    low = float(npix[obs].min())
    nf = p["p_oof"].clone()
    nf[:, 0] += nx * p["p_stripe"]
    three, phi, sc = chain == "three", 0.0, s
    if three:
        phi = 0.5 * low
        tau_a, tau_b = 0.9 * float(p["p_oof"].min()), 0.9 * phi
        nb_a = p["p_oof"] - tau_a
        nb_b = torch.full_like(s, phi - tau_b)
        nb_b[:, 0] += nx * p["p_stripe"]
    elif chain == "merged":
        tau_a = 0.9 * float(nf.min())
        nb_a = nf - tau_a
    else:
        sc = s + nf
    tau_w = low - phi
    nb_w = npix - (phi + tau_w)
    zero = torch.zeros(s.shape, dtype=torch.complex128, device=d.device)
    t_a, d_a, t_b, out = zero, zero, zero, zero
    lam = lam_prev = lambdas[0] if lambdas is not None else 1.0e4
    total = len(lambdas) if lambdas is not None else adaptive[1]
    dd_prev = k_prev = None
    count = 0
    for k in range(total):
        if lambdas is not None:
            lam_prev, lam = lam if k else lambdas[0], lambdas[k]
        tw, ta = lam * tau_w, lam * (0.0 if chain == "augmented" else tau_a)
        d1 = torch.fft.irfft2(out, s=(ny, nx))
        t2 = torch.fft.rfft2(torch.where(obs, d1 + tw / (nb_w + tw) * (d - d1), d1))
        if chain == "augmented":
            t_a, tau0 = t2, tau_w
            out = t2 * (sc / (sc + tw))
        else:
            tau0 = tau_a
            so = t_a * (s / (s + lam_prev * tau_a))
            if three:
                tb = lam * tau_b
                out = (nb_b * t2 + tw * t_b) / (nb_b + tw)
                t_b = (tb * out + nb_b * d_a) / (nb_b + tb)
                d_a = (nb_a * t_b + tb * t_a) / (nb_a + tb)
            else:
                out = d_a = (nb_a * t2 + tw * t_a) / (nb_a + tw)
            t_a = (ta * d_a + nb_a * so) / (nb_a + ta)
        count, x = k + 1, None
        lam_used, lam_prev = lam, lam
        if adaptive is not None and ((k + 1) % adaptive[0] == 0 or k + 1 == total):
            x = t_a / (sc + lam * tau0)
            r = torch.fft.irfft2((s + nf) * x, s=(ny, nx)) - d
            r = torch.where(obs, r + npix * torch.fft.irfft2(x, s=(ny, nx)), 0.0)
            dd = float(r.square().sum())
            d2 = float(d[obs].square().sum())
            if lam == 1.0 and math.sqrt(dd / d2) <= adaptive[3]:
                break
            if dd_prev is not None and abs(dd - dd_prev) < 1e-2 * (k - k_prev) * dd:
                lam = lam ** adaptive[2]
                lam = 1.0 if lam - 1.0 < 1e-3 else lam
            dd_prev, k_prev = dd, k
    x = t_a / (sc + lam_used * tau0)
    return torch.fft.irfft2((sc if chain_field else s) * x, s=(ny, nx)), count


def _exact_filter(p):
    """S (S + N)^-1 d without a mask, by conjugate gradients in float64."""
    d, ny, nx = p["d"], *p["d"].shape
    cov = p["s_k"] + p["p_oof"]
    cov[:, 0] += nx * p["p_stripe"]
    npix = p["n_pix"]
    pre = 1.0 / (cov + npix.mean())

    def mul(k, v):
        return torch.fft.irfft2(k * torch.fft.rfft2(v), s=(ny, nx))
    z = mul(pre, d)
    r = d - mul(cov, z) - npix * z
    y = mul(pre, r)
    q, ry = y, (r * y).sum()
    for _ in range(400):
        a = mul(cov, q) + npix * q
        al = ry / (q * a).sum()
        z, r = z + al * q, r - al * a
        y = mul(pre, r)
        new = (r * y).sum()
        if float(r.norm() / d.norm()) < 1e-14:
            break
        q, ry = y + (new / ry) * q, new
    return mul(p["s_k"], z)


LEVELS = [0, 0, 1, 1, 2, 2, 3, 3, 2, 2, 1, 1, 0, 0, 0]  # resolution of each convolution


def _exact_net(params, maps):
    """Prediction / sigma and sigma, by the network's definition."""
    d, npix, obs = maps["d"], maps["n_pix"], maps["mask"] != 0
    sig2 = (npix * obs).sum((1, 2), keepdim=True) / obs.sum((1, 2), keepdim=True)
    f0 = torch.where(obs, d / sig2.sqrt(), 0.0)
    rows = f0.sum(2, keepdim=True) / obs.sum(2, keepdim=True).clamp_min(1)
    x = torch.stack([f0, torch.where(obs, torch.log(npix / sig2), 0.0), obs.double(),
                     rows.expand_as(d)], dim=3)

    def conv(v, i):
        ci, co, w0, b0 = nn.layer_offsets()[i]
        w = params[w0:b0].view(3, 3, ci, co)
        out = params[b0:b0 + co].expand(v.shape[:3] + (co,))
        for dy in (-1, 0, 1):
            for dx in (-1, 0, 1):
                out = out + torch.roll(v, (-dy, -dx), (1, 2)) @ w[dy + 1, dx + 1][:v.shape[3]]
        return out

    def up(v):
        return v.repeat_interleave(2, 1).repeat_interleave(2, 2)

    enc, k = [], 0
    for lev in range(4):
        if lev:
            n, h, w, c = x.shape
            x = x.view(n, h // 2, 2, w // 2, 2, c).mean((2, 4))
        x = conv(conv(x, k).relu(), k + 1).relu()
        enc.append(x)
        k += 2
    for lev in (2, 1, 0):
        x = conv(conv(up(x), k).relu() + enc[lev], k + 1).relu()
        k += 2
    return conv(x, k)[..., 0], sig2.sqrt()


def exact(case, seed):
    kind = case["kind"]
    if kind in ("solve", "noalloc"):
        p = _problem(seed, case["ny"], case["nx"], case["mask"])[0]
        s, n = _exact_solve(p, case["chain"], _ramp(case["sweeps"]))
        return {"s": s, "sweeps": n}
    if kind == "adaptive":
        p = _problem(seed, case["ny"], case["nx"], case["mask"])[0]
        s, n = _exact_solve(p, case["chain"],
                            adaptive=(case["every"], case["sweeps"], 0.97, 1e-6))
        return {"s": s, "sweeps": n}
    if kind == "refined":
        p = _problem(seed, case["ny"], case["nx"], False)[0]
        return {"s": _exact_filter(p), "sweeps": None}
    if kind == "batch":
        return [_exact_solve(_problem(s, n, n, case["mask"], lv)[0], case["chain"],
                             _ramp(case["sweeps"]), chain_field=case["chain"] == "augmented")[0]
                for s, n, lv in _batch_maps(case, seed)]
    maps = _net_maps(case, seed)
    params = torch.tensor(_net_params(seed), dtype=torch.float64, device=_device())
    if kind == "predict":
        with torch.no_grad():
            parts = [{k: v[i:i + 1] for k, v in maps.items()} for i in range(case["n"])]
            made = [_exact_net(params, m) for m in parts]
            return torch.cat([y * s for y, s in made])
    params.requires_grad_(True)
    y, sig = _exact_net(params, maps)
    loss = (y - maps["s"] / sig).square().mean()
    loss.backward()
    g, p = params.grad, params.detach()
    # channels that only pad the stored layers take no gradient
    ci, co, w0, b0 = nn.layer_offsets()[-1]
    g[w0:b0].view(9 * ci, co)[:, 1:] = 0.0
    g[b0 + 1:] = 0.0
    return {"loss": float(loss.detach()), "params": p - LR * g / (g.abs() + 1e-8)}
