"""Performance cases: the work a program built on this package has it do.

Every case is one call (or the short chain of calls a program always makes
together) through the public entry points, with the geometry of the
repository's own workloads (two-telescope structure functions, phase screens
on square grids and pupils, pistons and tilts of aperture arrays, the
frozen-flow time series, batches of uneven screens, training of the learned
proposal).  ``listed`` names one case per use, ``draw`` gives others of the
same ranges, ``exact`` is the same result in 64 bits from plain torch.
"""
import decimal
import math

import numpy as np
import torch

import paper_2404_02978_amd as q
import workloads

DEV = "cuda:0"
F64 = torch.float64
PREC = {"fp64": q.PREC_FP64, "fp32": q.PREC_FP32, "split_bf16": q.PREC_SPLIT_BF16,
        "bf16x6": q.PREC_BF16X6, "fp16x3": q.PREC_FP16X3}
R0 = 0.1  # Fried parameter of every workload, m


def listed():
    return [
        # the smallest call: a quick look at a structure function (the sizes of
        # the smoke check), bound by launches and latency
        dict(name="sf_small", kind="structure", api="end_to_end", precision="fp32", K=512, R=300,
             R_block=100, nB=32, L0=25.0, along_x=True, eq3=False),
        # the benchmark's workload for one outer scale: frequencies, weights and
        # the structure function of 1e5 realisations
        dict(name="sf_headline", kind="structure", api="sets", precision="fp16x3", K=16384,
             R=100000, R_block=256, nB=32, L0=25.0, along_x=True, eq3=False),
        # the paper's own usage: fresh frequencies for every realisation
        dict(name="sf_fresh", kind="structure", api="sets", precision="fp16x3", K=16384, R=20000,
             R_block=1, nB=32, L0=25.0, along_x=True, eq3=False),
        # one static frequency set in binary64, the plain side of the benchmark's
        # fixed-error comparison
        dict(name="sf_static_f64", kind="structure", api="end_to_end", precision="fp64", K=4096,
             R=100000, R_block=100000, nB=32, L0=25.0, along_x=True, eq3=False),
        # the benchmark's phase workload: 128 small screens in binary64, each
        # from its own frequencies
        dict(name="phase_fresh_f64", kind="screen", precision="fp64", K=1024, n=32, side=1.0,
             disk=False, R=128, R_block=1, L0=25.0, eq3=False),
        # the same screens from one shared set in the default precision
        dict(name="phase_shared_f32", kind="screen", precision="fp32", K=1024, n=32, side=1.0,
             disk=False, R=128, R_block=128, L0=25.0, eq3=False),
        # a pupil of an ordinary size with nothing round about it: ragged
        # points, rows and frequencies, several sets, the literal Eq. 3 form
        dict(name="pupil_ragged", kind="screen", precision="bf16x6", K=10007, n=101, side=8.0,
             disk=True, R=777, R_block=259, L0=25.0, eq3=True),
        # the large screen, the largest work of the benchmark
        dict(name="screen_large", kind="screen", precision="fp16x3", K=65536, n=256, side=8.0,
             disk=False, R=4096, R_block=4096, L0=25.0, eq3=False),
        # pistons of a ten-telescope array of unequal apertures
        dict(name="pistons_array", kind="apertures", precision="fp32", K=4096, n_ap=10, R=10000,
             R_block=250, L0=25.0, tilt=False, eq3=False),
        # the frozen-flow experiment at the paper's sizes, in binary64
        dict(name="temporal_f64", kind="temporal", precision="fp64", N=44, M=1024, R=2000,
             R_block=1, L0=22.0),
        # a batch of uneven pupils, replayed from its graph
        dict(name="batch_pupils", kind="batch", precision="bf16x6", n_inst=16, k_lo=2048,
             k_hi=65536, n_lo=32, n_hi=512, R=256, R_block=256, apertures=False),
        # the first steps of training the learned proposal
        dict(name="train_proposal", kind="train", n_ctx=64, m=2048, ctx_per_step=16, steps=20,
             G=64),
    ]


# ------------------------------------------------------------------- draws ----
def _log_int(rng, lo, hi):
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    kind = rng.choice(["structure", "structure", "structure", "screen", "screen", "screen",
                       "apertures", "apertures", "temporal", "batch", "train"])
    L0 = round(rng.uniform(10.0, 100.0), 2)
    eq3 = rng.random() < 0.15
    prec = rng.choice(["fp64", "fp32", "split_bf16", "bf16x6", "fp16x3", "fp16x3"])
    if kind == "structure":
        K, R = _log_int(rng, 256, 16384), _log_int(rng, 200, 100000)
        nB = rng.choice([rng.randint(3, 31), 32, 32, rng.randint(33, 64)])
        form = rng.choice(["fresh", "shared", "shared", "static"])
        cap = 3.3e8 * 32 if form == "fresh" or prec == "fp64" else 5.3e10
        R = max(2, min(R, int(cap / (K * nB))))
        R_block = {"fresh": 1, "shared": min(R, rng.choice([64, 128, 256, rng.randint(50, 400)])),
                   "static": R}[form]
        return dict(kind=kind, api=rng.choice(["sets", "end_to_end"]), precision=prec, K=K, R=R,
                    R_block=R_block, nB=nB, L0=L0, along_x=rng.random() < 0.6, eq3=eq3)
    if kind == "screen":
        n = _log_int(rng, 12, 256)
        K, R = _log_int(rng, 200, 65536), _log_int(rng, 8, 4096)
        form = rng.choice(["fresh", "shared", "shared", "static"])
        cap = 1.3e9 if form == "fresh" or prec == "fp64" else 4e12 if prec == "fp32" else 1e13
        K = max(64, min(K, int(cap / (8 * n * n))))
        R = max(4, min(R, int(cap / (K * n * n))))
        R_block = {"fresh": 1, "shared": min(R, rng.randint(9, 600)), "static": R}[form]
        return dict(kind=kind, precision=prec, K=K, n=n, side=round(rng.uniform(1.0, 40.0), 3),
                    disk=rng.random() < 0.4, R=R, R_block=R_block, L0=L0, eq3=eq3)
    if kind == "apertures":
        n_ap = _log_int(rng, 2, 1500)
        K, R = _log_int(rng, 256, 16384), _log_int(rng, 32, 20000)
        cap = 1e9 if prec == "fp64" else 2e11
        K = max(64, min(K, int(cap / (32 * n_ap))))
        R = max(8, min(R, int(cap / (K * n_ap))))
        R_block = rng.choice([R, min(R, rng.randint(9, 400)), min(R, 256)])
        return dict(kind=kind, precision=prec, K=K, n_ap=n_ap, R=R, R_block=R_block, L0=L0,
                    tilt=rng.random() < 0.5, eq3=eq3)
    if kind == "temporal":
        N, M = rng.randint(16, 60), _log_int(rng, 64, 2000)
        R = max(8, min(_log_int(rng, 40, 2000), int(8e9 / (N * N * 2 * M))))
        return dict(kind=kind, precision=rng.choice(["fp64", "fp64", "fp32", "bf16x6"]), N=N, M=M,
                    R=R, R_block=rng.choice([1, 1, min(R, 50)]), L0=round(rng.uniform(10, 60), 2))
    if kind == "batch":
        R = rng.randint(20, 256)
        return dict(kind=kind, precision=rng.choice(["fp16x3", "bf16x6", "split_bf16"]),
                    n_inst=rng.randint(2, 12), k_lo=200, k_hi=_log_int(rng, 1000, 30000), n_lo=8,
                    n_hi=_log_int(rng, 32, 256), R=R,
                    R_block=rng.choice([R, R, max(9, R // 3)]), apertures=rng.random() < 0.3)
    n_ctx = rng.randint(16, 96)
    return dict(kind="train", n_ctx=n_ctx, m=_log_int(rng, 200, 4096),
                ctx_per_step=rng.randint(4, 16), steps=rng.randint(4, 24),
                G=rng.choice([32, 64, 100]))


# ------------------------------------------------------- inputs and passes ----
_context = []


def _ctx():
    """The one context a program keeps."""
    if not _context:
        _context.append(q.Context(0))
    return _context[0]


def _dev(a):
    return torch.as_tensor(np.ascontiguousarray(a, dtype=np.float64)).to(DEV)


def _seeds(seed):
    """R2 seeds (0.64 fixed point), Philox key and first realisation."""
    g = np.random.default_rng([seed, 71])
    sx, sy, key = (int(v) for v in g.integers(0, 1 << 64, 3, dtype=np.uint64))
    return dict(sx=sx, sy=sy, key=key, counter=int(g.integers(0, 1 << 30)))


def _grid(case):
    """Points of a screen: a regular grid, or its part inside the pupil."""
    if case["disk"]:
        return workloads.disk_mask_points(case["n"], case["side"])
    return workloads.grid_points(case["n"], 0.0, case["side"])


def _baselines(case, seed):
    bx, by = workloads.baselines(case["nB"])
    if not case["along_x"]:
        th = np.random.default_rng([seed, 72]).uniform(0.0, math.pi, case["nB"])
        bx, by = bx * np.cos(th), bx * np.sin(th)
    return bx, by


def _apertures(case, seed):
    """Centres over a 130 m array and unequal, partly obstructed apertures."""
    g = np.random.default_rng([seed, 73])
    n = case["n_ap"]
    cx, cy = g.uniform(0.0, 130.0, n), g.uniform(0.0, 130.0, n)
    D = np.where(g.random(n) < 0.5, 1.8, np.exp(g.uniform(math.log(0.5), math.log(8.2), n)))
    return cx, cy, D, np.where(g.random(n) < 0.5, 0.0, 0.14 * D)


def _instances(case, seed):
    """Sizes from the case alone, draws from the seed."""
    g = np.random.default_rng([case["n_inst"], case["k_hi"], case["n_hi"]])
    h = np.random.default_rng([seed, 74])
    out = []
    for i in range(case["n_inst"]):
        D = float(g.uniform(0.5, 39.0))
        n = int(round(math.exp(g.uniform(math.log(case["n_lo"]), math.log(case["n_hi"])))))
        K = int(round(math.exp(g.uniform(math.log(case["k_lo"]), math.log(case["k_hi"])))))
        px, py = workloads.disk_mask_points(n, D)
        d = dict(px=px, py=py, K=K, L0=float(g.uniform(10.0, 100.0)),
                 sx=int(h.integers(0, 1 << 64, dtype=np.uint64)), key=int(h.integers(0, 1 << 62)),
                 R=case["R"] - 3 * (i % 3), counter=1000 * i, apD=None, apd=None)
        d["R_block"] = min(d["R"], case["R_block"])
        if case["apertures"] and i % 2:
            d["apD"] = np.full(px.size, max(0.1, D / n))
            d["apd"] = np.zeros(px.size)
        out.append(d)
    return out


def _prepare_train(case, seed):
    """Contexts and rows (ln f, angle, variance share) of the plain sampler."""
    ctx4 = workloads.proposal_contexts(case["n_ctx"], seed=seed)
    s = q.logpolar_sampler(workloads.FMIN, workloads.FMAX, index=(seed % 1000003) * 4096)
    init = torch.as_tensor(workloads.mlp_init(seed), dtype=torch.float32).to(DEV)
    p = q.Proposal(_ctx(), workloads.FMIN, workloads.FMAX, init)
    c = _dev(ctx4)
    rows = p.rows(s, c, case["m"], R0)
    return dict(ctx4=c, rows=rows, init=init, shuffle=seed & 0xffffffff)


def prepare(case, seed):
    st = dict(case=case, ctx=_ctx(), prec=PREC.get(case.get("precision")), **_seeds(seed))
    st["mode"] = q.COEF_EQ3 if case.get("eq3") else q.COEF_GAUSS_CS
    kind = case["kind"]
    if kind == "structure":
        st["bx"], st["by"] = (_dev(v) for v in _baselines(case, seed))
    elif kind == "screen":
        st["px"], st["py"] = (_dev(v) for v in _grid(case))
    elif kind == "apertures":
        st["ap"] = [_dev(v) for v in _apertures(case, seed)]
    elif kind == "batch":
        inst = []
        for d in _instances(case, seed):
            i = dict(psd=q.psd(R0, d["L0"]), K=d["K"], px=_dev(d["px"]), py=_dev(d["py"]),
                     sampler=q.logpolar_sampler(workloads.FMIN, workloads.FMAX, seed_x=d["sx"]),
                     R=d["R"], R_block=d["R_block"], rng=q.Rng(d["key"], d["counter"], 0))
            if d["apD"] is not None:
                i["apD"], i["apd"] = _dev(d["apD"]), _dev(d["apd"])
            inst.append(i)
        st["batch"] = q.Batch(_ctx(), inst, precision=st["prec"])
    elif kind == "train":
        st.update(_prepare_train(case, seed))
    return st


def _trained(prm):
    """The parameters but for b3[0]: the density is exp(o0) over its own sum,
    so that bias changes nothing, its gradient is zero but for rounding, and
    Adam scales that rounding up to full steps."""
    return torch.cat([prm[:-2], prm[-1:]])


def _sampler(st):
    return q.logpolar_sampler(workloads.FMIN, workloads.FMAX, seed_x=st["sx"], seed_y=st["sy"])


def run(st):
    case, ctx, prec = st["case"], st["ctx"], st["prec"]
    kind = case["kind"]
    if kind == "batch":
        return list(st["batch"].execute(use_graph=True))
    if kind == "train":
        prop = q.Proposal(ctx, workloads.FMIN, workloads.FMAX, st["init"])
        prop.train(st["ctx4"], *st["rows"], steps=case["steps"],
                   ctx_per_step=case["ctx_per_step"], G=case["G"], lr=2e-3, seed=st["shuffle"])
        return _trained(prop.params())
    rng = q.Rng(st["key"], st["counter"], st.get("mode", 0))
    psd = q.psd(R0, case["L0"])
    R, Rb = case["R"], case["R_block"]
    if kind == "temporal":
        s = q.cartesian_sampler(case["N"], 0.25 / 22.0, seed_x=st["sx"], seed_y=st["sy"])
        sf, se = ctx.temporal_piston_structure(
            psd, q.Aperture(8.0, 1.1), (0.0, 0.0), (56.5, 0.0), (10.2, 0.0), 1e-3, case["M"], s,
            case["N"] ** 2, R, Rb, rng=rng, precision=prec)
        return dict(sf=sf, se=se)
    K, n_sets, s = case["K"], math.ceil(R / Rb), _sampler(st)
    if kind == "structure":
        ap = q.Aperture(1.8, 0.0)
        if case["api"] == "end_to_end":
            sf, se = ctx.diff_piston_structure(psd, ap, st["bx"], st["by"], s, K, R, Rb, rng=rng,
                                               precision=prec)
        else:
            f = ctx.sample_weights(s, n_sets, K, psd, ap, precision=prec)
            sf, se = ctx.diff_piston_structure_sets(K, *f, st["bx"], st["by"], R, Rb, rng=rng,
                                                    precision=prec)
        return dict(sf=sf, se=se)
    fx, fy, area = ctx.sample_frequencies(s, n_sets, K)
    w = ctx.weights(psd, fx, fy, area)
    if kind == "screen":
        return ctx.synthesize_phase(K, fx, fy, w, st["px"], st["py"], R, Rb, rng=rng,
                                    precision=prec)
    if case["tilt"]:
        return ctx.tilt(K, fx, fy, w, *st["ap"], (0.6, 0.8), R, Rb, rng=rng, precision=prec)
    return ctx.piston(K, fx, fy, w, *st["ap"], R, Rb, rng=rng, precision=prec)


def _n_points(case):
    if not case["disk"]:
        return case["n"] ** 2
    return workloads.disk_mask_points(case["n"], case["side"])[0].size


def work(case):
    """Reads and writes of the arrays the program holds or gets; 4 flops per
    term (r, k, p) and 16 operations per drawn coefficient."""
    kind = case["kind"]
    if kind == "batch":
        ds = _instances(case, 0)
        return {"bytes": float(sum(4 * d["R"] * d["px"].size + 16 * d["px"].size for d in ds)),
                "flops": float(sum(4 * d["R"] * d["K"] * d["px"].size + 32 * d["R"] * d["K"]
                                   for d in ds))}
    if kind == "train":
        rows = case["ctx_per_step"] * (case["m"] + case["G"])
        return {"bytes": float(case["steps"] * case["ctx_per_step"] * case["m"] * 24 + 8 * 17538),
                "flops": float(case["steps"] * rows * 6 * (5 * 128 + 128 * 128 + 256))}
    R = case["R"]
    n_sets = math.ceil(R / case["R_block"])
    esize = 8 if case["precision"] == "fp64" else 4
    if kind == "temporal":
        K, M = case["N"] ** 2, case["M"]
        return {"bytes": 16.0 * M, "flops": 8.0 * R * K * M + 32.0 * R * K + 1.5 * R * M * M}
    K = case["K"]
    if kind == "structure":
        freq = 24 * n_sets * K if case["api"] == "sets" else 0
        return {"bytes": float(2 * freq + 32 * case["nB"]),
                "flops": 4.0 * R * K * case["nB"] + 32.0 * R * K}
    P = _n_points(case) if kind == "screen" else case["n_ap"]
    return {"bytes": float(7 * 8 * n_sets * K + 16 * P + esize * R * P),
            "flops": 4.0 * R * K * P + 32.0 * R * K}


# ------------------------------------------------- the same in 64 bits ----
def _r2_increments():
    """round(2^64 / psi^j), psi the real root of x^3 = x + 1."""
    with decimal.localcontext() as c:
        c.prec = 60
        x = decimal.Decimal("1.3247")
        for _ in range(8):
            x -= (x ** 3 - x - 1) / (3 * x * x - 1)
        return [int((decimal.Decimal(1 << 64) / x ** j).to_integral_value()) for j in (1, 2)]


def _signed(v):
    v &= (1 << 64) - 1
    return v - (1 << 64) if v >> 63 else v


def _r2(n, sx, sy):
    """Points 1 .. n of the sequence, as binary64 in [0, 1)."""
    i = torch.arange(1, n + 1, dtype=torch.int64, device=DEV)
    return [((_signed(s) + i * _signed(a)) >> 11 & ((1 << 53) - 1)).double() * 2.0 ** -53
            for s, a in zip((sx, sy), _r2_increments())]


def _filter(f, D, d):
    """Aperture filter 2 (D J1(pi D f) - d J1(pi d f)) / (pi (D^2 - d^2) f)."""
    pf = math.pi * torch.clamp(f, min=1e-300)
    j1 = torch.special.bessel_j1
    return 2 * (D * j1(pf * D) - d * j1(pf * d)) / ((D * D - d * d) * pf)


def _weights(fx, fy, area, L0, ap=None):
    c = math.gamma(11 / 6) ** 2 / (2 * math.pi ** (11 / 3)) * (4.8 * math.gamma(1.2)) ** (5 / 6)
    f2 = fx * fx + fy * fy
    w = torch.sqrt(c * R0 ** (-5 / 3) * (f2 + L0 ** -2) ** (-11 / 6) * area)
    return w if ap is None else w * _filter(torch.sqrt(f2), *ap)


def _logpolar(n_sets, K, sx, sy, L0, ap=None):
    ux, uy = _r2(n_sets * K, sx, sy)
    lr = math.log(workloads.FMAX / workloads.FMIN)
    f = workloads.FMIN * torch.exp(lr * ux)
    fx, fy = f * torch.cos(2 * math.pi * uy), f * torch.sin(2 * math.pi * uy)
    w = _weights(fx, fy, 2 * math.pi * lr * f * f / K, L0, ap)
    return fx.view(n_sets, K), fy.view(n_sets, K), w.view(n_sets, K)


M32 = 0xffffffff


def _philox(t, real, seed):
    """Philox4x32-10 words of counter (t, real lo, real hi, 0)."""
    t, real = torch.broadcast_tensors(t, real)
    c0, c1, c2, c3 = t & M32, real & M32, real >> 32 & M32, torch.zeros_like(t)
    k0, k1 = seed & M32, seed >> 32 & M32
    for _ in range(10):
        p0, p1 = c0 * 0xD2511F53, c2 * 0xCD9E8D57
        c0, c1, c2, c3 = (p1 >> 32 & M32) ^ c1 ^ k0, p1 & M32, (p0 >> 32 & M32) ^ c3 ^ k1, p0 & M32
        k0, k1 = (k0 + 0x9E3779B9) & M32, (k1 + 0xBB67AE85) & M32
    return c0, c1, c2, c3


def _coefs(rows, K, key, counter, eq3):
    """Coefficients [rows][K] of cos and of sin for realisations `rows`."""
    nt = K if eq3 else (K + 1) // 2
    real = (rows + counter)[:, None]
    u = [((x >> 9).double() + 0.5) * 2.0 ** -23
         for x in _philox(torch.arange(nt, device=DEV)[None, :], real, key)]
    rho = torch.sqrt(-2 * torch.log(u[0]))
    if eq3:
        g = math.sqrt(2) * rho * torch.cos(2 * math.pi * u[1])
        return g * torch.cos(2 * math.pi * u[2]), -g * torch.sin(2 * math.pi * u[2])
    rho2 = torch.sqrt(-2 * torch.log(u[2]))
    a = torch.stack([rho * torch.cos(2 * math.pi * u[1]), rho2 * torch.cos(2 * math.pi * u[3])], 2)
    b = torch.stack([rho * torch.sin(2 * math.pi * u[1]), rho2 * torch.sin(2 * math.pi * u[3])], 2)
    return a.flatten(1)[:, :K].contiguous(), b.flatten(1)[:, :K].contiguous()


def _cycles(fx, fy, px, py):
    """f.x modulo one cycle, [K][P]."""
    t = fx[:, None] * px[None, :] + fy[:, None] * py[None, :]
    return t - torch.round(t)


def _sums(fx, fy, w, px, py, R, Rb, key, counter, eq3=False, diff=False, ap=None, u=None):
    """Eq. 3 at the points: [R][P].  diff: minus its value at the origin;
    ap: times the filters of apertures (D, d) [P]; u: gradient along u."""
    n_sets, K = fx.shape
    P = px.numel()
    out = torch.empty((R, P), dtype=F64, device=DEV)
    rows_max = max(Rb, (1 << 25) // K // Rb * Rb) if Rb * K < 1 << 25 else 256
    cols = max(1, min(P, (1 << 26) // K))
    for r0 in range(0, R, rows_max):
        # rows of whole sets, or part of the rows of one set
        r1 = min(R, r0 + rows_max) if rows_max >= Rb else min(R, r0 + rows_max, (r0 // Rb + 1) * Rb)
        a, b = _coefs(torch.arange(r0, r1, device=DEV), K, key, counter, eq3)
        for s in range(r0 // Rb, (r1 - 1) // Rb + 1):
            i, j = max(r0, s * Rb), min(r1, (s + 1) * Rb)
            aw, bw = a[i - r0:j - r0] * w[s], b[i - r0:j - r0] * w[s]
            for p in range(0, P, cols):
                e = min(P, p + cols)
                t = 2 * math.pi * _cycles(fx[s], fy[s], px[p:e], py[p:e])
                if diff:
                    c, sn = -2 * torch.sin(t / 2) ** 2, torch.sin(t)
                elif u is not None:
                    g = 2 * math.pi * (u[0] * fx[s] + u[1] * fy[s])[:, None]
                    c, sn = -g * torch.sin(t), g * torch.cos(t)
                else:
                    c, sn = torch.cos(t), torch.sin(t)
                if ap is not None:
                    F = _filter(torch.hypot(fx[s], fy[s])[:, None], ap[0][None, p:e],
                                ap[1][None, p:e])
                    c, sn = c * F, sn * F
                out[i:j, p:e] = aw @ c + bw @ sn
    return out


def _sums_static(fx, fy, w, px, py, R, key, counter, eq3):
    """One set for all realisations and many points: coefficients held once."""
    K, P = fx.shape[1], px.numel()
    a, b = (torch.empty((R, K), dtype=F64, device=DEV) for _ in range(2))
    for r0 in range(0, R, 128):
        r1 = min(R, r0 + 128)
        c, s = _coefs(torch.arange(r0, r1, device=DEV), K, key, counter, eq3)
        a[r0:r1], b[r0:r1] = c * w[0], s * w[0]
    out = torch.empty((R, P), dtype=F64, device=DEV)
    cols = max(1, min(P, (1 << 26) // K))
    for p in range(0, P, cols):
        e = min(P, p + cols)
        t = 2 * math.pi * _cycles(fx[0], fy[0], px[p:e], py[p:e])
        out[:, p:e] = a @ torch.cos(t) + b @ torch.sin(t)
    return out


def _diff_fresh(fx, fy, w, bx, by, R, key, counter, eq3):
    """Differential pistons when every realisation has its own frequencies."""
    K = fx.shape[1]
    out = torch.empty((R, bx.numel()), dtype=F64, device=DEV)
    step = max(1, (1 << 25) // (K * bx.numel()))
    for r0 in range(0, R, step):
        r1 = min(R, r0 + step)
        a, b = _coefs(torch.arange(r0, r1, device=DEV), K, key, counter, eq3)
        t = fx[r0:r1, :, None] * bx + fy[r0:r1, :, None] * by
        t = 2 * math.pi * (t - torch.round(t))
        out[r0:r1] = ((a * w[r0:r1])[:, :, None] * (-2 * torch.sin(t / 2) ** 2)
                      + (b * w[r0:r1])[:, :, None] * torch.sin(t)).sum(1)
    return out


def _mean_and_error(v):
    """Mean over realisations and its standard error, per column."""
    R = v.shape[0]
    s1, s2 = v.sum(0), (v * v).sum(0)
    var = (s2 - s1 * s1 / R) / max(1, R - 1)
    return dict(sf=s1 / R, se=torch.sqrt(torch.clamp(var, min=0.0) / R))


def _exact_train(case, seed):
    """The same steps of Adam on the cross-entropy, by autograd in binary64."""
    st = _prepare_train(case, seed)
    (ell, theta, h), ctx4 = st["rows"], st["ctx4"]
    m, G, n_ctx, per = case["m"], case["G"], case["n_ctx"], case["ctx_per_step"]
    lmin, Lw = math.log(workloads.FMIN), math.log(workloads.FMAX / workloads.FMIN)
    grid = lmin + (torch.arange(G, dtype=F64, device=DEV) + 0.5) * Lw / G
    prm = st["init"].double().clone().requires_grad_(True)
    m1, m2 = torch.zeros_like(prm), torch.zeros_like(prm)

    def net(l, c):
        x = torch.stack([2 * (l - lmin) / Lw - 1, 2 * c[:, 3] / math.pi - 1, torch.log(c[:, 0]) / 4,
                         torch.log(c[:, 1]) / 4 - 1, torch.log(c[:, 2]) / 4 - 0.5], 1)
        W1, b1, W2, b2, W3, b3 = torch.split(prm, [640, 128, 16384, 128, 256, 2])
        y = torch.tanh(x @ W1.view(128, 5).t() + b1)
        y = torch.tanh(y @ W2.view(128, 128).t() + b2)
        return y @ W3.view(2, 128).t() + b3

    order, state, pos = list(range(n_ctx)), st["shuffle"], n_ctx
    for t in range(1, case["steps"] + 1):
        ids = []
        for _ in range(per):
            if pos == n_ctx:
                for k in range(n_ctx - 1, 0, -1):
                    state = state + 0x9E3779B97F4A7C15 & (1 << 64) - 1
                    z = state
                    z = (z ^ z >> 30) * 0xBF58476D1CE4E5B9 & (1 << 64) - 1
                    z = (z ^ z >> 27) * 0x94D049BB133111EB & (1 << 64) - 1
                    j = (z ^ z >> 31) % (k + 1)
                    order[k], order[j] = order[j], order[k]
                pos = 0
            ids.append(order[pos])
            pos += 1
        c = ctx4.view(n_ctx, 4)[ids]
        l, th, hh = (v.view(n_ctx, m)[ids] for v in (ell, theta, h))
        o = net(l.flatten(), c.repeat_interleave(m, 0)).view(per, m, 2)
        og = net(grid.repeat(per), c.repeat_interleave(G, 0)).view(per, G, 2)[:, :, 0]
        logq = o[:, :, 0] - (torch.logsumexp(og, 1) + math.log(Lw / G))[:, None] + torch.log(
            1 + 0.9 * torch.tanh(o[:, :, 1]) * torch.cos(2 * (th - c[:, 3:4])))
        loss = -(hh * logq).sum() / hh.sum()
        g, = torch.autograd.grad(loss, prm)
        m1, m2 = 0.9 * m1 + 0.1 * g, 0.999 * m2 + 0.001 * g * g
        with torch.no_grad():
            prm -= 2e-3 * (m1 / (1 - 0.9 ** t)) / (torch.sqrt(m2 / (1 - 0.999 ** t)) + 1e-8)
    return _trained(prm.detach())


def exact(case, seed):
    kind, g = case["kind"], _seeds(seed)
    key, counter, eq3 = g["key"], g["counter"], case.get("eq3", False)
    if kind == "train":
        return _exact_train(case, seed)
    if kind == "batch":
        out = []
        for d in _instances(case, seed):
            n_sets = math.ceil(d["R"] / d["R_block"])
            f = _logpolar(n_sets, d["K"], d["sx"], 1 << 63, d["L0"])
            ap = None if d["apD"] is None else (_dev(d["apD"]), _dev(d["apd"]))
            out.append(_sums(*f, _dev(d["px"]), _dev(d["py"]), d["R"], d["R_block"], d["key"],
                             d["counter"], ap=ap))
        return out
    R, Rb = case["R"], case["R_block"]
    n_sets = math.ceil(R / Rb)
    if kind == "temporal":
        K, M, L = case["N"] ** 2, case["M"], case["N"] * (0.25 / 22.0)
        ux, uy = _r2(n_sets * K, g["sx"], g["sy"])
        fx, fy = L * (ux - 0.5), L * (uy - 0.5)
        w = _weights(fx, fy, torch.full_like(fx, L * L / K), case["L0"], (8.0, 1.1))
        x = -10.2 * 1e-3 * torch.arange(M, dtype=F64, device=DEV)
        p = _sums(fx.view(n_sets, K), fy.view(n_sets, K), w.view(n_sets, K),
                  torch.cat([x, x + 56.5]), torch.zeros(2 * M, dtype=F64, device=DEV), R, Rb, key,
                  counter)
        dp = p[:, :M] - p[:, M:]
        v = torch.zeros((R, M), dtype=F64, device=DEV)
        for j in range(1, M):
            v[:, j] = ((dp[:, j:] - dp[:, :-j]) ** 2).mean(1)
        return _mean_and_error(v)
    K = case["K"]
    f = _logpolar(n_sets, K, g["sx"], g["sy"], case["L0"],
                  (1.8, 0.0) if kind == "structure" else None)
    if kind == "structure":
        b = [_dev(v) for v in _baselines(case, seed)]
        if Rb == 1:
            dp = _diff_fresh(*f, *b, R, key, counter, eq3)
        else:
            dp = _sums(*f, *b, R, Rb, key, counter, eq3, diff=True)
        return _mean_and_error(dp * dp)
    if kind == "screen":
        p = [_dev(v) for v in _grid(case)]
        if n_sets == 1:
            return _sums_static(*f, *p, R, key, counter, eq3)
        return _sums(*f, *p, R, Rb, key, counter, eq3)
    cx, cy, D, d = (_dev(v) for v in _apertures(case, seed))
    return _sums(*f, cx, cy, R, Rb, key, counter, eq3, ap=(D, d),
                 u=(0.6, 0.8) if case["tilt"] else None)
