"""The work that users of this library have it do, as cases that can be timed and
compared: the fitness, the multi-wavelength objective, the relaxation with its
adjoint, the optimiser's steps, and whole single-design and batched runs, all
through the Python binding.

A case is a dict of plain values; `listed()` names the ones that stand for the
workloads of the benchmark and the tests, `draw(rng)` gives more of the same
ranges, `prepare` makes a program's state on the GPU (designs, packed genomes,
genes, theta), `run` is one pass, `work` its unavoidable bytes and operations
and `exact` the same outputs in 64-bit arithmetic.
"""
import math

import numpy as np
import torch

from paper_2511_01255_amd import inputs, qpm

PREC = {"f32": qpm.PREC_F32, "f64": qpm.PREC_F64}
SHG_PERIODS = (6.2, 6.9, 8.1, 9.3, 11.7, 7.4, 10.2, 12.5)  # um
THG_DKS = ((inputs.DK1, inputs.DK2), (0.30, 0.90), (0.31, 0.97), (0.35, 0.88))  # 1/um
U32 = 0xFFFFFFFF


def listed():
    return [
        # the smallest evaluation: a script that scores a handful of designs
        # of the plain configuration (N = 256, NP = 32); latency and launches
        {"name": "fitness-256x32-f64", "kind": "fitness", "n": 256, "np": 32, "prec": "f64", "jitter": 0.0},
        # the fitness-throughput population: iid genomes and periodic seeds
        {"name": "fitness-10000x4096-f32", "kind": "fitness", "n": 10000, "np": 4096, "prec": "f32", "jitter": 0.0},
        # a long crystal with uneven domains and a ragged population, FP64
        {"name": "fitness-49999x1001-f64", "kind": "fitness", "n": 49999, "np": 1001, "prec": "f64", "jitter": 0.3},
        # scoring 64 independent uneven designs in one call
        {"name": "batch-fitness-64x256-f32", "kind": "batch_fitness", "inst": 64, "n_lo": 1000, "n_hi": 50000,
         "np": 256, "prec": "f32"},
        # the five-wavelength second-harmonic objective, 9 mm crystal
        {"name": "objective-shg5-3000x5000-f32", "kind": "objective", "n": 3000, "np": 5000, "prec": "f32",
         "obj": "shg", "K": 5},
        # gradient design: the relaxation and its adjoint through autograd
        {"name": "relax-50000x256-f32", "kind": "relax", "n": 50000, "B": 256, "prec": "f32"},
        # the same in FP64 on a ragged batch of a ragged crystal
        {"name": "relax-9999x100-f64", "kind": "relax", "n": 9999, "B": 100, "prec": "f64"},
        # one DE step of a caller's own loop, benchmark population
        {"name": "de-10000x4096", "kind": "de", "n": 10000, "np": 4096, "F": 0.5, "CR": 0.9},
        # one grey-wolf step of a caller's own loop, the paper's population
        {"name": "gwo-6600x5000", "kind": "gwo", "n": 6600, "np": 5000, "a": 1.3, "variant": 0},
        # the plain configuration, whole: N = 256, NP = 32, 200 generations
        {"name": "run-256x32-f64", "kind": "run", "n": 256, "np": 32, "G": 200, "prec": "f64", "control": "fixed",
         "algo": "hwsda", "variant": 0, "obj": "deff", "K": 1},
        # a whole run of the N = 10^4, NP = 1024 configuration
        {"name": "run-10000x1024-f32", "kind": "run", "n": 10000, "np": 1024, "G": 300, "prec": "f32",
         "control": "fixed", "algo": "hwsda", "variant": 0, "obj": "deff", "K": 1},
        # uneven designs optimised together, NP = 256 each
        {"name": "batch-run-32x256-f32", "kind": "batch_run", "inst": 32, "n_lo": 1000, "n_hi": 50000, "np": 256,
         "G": 20, "prec": "f32"},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case of the listed ranges; no dearer than the dearest listed one."""
    kind = rng.choice(["fitness", "fitness", "batch_fitness", "objective", "relax", "relax", "de", "gwo", "run",
                       "run", "run", "batch_run"])
    prec = rng.choice(["f32", "f64"])
    n = _log(rng, 256, 50000)
    if kind == "fitness":
        return {"kind": kind, "n": n, "np": _log(rng, 32, min(8192, 10 ** 8 // n)), "prec": prec,
                "jitter": rng.choice([0.0, 0.3])}
    if kind == "batch_fitness":
        lo = _log(rng, 256, 4000)
        return {"kind": kind, "inst": _log(rng, 4, 64), "n_lo": lo, "n_hi": lo * rng.randint(2, 12),
                "np": _log(rng, 32, 512), "prec": prec}
    if kind == "objective":
        obj = rng.choice(["shg", "thg"])
        n = _log(rng, 256, 13200)
        return {"kind": kind, "n": n, "np": _log(rng, 64, min(5000, 2 * 10 ** 7 // n)), "prec": prec, "obj": obj,
                "K": rng.randint(2, 5) if obj == "shg" else rng.randint(1, 3)}
    if kind == "relax":
        return {"kind": kind, "n": n, "B": _log(rng, 3, 256 if prec == "f32" else 64), "prec": prec}
    if kind == "de":
        return {"kind": kind, "n": n, "np": _log(rng, 32, min(8192, 5 * 10 ** 7 // n)), "F": rng.choice([0.5, 0.05, 0.8]),
                "CR": rng.choice([0.9, 0.5])}
    if kind == "gwo":
        return {"kind": kind, "n": n, "np": _log(rng, 32, min(8192, 5 * 10 ** 7 // n)),
                "a": round(rng.uniform(0.02, 2.0), 3), "variant": rng.choice([0, 0, 1])}
    if kind == "batch_run":
        lo = _log(rng, 256, 4000)
        return {"kind": kind, "inst": _log(rng, 4, 24), "n_lo": lo, "n_hi": lo * rng.randint(2, 6),
                "np": rng.choice([64, 100, 128, 250]), "G": rng.randint(10, 20), "prec": prec}
    # runs: from the plain configuration to the paper's NP = 5000
    n = _log(rng, 200, 13200)
    np_ = _log(rng, 16, min(5000, 2 * 10 ** 7 // n))
    G = max(20, min(200, int(10 ** 9 / (n * np_))))
    obj = rng.choice(["deff", "deff", "deff", "shg", "thg"])
    return {"kind": "run", "n": n, "np": np_, "G": G, "prec": prec,
            "control": rng.choice(["fixed", "decay"] if obj != "deff" else ["fixed", "fixed", "decay", "adaptive"]),
            "algo": rng.choice(["hwsda", "hwsda", "hwsda", "de", "gwo"]), "variant": rng.choice([0, 0, 0, 1, 2]),
            "obj": obj, "K": {"deff": 1, "shg": rng.randint(2, 5), "thg": rng.randint(1, 3)}[obj]}


# ------------------------------------------------------------------ inputs


def _gen(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed) & 0x7FFFFFFF)
    return g


def _boundaries(case, seed):
    n, w = case["n"], (0.1 if case["kind"] == "run" and case["np"] > 4096 else 2.0)
    if case["kind"] == "objective" or case.get("obj") in ("shg", "thg"):
        w = 3.0
    if case.get("jitter"):
        return inputs.jittered_boundaries(n, w, case["jitter"], seed)
    return inputs.uniform_boundaries(n, w)


def _dks(case):
    obj, K = case.get("obj", "deff"), case.get("K", 1)
    if obj == "shg":
        return [(2.0 * math.pi / p, 0.0) for p in SHG_PERIODS[:K]]
    return list(THG_DKS[:K])


def _specs(case, seed):
    """(z, dk1, dk2) of a batch's designs; sizes are the case's own, the rest follows the seed."""
    sizes = np.random.default_rng(case["inst"]).integers(case["n_lo"], case["n_hi"] + 1, size=case["inst"])
    rng = np.random.default_rng(seed)
    return [(inputs.uniform_boundaries(int(n), rng.uniform(1.5, 3.0)), 2.0 * math.pi / rng.uniform(18.0, 21.0),
             2.0 * math.pi / rng.uniform(6.2, 7.0)) for n in sizes]


def _pack(neg):
    """bool (np, n) -> int32 words (W, np) of the population-major layout."""
    m, n = neg.shape
    W = inputs.words(n)
    full = torch.zeros((m, W * 32), dtype=torch.int64, device=neg.device)
    full[:, :n] = neg
    w = (full.view(m, W, 32) << torch.arange(32, device=neg.device)).sum(-1)
    return torch.where(w > 0x7FFFFFFF, w - (1 << 32), w).to(torch.int32).t().contiguous()


def _genomes(gen, n, np_, z, n_periodic):
    """Packed genomes: iid signs, the last n_periodic first-order periodic seeds with random phases."""
    W, ld = inputs.words(n), inputs.ld_for(np_)
    bits = torch.randint(-(1 << 31), 1 << 31, (W, ld), generator=gen, device="cuda", dtype=torch.int64).to(torch.int32)
    if n_periodic:
        zt = torch.from_numpy(z).cuda()
        mid = 0.5 * (zt[1:] + zt[:-1])
        phi = torch.rand(n_periodic, 1, generator=gen, device="cuda", dtype=torch.float64) * 19.5
        bits[:, np_ - n_periodic:np_] = _pack(torch.cos(2.0 * math.pi / 19.5 * (mid[None] - phi)) < 0)
    if n % 32:
        bits[-1] &= (1 << (n % 32)) - 1
    bits[:, np_:] = 0
    return bits


def prepare(case, seed):
    kind, gen = case["kind"], _gen(seed)
    if kind == "fitness":
        z = _boundaries(case, seed)
        return {"case": case, "design": qpm.precompute_phases(z, inputs.DK1, inputs.DK2),
                "bits": _genomes(gen, case["n"], case["np"], z, min(32, case["np"] // 4))}
    if kind == "batch_fitness":
        specs = _specs(case, seed)
        batch = qpm.precompute_phases_batched(*[[s[k] for s in specs] for k in range(3)])
        bits = torch.cat([_genomes(gen, len(s[0]) - 1, case["np"], s[0], 0) for s in specs])
        return {"case": case, "batch": batch, "bits": bits}
    if kind == "objective":
        z = _boundaries(case, seed)
        obj = qpm.Objective([qpm.precompute_phases(z, a, b) for a, b in _dks(case)],
                            qpm.OBJ_SHG if case["obj"] == "shg" else qpm.OBJ_THG, 1.0, 1.0)
        return {"case": case, "obj": obj, "bits": _genomes(gen, case["n"], case["np"], z, 0)}
    if kind == "relax":
        theta = torch.randn(case["B"], case["n"], generator=gen, device="cuda").requires_grad_()
        return {"case": case, "design": qpm.precompute_phases(_boundaries(case, seed), inputs.DK1, inputs.DK2),
                "theta": theta, "w": torch.rand(case["B"], generator=gen, device="cuda") + 0.5}
    if kind in ("de", "gwo"):
        x = torch.zeros(case["np"], qpm.ldx_for(case["n"]), device="cuda")
        x[:, :case["n"]] = torch.rand(case["np"], case["n"], generator=gen, device="cuda") * 2.0 - 1.0
        leaders = np.random.default_rng(seed).choice(case["np"], 3, replace=False).astype(np.int32)
        return {"case": case, "x": x, "leaders": leaders, "seed": int(seed)}
    if kind == "run":
        z = _boundaries(case, seed)
        d = [qpm.precompute_phases(z, a, b) for a, b in _dks(case)]
        if case["obj"] != "deff":
            d = [qpm.Objective(d, qpm.OBJ_SHG if case["obj"] == "shg" else qpm.OBJ_THG, 1.0, 1.0)]
        return {"case": case, "design": d[0], "seed": int(seed)}
    specs = _specs(case, seed)
    return {"case": case, "batch": qpm.precompute_phases_batched(*[[s[k] for s in specs] for k in range(3)]),
            "seed": int(seed)}


# ------------------------------------------------------------------ one pass


def run(state):
    case = state["case"]
    kind, prec = case["kind"], PREC.get(case.get("prec"))
    if kind == "fitness":
        return qpm.eval_fitness(state["design"], state["bits"], case["np"], prec)
    if kind == "batch_fitness":
        return qpm.batch_eval_fitness(state["batch"], state["bits"], case["np"], prec)
    if kind == "objective":
        return qpm.eval_objective(state["obj"], state["bits"], case["np"], prec, with_G=True)
    if kind == "relax":
        f = qpm.relax(state["theta"], state["design"], prec)
        (g,) = torch.autograd.grad(f, state["theta"], state["w"])
        return f.detach(), g
    if kind == "de":
        return qpm.de_step(state["x"], case["n"], case["F"], case["CR"], state["seed"], 3)
    if kind == "gwo":
        return qpm.gwo_step(state["x"], case["n"], state["leaders"], case["a"], state["seed"], 3,
                            variant=case["variant"])
    if kind == "run":
        R = qpm.Run(state["design"], case["np"], case["G"], seed=state["seed"], prec=prec,
                    gwo_variant=case["variant"],
                    control={"fixed": qpm.CONTROL_FIXED, "decay": qpm.CONTROL_DECAY,
                             "adaptive": qpm.CONTROL_ADAPTIVE}[case["control"]],
                    algo={"hwsda": qpm.ALGO_HWSDA, "de": qpm.ALGO_DE, "gwo": qpm.ALGO_GWO}[case["algo"]])
        R.advance(case["G"])
        x, f, leaders, _ = R.read()
        R.destroy()
        return x, f, leaders
    # (tune off: the launch shape follows the sizes, not a timing)
    R = qpm.BatchRun(state["batch"], case["np"], case["G"], seed=state["seed"], prec=prec, tune=0)
    R.advance(case["G"])
    out = [R.read(b) for b in range(case["inst"])]
    R.destroy()
    return [o[0] for o in out], torch.stack([o[1] for o in out]), np.array([o[2] for o in out])


def work(case):
    """Inputs read once and outputs written once; a domain evaluation is 10
    operations, a relaxed one 15 forward and 20 in the adjoint, a DE gene 5
    and a grey-wolf gene 25."""
    kind = case["kind"]
    es = 8 if case.get("prec") == "f64" else 4
    if kind in ("batch_fitness", "batch_run"):
        total = sum(len(s[0]) - 1 for s in _specs(case, 0))
        if kind == "batch_fitness":
            return {"bytes": case["np"] * (total / 8 + es * case["inst"]) + 8 * total,
                    "flops": 10.0 * case["np"] * total}
        return {"bytes": case["np"] * (4.0 * total + es * case["inst"]) + 8 * total,
                "flops": case["G"] * (2 * case["np"] * 10.0 + case["np"] * 30.0) * total}
    n = case["n"]
    if kind == "relax":
        return {"bytes": 12.0 * case["B"] * n + 8 * n, "flops": 35.0 * case["B"] * n}
    np_ = case["np"]
    if kind == "fitness":
        return {"bytes": np_ * (n / 8 + es) + 8 * n, "flops": 10.0 * np_ * n}
    if kind == "objective":
        per = 10.0 if case["obj"] == "thg" else 2.0
        return {"bytes": np_ * (n / 8 + es + 8 * case["K"]) + 8 * n, "flops": per * case["K"] * np_ * n}
    if kind in ("de", "gwo"):
        return {"bytes": np_ * n * 8.125, "flops": (5.0 if kind == "de" else 25.0) * np_ * n}
    ev = {"deff": 10.0, "thg": 10.0 * case["K"], "shg": 2.0 * case["K"]}[case["obj"]]
    per = {"hwsda": 2 * ev + 30.0, "de": ev + 5.0, "gwo": ev + 25.0}[case["algo"]]
    return {"bytes": np_ * (4.0 * n + es) + 8 * n, "flops": case["G"] * per * np_ * n}


# ------------------------------------------------------------------ in 64 bits


def _integrals(z, k1, k2):
    """a, b (complex128 tensors) and c (numpy clongdouble parts) of the
    domains, the phases reduced in long double; dk2 = 0 and dk1 != 0 are fine."""
    zl = z.astype(np.longdouble)
    w, lo = zl[1:] - zl[:-1], zl[:-1]

    def E(k):
        h = np.longdouble(k) * w / 2
        s = np.where(np.abs(h) < 1e-6, 1 - h * h / 6, np.sin(h) / np.where(h == 0, 1, h))
        return w * s * np.cos(h), -w * s * np.sin(h)

    def mul(x, y):
        return x[0] * y[0] - x[1] * y[1], x[0] * y[1] + x[1] * y[0]

    def ph(k):
        return np.cos(np.longdouble(k) * lo), -np.sin(np.longdouble(k) * lo)

    e2, e12, p1, p2 = E(k2), E(np.longdouble(k1) + np.longdouble(k2)), ph(k1), ph(k2)
    a, b = mul(p1, E(k1)), mul(p2, e2)
    G = ((e2[1] - e12[1]) / np.longdouble(k1), -(e2[0] - e12[0]) / np.longdouble(k1))
    c = mul(mul(p1, p2), G)
    t = lambda v: [torch.from_numpy(u.astype(np.float64)).cuda() for u in v]  # noqa: E731
    return t(a), t(b), t(c), (float(c[0].sum()), float(c[1].sum()))


def _signs(bits, np_, n):
    """(np, n) +-1 doubles of int32 words (W, >= np)."""
    w = bits[:, :np_].t().to(torch.int64)
    b = (w[:, :, None] >> torch.arange(32, device=bits.device)) & 1
    return 1.0 - 2.0 * b.reshape(np_, -1)[:, :n].double()


def _deff(bits, np_, n, tabs, single=False):
    """d_eff (re, im) of the genomes, or sum d a with `single`."""
    a, b, _, C = tabs
    out = []
    step = max(1, 4_000_000 // n)
    for i in range(0, np_, step):
        d = _signs(bits[:, i:min(np_, i + step)], min(step, np_ - i), n)
        if single:
            out.append(torch.stack([(d * a[0]).sum(1), (d * a[1]).sum(1)]))
            continue
        ar, ai, br, bi = d * a[0], d * a[1], d * b[0], d * b[1]
        Pr, Pi = torch.cumsum(ar, 1) - ar, torch.cumsum(ai, 1) - ai
        out.append(torch.stack([(br * Pr - bi * Pi).sum(1) + C[0], (br * Pi + bi * Pr).sum(1) + C[1]]))
    return torch.cat(out, 1)


def _philox(c0, c1, c2, c3, seed):
    """Philox4x32-10 on int64 tensors holding 32-bit words."""
    k0, k1 = seed & U32, (seed >> 32) & U32

    def mul(m, x):
        t, u = m * (x & 0xFFFF), m * (x >> 16)
        v = u + (t >> 16)
        return v >> 16, ((v & 0xFFFF) << 16) | (t & 0xFFFF)

    for _ in range(10):
        (ah, al), (bh, bl) = mul(0xD2511F53, c0), mul(0xCD9E8D57, c2)
        c0, c1, c2, c3 = bh ^ c1 ^ k0, bl, ah ^ c3 ^ k1, al
        k0, k1 = (k0 + 0x9E3779B9) & U32, (k1 + 0xBB67AE85) & U32
    return c0, c1, c2, c3


def _rows(np_, n, r0, r1):
    i = torch.arange(r0, r1, device="cuda", dtype=torch.int64)[:, None]
    q = torch.arange((n + 3) // 4, device="cuda", dtype=torch.int64)[None]
    return i + 0 * q, q + 0 * i


def _exact_de(case, x, seed):
    np_, n, g = case["np"], case["n"], 3
    i = torch.arange(np_, device="cuda", dtype=torch.int64)
    zero = torch.zeros_like(i)
    o = [v.cpu().numpy() for v in _philox(zero, i, zero + g, zero + 2, seed)]
    r = np.zeros((3, np_), dtype=np.int64)
    for m in range(3):
        ex = np.sort(np.vstack([np.arange(np_)[None], r[:m]]), axis=0)
        k = (o[m] * (np_ - 1 - m)) >> 32
        for e in ex:
            k = k + (k >= e)
        r[m] = k
    jr = (o[3] * n) >> 32
    F = float(np.float32(case["F"]))
    cr = float(np.float32(case["CR"]))
    u = torch.zeros(np_, x.shape[1], device="cuda", dtype=torch.float64)
    for r0 in range(0, np_, 512):
        r1 = min(np_, r0 + 512)
        ii, qq = _rows(np_, n, r0, r1)
        w = torch.stack(_philox(qq, ii, 0 * qq + g, 0 * qq + 3, seed), -1).reshape(r1 - r0, -1)[:, :n]
        take = (w >> 8).double() * 2.0 ** -24 <= cr
        take[torch.arange(r1 - r0, device="cuda"), torch.from_numpy(jr[r0:r1]).cuda()] = True
        a, b, c = (x[torch.from_numpy(r[m][r0:r1]).cuda(), :n].double() for m in range(3))
        # (F, differences and clamp as the step states them; the difference is a binary32 one)
        v = (a + F * (b.float() - c.float()).double()).clamp(-1.0, 1.0)
        u[r0:r1, :n] = torch.where(take, v, x[r0:r1, :n].double())
    return u, None


def _exact_gwo(case, x, leaders, seed):
    np_, n, g = case["np"], case["n"], 3
    a = float(np.float32(case["a"]))
    y = x.double()
    X = [x[int(k), :n].double() for k in leaders]
    for r0 in range(0, np_, 512):
        r1 = min(np_, r0 + 512)
        ii, qq = _rows(np_, n, r0, r1)
        w = torch.cat([torch.stack(_philox(3 * qq + t, ii, 0 * qq + g, 0 * qq + 4, seed), -1) for t in range(3)], -1)
        w = w.reshape(r1 - r0, -1, 3)[:, :n]
        xs = x[r0:r1, :n].double()
        num, den = 0.0, 0.0
        for k in range(3):
            A = 2.0 * a * ((w[..., k] & 0xFFFF).double() * 2.0 ** -16) - a
            Y = X[k] - A * ((w[..., k] >> 16).double() * 2.0 ** -15 * X[k] - xs).abs()
            num = num + (Y if case["variant"] == 1 else Y.abs() * Y)
            den = den + (1.0 / 3.0 if case["variant"] == 1 else Y.abs())
        keep = torch.ones(r1 - r0, dtype=torch.bool, device="cuda")
        for k in leaders:
            if r0 <= k < r1:
                keep[int(k) - r0] = False
        new = torch.where(den == 0, torch.zeros_like(num), num / den / 3.0).clamp(-1.0, 1.0)
        y[r0:r1, :n] = torch.where(keep[:, None], new, xs)
    return y, None


def exact(case, seed):
    kind = case["kind"]
    if kind in ("run", "batch_run"):
        return None  # a trajectory of decisions
    if kind in ("de", "gwo"):
        s = prepare(case, seed)
        return _exact_de(case, s["x"], s["seed"]) if kind == "de" else _exact_gwo(case, s["x"], s["leaders"], s["seed"])
    gen = _gen(seed)
    if kind == "batch_fitness":
        out = []
        for z, k1, k2 in _specs(case, seed):
            n = len(z) - 1
            S = _deff(_genomes(gen, n, case["np"], z, 0), case["np"], n, _integrals(z, k1, k2))
            out.append(S[0] ** 2 + S[1] ** 2)
        return torch.stack(out)
    n, z = case["n"], _boundaries(case, seed)
    if kind == "fitness":
        bits = _genomes(gen, n, case["np"], z, min(32, case["np"] // 4))
        S = _deff(bits, case["np"], n, _integrals(z, inputs.DK1, inputs.DK2))
        return S[0] ** 2 + S[1] ** 2
    if kind == "objective":
        bits, L = _genomes(gen, n, case["np"], z, 0), z[-1] - z[0]
        shg = case["obj"] == "shg"
        G = []
        for k1, k2 in _dks(case):
            S = _deff(bits, case["np"], n, _integrals(z, k1, k2), single=shg)
            G.append(torch.sqrt(S[0] ** 2 + S[1] ** 2) / (L if shg else L * L))
        G = torch.stack(G)
        return -((1.0 - G).abs().sum(0) + (G.max(0).values - G.min(0).values)), G
    # relax: S = sum_{m<n} d_m d_n a_m b_n + sum d^2 c, f = |S|^2 and its gradient
    theta = torch.randn(case["B"], n, generator=gen, device="cuda")
    w = (torch.rand(case["B"], generator=gen, device="cuda") + 0.5).double()
    a, b, c, _ = _integrals(z, inputs.DK1, inputs.DK2)
    fs, gs = [], []
    step = max(1, 4_000_000 // n)
    for i in range(0, case["B"], step):
        d = torch.tanh(theta[i:i + step].double())
        ar, ai, br, bi = d * a[0], d * a[1], d * b[0], d * b[1]
        Pr, Pi = torch.cumsum(ar, 1) - ar, torch.cumsum(ai, 1) - ai
        Sr = (br * Pr - bi * Pi + d * d * c[0]).sum(1, keepdim=True)
        Si = (br * Pi + bi * Pr + d * d * c[1]).sum(1, keepdim=True)
        Rr = br.sum(1, keepdim=True) - torch.cumsum(br, 1)
        Ri = bi.sum(1, keepdim=True) - torch.cumsum(bi, 1)
        dr = b[0] * Pr - b[1] * Pi + a[0] * Rr - a[1] * Ri + 2 * d * c[0]
        di = b[0] * Pi + b[1] * Pr + a[0] * Ri + a[1] * Rr + 2 * d * c[1]
        fs.append((Sr * Sr + Si * Si)[:, 0])
        gs.append(2 * w[i:i + step, None] * (Sr * dr + Si * di) * (1 - d * d))
    return torch.cat(fs), torch.cat(gs)
