"""Timed cases of the Monte Carlo engine: what programs have it do, from one small quote to a
batch of 64 term structures, each through a public entry point of ``paper_1006_3340_amd``.

A case is a dict of plain values.  ``prepare`` makes the inputs a program holds before the call
(term structure, plan, batch, pricer or network), ``run`` is one pass, ``exact`` the same outputs
in 64 bits by plain torch: the 64-node rule of the coupling integral, the driver's increments from
the published Philox-4x32-10, the Euler step and the payoffs, written out here.

An FP32 plan returns its prices in FP64 storage; they are FP32 path arithmetic under FP64 sums
(about 1e-7 of the price), so the cases keep them as the FP32 numbers they are.  FP64 plans' prices
stay FP64.
"""
import math

import numpy as np
import torch

import paper_1006_3340_amd as lll
import workloads
from paper_1006_3340_amd.autograd import CapletPricer

SCHEMES = {"full": lll.FULL, "picard": lll.PICARD, "frozen": lll.FROZEN,
           "first_order": lll.FIRST_ORDER, "second_order": lll.SECOND_ORDER,
           "picard_mp": lll.PICARD_MP, "exact": lll.EXACT}


# ---- the cases -------------------------------------------------------------------------------

def listed():
    return [
        # a single small quote from a resident plan, prices wanted on the host: launches and latency
        {"name": "quote_n5", "kind": "plan", "scheme": "full", "fp64": False, "N": 5, "s": 2,
         "S": 1, "delta": 0.5, "paths": 500, "tails": "light", "swaptions": False, "host": True},
        # the plain method in FP64, one shot from host inputs to host prices: 10 semiannual rates,
        # 10 steps a period, 10^4 paths
        {"name": "oneshot_n10", "kind": "oneshot", "scheme": "full", "fp64": True, "N": 10, "s": 10,
         "S": 1, "delta": 0.5, "paths": 10000, "tails": "light", "swaptions": False, "host": True},
        # the paper's own setting (9 rates, 5 steps a period, NIG tails near the moment limit) with
        # its second-order expansion, an odd path count
        {"name": "second_n9", "kind": "plan", "scheme": "second_order", "fp64": False, "N": 9,
         "s": 5, "S": 5, "delta": 0.5, "paths": 100003, "tails": "heavy", "swaptions": False,
         "host": False},
        # the benchmark's pricing pass: 20 semiannual rates, 400 steps, 2^20 paths
        {"name": "full_n20", "kind": "plan", "scheme": "full", "fp64": False, "N": 20, "s": 20,
         "S": 3, "delta": 0.5, "paths": 1 << 20, "tails": "light", "swaptions": False,
         "host": False},
        # quarterly structure of 40 rates under the Picard drift, swaptions, a ragged path count
        {"name": "picard_n40", "kind": "plan", "scheme": "picard", "fp64": False, "N": 40, "s": 10,
         "S": 3, "delta": 0.25, "paths": (1 << 19) + 77, "tails": "light", "swaptions": True,
         "host": False},
        # end-of-day pricing of many term structures at once: 8 to 40 rates, 7 strikes, 2^18 paths
        {"name": "batch_64", "kind": "batch", "scheme": "full", "count": 64, "paths": 1 << 18},
        # calibration step: prices forward, gradient with respect to forwards and vols backward
        {"name": "autograd_n40", "kind": "autograd", "N": 40, "s": 10, "S": 1, "delta": 0.25,
         "paths": 1 << 18, "tails": "light", "swaptions": False},
        # risk report: the whole Jacobian of 40 caplet prices
        {"name": "greeks_n40", "kind": "greeks", "N": 40, "s": 10, "S": 1, "delta": 0.25,
         "paths": 1 << 17, "tails": "light", "swaptions": False},
        # few paths, many rates: the maturity-parallel layout at 60 rates
        {"name": "picard_mp_n60", "kind": "plan", "scheme": "picard_mp", "fp64": False, "N": 60,
         "s": 10, "S": 3, "delta": 0.25, "paths": 10000, "tails": "light", "swaptions": False,
         "host": False},
        # the exact subset-expansion drift at its largest rate count
        {"name": "exact_n20", "kind": "plan", "scheme": "exact", "fp64": False, "N": 20, "s": 20,
         "S": 3, "delta": 0.5, "paths": 1 << 15, "tails": "light", "swaptions": False,
         "host": False},
        # pricing with the trained drift network
        {"name": "surrogate_n40", "kind": "surrogate", "N": 40, "s": 10, "S": 3, "delta": 0.25,
         "paths": 1 << 16, "tails": "light", "swaptions": False},
        # training the drift network on resident pairs: forward, backward and Adam
        {"name": "train_16k", "kind": "train", "pairs": 1 << 18, "batch": 16384, "steps": 40},
    ]


def draw(rng):
    def logint(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    kind = rng.choice(["plan"] * 8 + ["oneshot"] * 3 + ["batch"] * 2
                      + ["autograd", "greeks", "picard_mp", "exact", "surrogate", "train"])
    delta = rng.choice([0.25, 0.5])
    if kind == "train":
        return {"kind": "train", "pairs": logint(1 << 12, 1 << 19), "batch": logint(1024, 32768),
                "steps": rng.randint(5, 60)}
    if kind == "batch":
        return {"kind": "batch", "scheme": rng.choice(["full", "picard"]),
                "count": rng.randint(2, 64), "paths": logint(1000, 1 << 17)}
    if kind == "surrogate":
        return {"kind": "surrogate", "N": 40, "s": rng.randint(2, 10), "S": rng.randint(1, 5),
                "delta": delta, "paths": logint(1000, 1 << 16), "tails": "light",
                "swaptions": rng.random() < 0.3}
    if kind in ("autograd", "greeks"):
        # gradients take many paths: an indicator that flips on one path weighs 1 / paths
        return {"kind": kind, "N": rng.randint(3, 40), "s": rng.randint(1, 10), "S": 1,
                "delta": delta, "paths": logint(1 << 17, 1 << 18) + rng.randint(0, 99),
                "tails": "light", "swaptions": rng.random() < 0.3}
    if kind == "picard_mp":
        return {"kind": "plan", "scheme": "picard_mp", "fp64": False, "N": rng.randint(2, 64),
                "s": rng.randint(1, 20), "S": rng.randint(1, 5), "delta": delta,
                "paths": logint(100, 30000), "tails": "light", "swaptions": rng.random() < 0.3,
                "host": False}
    if kind == "exact":
        return {"kind": "plan", "scheme": "exact", "fp64": rng.random() < 0.3,
                "N": rng.randint(2, 18), "s": rng.randint(1, 20), "S": rng.randint(1, 5),
                "delta": delta, "paths": logint(1000, 1 << 16), "tails": "light",
                "swaptions": rng.random() < 0.3, "host": False}
    fp64 = rng.random() < 0.3
    heavy = rng.random() < 0.15
    return {"kind": kind, "scheme": rng.choice(["full", "full", "picard", "picard", "frozen",
                                                "first_order", "second_order"]),
            "fp64": fp64, "N": rng.randint(2, 9 if heavy else 24 if fp64 else 40),
            "s": rng.randint(1, 20), "S": rng.randint(1, 8), "delta": delta,
            "paths": logint(100, 1 << (17 if kind == "oneshot" else 18 if fp64 else 20)),
            "tails": "heavy" if heavy else "light", "swaptions": rng.random() < 0.3,
            "host": kind == "oneshot" or rng.random() < 0.3}


# ---- inputs ----------------------------------------------------------------------------------

def structure(case, rng, struct_id=0):
    """Arrays of one term structure: forwards 1-6 %, volatilities 0.12 + 0.1 e^{-(T-t)/2} about
    their level, a NIG driver of light (alpha 12-25) or heavy (1.5, as in the paper) tails, strikes
    0.7-1.3 times the forward (swap) rate."""
    N, s, S, delta = case["N"], case["s"], case["S"], case["delta"]
    heavy = case["tails"] == "heavy"
    tenor = delta * np.arange(1, N + 1, dtype=np.float64)
    dl = np.full(N, delta)
    L0 = rng.uniform(0.01, 0.06, N)
    t = (np.arange(N * s) / s) * delta
    if heavy:
        level = 0.20 - 0.01 * np.arange(N) + rng.uniform(-0.002, 0.002, N)
        vol = np.broadcast_to(level, (N * s, N)).copy()
    else:
        level = rng.uniform(0.115, 0.125, N)
        vol = level + 0.1 * np.exp(-0.5 * (tenor[None, :] - t[:, None]))
    vol[np.arange(N)[None, :] < (np.arange(N * s) // s)[:, None]] = 0.0
    B0_T1 = 1.0 / (1.0 + tenor[0] * L0[0])
    base = L0
    if case["swaptions"]:
        P = B0_T1 / np.concatenate([[1.0], np.cumprod(1.0 + dl * L0)])
        base = (P[:-1] - P[-1]) / np.cumsum((dl * P[1:])[::-1])[::-1]
    mult = np.array([1.0]) if S == 1 else np.linspace(0.7, 1.3, S)
    alpha, beta, dnig = ((1.5, 0.0, 1.5) if heavy else
                         (rng.uniform(12.0, 25.0), rng.uniform(-5.0, 0.0), rng.uniform(0.5, 1.5)))
    return dict(tenor=tenor, delta=dl, L0=L0, B0_T1=B0_T1, steps_per_period=s, vol=vol,
                strikes=base[:, None] * mult[None, :], alpha=float(alpha), beta=float(beta),
                delta_nig=float(dnig), struct_id=struct_id, product=int(case["swaptions"]))


def batch_structures(case, rng):
    out, sizes = [], generator(case["count"])  # the case's sizes; the values come from rng
    for i in range(case["count"]):
        delta = float(sizes.choice([0.25, 0.5]))
        out.append(structure({"N": int(sizes.integers(8, 41)), "s": round(delta / 0.025), "S": 7,
                              "delta": delta, "tails": "light", "swaptions": False}, rng, i))
    return out


def generator(seed):
    return np.random.Generator(np.random.PCG64(seed))


def path_seed(seed):
    return 1 + seed * 2654435761 % (1 << 40)


def training_data(case, seed):
    """Pairs as the network sees them: time, 39 later log-rates, one-hot rate, and smooth labels."""
    g = torch.Generator(device="cuda").manual_seed(seed)
    n = case["pairs"]
    f = torch.zeros(n, 96, device="cuda")
    f[:, 0] = torch.rand(n, generator=g, device="cuda")
    rate = torch.randint(0, 39, (n,), generator=g, device="cuda")
    X = 0.1 * torch.randn(n, 40, generator=g, device="cuda")
    X *= torch.arange(40, device="cuda")[None, :] > rate[:, None]
    f[:, 1:41] = X
    f[torch.arange(n, device="cuda"), 41 + rate] = 1.0
    label = X.square().sum(1) * (1.0 + f[:, 0]) + 0.3 * torch.sin(10.0 * X.sum(1))
    p0 = 0.1 * torch.randn(14593, generator=g, device="cuda")
    return f.to(torch.bfloat16), label, p0.cpu().numpy()


def prepare(case, seed):
    kind, rng = case["kind"], generator(seed)
    st = {"case": case, "seed": path_seed(seed)}
    f64 = dict(dtype=torch.float64, device="cuda")
    if kind == "train":
        feat, label, p0 = training_data(case, seed)
        st.update(feat=feat, label=label, p0=p0, mlp=lll.Mlp(seed=1), sigma=float(label.std()),
                  loss=torch.empty(case["steps"], device="cuda"))
        return st
    if kind == "batch":
        ts = [workloads.TermStructure(**d) for d in batch_structures(case, rng)]
        st["batch"] = lll.Batch(ts, max_paths_each=case["paths"])
        return st
    ts = workloads.TermStructure(**structure(case, rng))
    N, S, P = case["N"], case["S"], case["paths"]
    if kind == "oneshot":
        st["ts"] = ts
    elif kind == "autograd":
        st["pricer"] = CapletPricer(ts, P, seed=st["seed"])
        st["L0"] = torch.tensor(ts.L0, dtype=torch.float32, device="cuda", requires_grad=True)
        st["levels"] = torch.tensor(rng.uniform(-0.002, 0.002, N), dtype=torch.float32,
                                    device="cuda", requires_grad=True)
        st["g"] = torch.tensor(rng.uniform(0.5, 1.5, N), dtype=torch.float32, device="cuda")
    elif kind == "greeks":
        st["plan"] = lll.Plan(ts, precision=lll.FP32, max_paths=P)
        st["out"] = [torch.empty(n, **f64) for n in ((N,), (N, N), (N, N))]
    else:
        st["plan"] = lll.Plan(ts, precision=lll.FP64 if case.get("fp64") else lll.FP32, max_paths=P)
        st["out"] = [torch.empty(N, S, **f64) for _ in range(2)]
        if kind == "surrogate":
            st["mlp"] = lll.Mlp(seed=3)
            st["mlp"].generate(st["plan"], min(P, 12800), 16, seed=5)
            st["mlp"].train(60, 8192, 2e-3, seed=7)
            st["plan"].attach_mlp(st["mlp"])
    return st


# ---- one pass --------------------------------------------------------------------------------

def run(st):
    case, kind = st["case"], st["case"]["kind"]
    stream = torch.cuda.current_stream()
    if kind == "train":
        st["mlp"].set_params(st["p0"])
        st["mlp"].train_dev(st["feat"], st["label"], st["sigma"], case["steps"],
                            batch=case["batch"], lr=2e-3, seed=11, loss=st["loss"], stream=stream)
        return {"loss": st["loss"], "params": st["mlp"].params()}
    if kind == "batch":
        b = st["batch"]
        b.execute(SCHEMES[case["scheme"]], case["paths"], seed=st["seed"], stream=stream)
        r = [b.results(i, stream=stream) for i in range(case["count"])]
        return {k: np.concatenate([x[k].ravel() for x in r]).astype(np.float32)
                for k in ("price", "stderr")}
    if kind == "autograd":
        price = st["pricer"](st["L0"], st["levels"])
        gL, gV = torch.autograd.grad(price, (st["L0"], st["levels"]), st["g"])
        return {"price": price.detach(), "dL0": gL, "dvol": gV}
    if kind == "oneshot":
        r = lll.price_caplets(st["ts"], case["paths"], SCHEMES[case["scheme"]], seed=st["seed"],
                              precision=lll.FP64 if case["fp64"] else lll.FP32, stream=stream)
        return {k: as_held(case, r[k]) for k in ("price", "stderr")}
    plan = st["plan"]
    if kind == "greeks":
        plan.greeks(case["paths"], seed=st["seed"], stream=stream)
        plan.greeks_results_dev(*st["out"], stream=stream)
        return [t.float() for t in st["out"]]
    scheme = lll.MLP_DRIFT if kind == "surrogate" else SCHEMES[case["scheme"]]
    plan.execute(scheme, case["paths"], seed=st["seed"], stream=stream)
    if case.get("host"):
        r = plan.results(stream=stream)
        return {k: as_held(case, r[k]) for k in ("price", "stderr")}
    plan.results_dev(price=st["out"][0], stderr=st["out"][1], stream=stream)
    return {"price": as_held(case, st["out"][0]), "stderr": as_held(case, st["out"][1])}


def as_held(case, v):
    """An FP32 plan's results as FP32 numbers, an FP64 plan's as they are."""
    if case.get("fp64"):
        return v
    return v.float() if isinstance(v, torch.Tensor) else v.astype(np.float32)


# ---- what a pass cannot do without -----------------------------------------------------------

def work(case):
    """Bytes in and out (the term structure, the prices) and the arithmetic of the paths: per step
    an increment (about 40 operations), and per live rate its state, ell and coupling.  The coupling
    integral is counted on 8 nodes, where a Gauss rule of the driver's measure is as good as
    rounding; the reverse pass as twice the forward's work; the exact drift by its subset terms."""
    kind = case["kind"]
    if kind == "train":
        n = case["steps"] * case["batch"]
        return {"bytes": n * (2 * 96 + 4) + 8 * 14593, "flops": n * 6 * (96 * 64 + 2 * 64 * 64 + 64)}
    if kind == "batch":
        b = f = 0
        for d in batch_structures(case, generator(0)):
            w = path_work(len(d["L0"]), d["steps_per_period"], 7, case["paths"], case["scheme"])
            b, f = b + w[0], f + w[1]
        return {"bytes": b, "flops": f}
    N, s, S, P = case["N"], case["s"], case["S"], case["paths"]
    if kind == "surrogate":
        b, f = path_work(N, s, S, P, "first_order")
        return {"bytes": b + 4 * 14593,
                "flops": f + P * s * sum(n * (64 * n + 2 * 64 * 64 * 2 + 128) for n in range(1, N))}
    if kind in ("autograd", "greeks"):
        b, f = path_work(N, s, S, P, "full")
        sweeps = 1 if kind == "autograd" else N / 3.0
        return {"bytes": b, "flops": f * (1 + 2 * sweeps)}
    b, f = path_work(N, s, S, P, case["scheme"])
    return {"bytes": b, "flops": f}


def path_work(N, s, S, P, scheme):
    live = s * N * (N + 1) // 2
    per = {"frozen": 2, "first_order": 8 + N, "exact": 8}.get(scheme, 8 + 6 * 8)
    f = P * (40.0 * N * s + per * live)
    if scheme == "exact":
        f += P * s * 2.0 * 2 ** N * 2
    return 8 * (N * s * N + N * S + 4 * N) + 16 * N * S, f


# ---- the same in 64 bits ---------------------------------------------------------------------

def exact(case, seed):
    kind = case["kind"]
    if kind == "train":
        return exact_training(case, seed)
    if kind in ("autograd", "greeks", "surrogate"):
        return None  # reverse sweeps over 2^17 paths in 64 bits take minutes; the network of the
        #              surrogate is trained by the framework itself
    if kind == "batch":
        ds = batch_structures(case, generator(seed))
        if case["paths"] * sum(rate_steps(d) for d in ds) > 2.5e10:
            return None  # over 20 seconds
        r = [exact_prices(d, case["scheme"], case["paths"], path_seed(seed)) for d in ds]
        return {"price": np.concatenate([p.ravel() for p, _ in r]),
                "stderr": np.concatenate([e.ravel() for _, e in r])}
    d = structure(case, generator(seed))
    if case["paths"] * rate_steps(d) > 2.5e10:
        return None  # over 20 seconds
    price, se = exact_prices(d, case["scheme"], case["paths"], path_seed(seed))
    return {"price": price, "stderr": se}


def rate_steps(d):
    return d["steps_per_period"] * len(d["L0"]) * (len(d["L0"]) + 1) // 2


def philox(c0, c1, c2, c3, k0, k1):
    """Philox-4x32-10 (Salmon et al. 2011) on int64 tensors holding 32-bit words."""
    M = 0xFFFFFFFF
    for _ in range(10):
        p0, p1 = c0 * 0xD2511F53, c2 * 0xCD9E8D57
        c0, c1, c2, c3 = ((p1 >> 32) & M) ^ c1 ^ k0, p1 & M, ((p0 >> 32) & M) ^ c3 ^ k1, p0 & M
        k0, k1 = (k0 + 0x9E3779B9) & M, (k1 + 0xBB67AE85) & M
    return c0, c1, c2


def rule(d):
    """The 64-node rule: 32 Gauss-Legendre points a side mapped by x = +-X v^2, times the NIG Levy
    density, cut where the integrand is below e^-36."""
    N, s, a, b, dn = len(d["L0"]), d["steps_per_period"], d["alpha"], d["beta"], d["delta_nig"]
    lam = max(d["vol"][k, k // s:].sum() for k in range(N * s))
    g, w = np.polynomial.legendre.leggauss(32)
    v, w = 0.5 * (g + 1.0), 0.5 * w
    X = min(36.0 / (a - b - lam), 40.0), min(36.0 / (a + b), 40.0)
    x = np.concatenate([X[0] * v * v, -X[1] * v * v])
    jac = np.concatenate([2 * X[0] * v * w, 2 * X[1] * v * w])
    z = torch.tensor(a * np.abs(x))
    k1e = torch.special.scaled_modified_bessel_k1(z).numpy()
    return x, jac * dn * a / math.pi * np.exp(b * x - a * np.abs(x)) * k1e / np.abs(x)


def kappa(u, d):
    """NIG cumulant of the martingale driver, without cancellation."""
    a, b, dn = d["alpha"], d["beta"], d["delta_nig"]
    g = math.sqrt(a * a - b * b)
    s = np.sqrt(a * a - (b + u) ** 2)
    return dn * u * u * (g + b * (2 * b + u) / (g + s)) / (g * (g + s))


def coupling(scheme, ell, lam, d, E, WE):
    """C_i = sum_q W E_i (prod_{l>i} (1 + ell_l E_l) - 1) over the live rates, or its expansions."""
    P, n = ell.shape
    C = torch.zeros_like(ell)
    if scheme == "first_order":
        k2 = kappa(lam[:, None] + lam[None, :], d) - kappa(lam, d)[:, None] - kappa(lam, d)[None, :]
        return ell @ torch.tensor(np.triu(k2, 1).T.copy(), device=ell.device)
    R = torch.zeros(P, 64, dtype=torch.float64, device=ell.device)
    u = torch.ones_like(R) if scheme == "second_order" else None
    for j in range(n - 1, -1, -1):
        if j < n - 1:
            C[:, j] = R @ WE[j]
        if j:
            t = ell[:, j, None] * E[j]
            if u is None:
                R.addcmul_(R, t).add_(t)
            else:
                R.addcmul_(t, u)
                u.add_(t)
    return C


def exact_prices(d, scheme, n_paths, seed):
    N, s = len(d["L0"]), d["steps_per_period"]
    S = d["strikes"].shape[1]
    dev = lambda v: torch.tensor(v, dtype=torch.float64, device="cuda")  # noqa: E731
    x, W = rule(d)
    L0, dl, strikes = dev(d["L0"]), dev(d["delta"]), dev(d["strikes"])
    kap = kappa(d["vol"], d)
    ell0 = dl * L0 / (1 + dl * L0)
    gamma = math.sqrt(d["alpha"] ** 2 - d["beta"] ** 2)
    lams, Es, b0s = [], [], []
    for k in range(N * s):
        m = k // s
        lam = d["vol"][k, m:]
        E = np.expm1(lam[:, None] * x[None, :])
        Es.append((dev(E), dev(E * W)))
        lams.append(dev(lam))
        b0s.append(-dev(kap[k, m:]) - coupling("full", ell0[None, m:], lam, d, *Es[-1])[0])
    sums = torch.zeros(2, N, S, dtype=torch.float64, device="cuda")
    for p0 in range(0, n_paths, 1 << 16):
        p = torch.arange(p0, min(n_paths, p0 + (1 << 16)), device="cuda")
        X = torch.zeros(len(p), N, dtype=torch.float64, device="cuda")
        X1 = torch.zeros_like(X)
        for k in range(N * s):
            m = k // s
            dt = (d["tenor"][m] - (d["tenor"][m - 1] if m else 0.0)) / s
            w = philox(torch.full_like(p, k), p & 0xFFFFFFFF, p >> 32,
                       torch.full_like(p, d["struct_id"]), seed & 0xFFFFFFFF, seed >> 32)
            u0, u1, u2 = ((v >> 8).double().add(0.5) / (1 << 24) for v in w)
            r = torch.sqrt(-2 * torch.log(u0))
            z1, z2 = r * torch.cos(2 * math.pi * u1), r * torch.sin(2 * math.pi * u1)
            mean, shape = d["delta_nig"] * dt / gamma, (d["delta_nig"] * dt) ** 2
            a = mean * z1 * z1
            y = 4 * mean * shape * a / (a + torch.sqrt(a * a + 4 * shape * a)) ** 2
            y = torch.where(a > 0, y, torch.full_like(y, mean))
            V = torch.where(u2 <= mean / (mean + y), y, mean * mean / y)
            dH = (-d["delta_nig"] * d["beta"] / gamma * dt + d["beta"] * V + torch.sqrt(V) * z2)
            move = lams[k] * dH[:, None]
            if scheme == "frozen":
                X[:, m:] += b0s[k] * dt + move
            else:
                Y = X1 if scheme in ("picard", "picard_mp") else X
                L = L0[m:] * torch.exp(Y[:, m:])
                ell = dl[m:] * L / (1 + dl[m:] * L)
                C = coupling(scheme, ell, d["vol"][k, m:], d, *Es[k])
                X[:, m:] += (-dev(kap[k, m:]) - C) * dt + move
                if Y is X1:
                    X1[:, m:] += b0s[k] * dt + move
            if (k + 1) % s == 0:
                L = L0[m:] * torch.exp(X[:, m:])
                b = 1 + dl[m:] * L
                Q = torch.flip(torch.cumprod(torch.flip(b, [1]), 1), [1])   # prod_{j>=l}
                above = torch.cat([Q[:, 1:], torch.ones_like(Q[:, :1])], 1)  # prod_{j>l}
                if d["product"]:
                    pay = (Q[:, :1] - 1) - strikes[m] * (dl[m:] * above).sum(1, keepdim=True)
                else:
                    pay = above[:, :1] * (L[:, :1] - strikes[m])
                pay = pay.clamp_min(0.0)
                sums[0, m] += pay.sum(0)
                sums[1, m] += pay.square().sum(0)
    B0T = d["B0_T1"] / float(np.prod(1 + d["delta"] * d["L0"]))
    scale = torch.full((N, 1), B0T, dtype=torch.float64, device="cuda")
    if not d["product"]:
        scale = scale * dl[:, None]
    mean = sums[0] / n_paths
    var = (sums[1] / n_paths - mean * mean).clamp_min(0.0)
    return ((scale * mean).cpu().numpy(),
            (scale * torch.sqrt(var / max(n_paths - 1, 1))).cpu().numpy())


def exact_training(case, seed):
    """The training loop with plain 64-bit matrix products (96-64-64-64-1, tanh-form GELU)."""
    feat, label, p0 = training_data(case, seed)
    p = torch.tensor(p0, dtype=torch.float64, device="cuda", requires_grad=True)
    y = label.double() / float(np.float32(float(label.std())))
    cut = np.cumsum([0, 6144, 64, 4096, 64, 4096, 64, 64, 1])
    m, v = torch.zeros_like(p), torch.zeros_like(p)
    i = torch.arange(case["batch"], device="cuda")
    losses = []
    for t in range(1, case["steps"] + 1):
        w = philox(torch.full_like(i, t), i, torch.ones_like(i), torch.full_like(i, 2 << 24), 11, 0)
        idx = ((w[0] % case["pairs"]) * ((1 << 32) % case["pairs"]) + w[1]) % case["pairs"]
        q = [p[cut[j]:cut[j + 1]] for j in range(8)]
        h = feat[idx].double()
        for W, b, n in ((q[0], q[1], 96), (q[2], q[3], 64), (q[4], q[5], 64)):
            h = torch.nn.functional.gelu(h @ W.view(64, n).T + b, approximate="tanh")
        loss = (h @ q[6] + q[7] - y[idx]).square().sum() / (2 * case["batch"])
        (g,) = torch.autograd.grad(loss, p)
        losses.append(loss.detach())
        m, v = 0.9 * m + 0.1 * g, 0.999 * v + 0.001 * g * g
        lr = 2e-3 * (0.01 + 0.99 * 0.5 * (1 + math.cos(math.pi * (t - 1) / case["steps"])))
        with torch.no_grad():
            p -= lr * (m / (1 - 0.9 ** t)) / (torch.sqrt(v / (1 - 0.999 ** t)) + 1e-8)
    return {"loss": torch.stack(losses), "params": p.detach()}
