"""Timed cases of the library's public entry points on one GPU.

Each case is a dict of plain values; `prepare` makes what a program holds
before the call, `run` is one pass through the public entry points, `work`
the bytes and operations a pass cannot do without and `exact` its outputs in
64-bit torch arithmetic.  Kinds of case:

  techniques  Black-Scholes prices of n options under the exact region, iACT,
              TAF and perforation, each one call of its own
  greeks      prices and their derivatives through torch.autograd
  surrogate   MLP inference with the exact region outside its box
  train       one optimiser step (gradient and Adam) of that network
  hydro       a Sedov blast: initial state, then a number of time steps
  binomial    call and put on a Cox-Ross-Rubinstein tree, one call
"""
import math

import numpy as np
import torch

from paper_2308_16877_amd import greeks, hpac, hydro, surrogate

DEV = "cuda:0"
BIG = 1 << 24

# box of the options: spot, strike, years, rate, volatility
LO = (5.0, 1.0, 0.25, 0.02, 0.1)
HI = (30.0, 100.0, 10.0, 0.02, 0.5)

TECHS = {
    "exact": (hpac.hpac_exact, {}),
    "iact": (hpac.hpac_iact, dict(table_size=8, threshold=0.05)),
    "taf": (hpac.hpac_taf, dict(history_size=4, prediction_size=4, rsd_threshold=0.01)),
    "perfo": (hpac.hpac_perfo, dict(kind="small", param=10)),
}
# items per lane of the four calls: the memo techniques need a sequence of items
TECH_IPT = {"exact": 1, "iact": 16, "taf": 16, "perfo": 20}

BO_TECHS = {
    "exact": (hpac.hpac_bo_exact, 1, {}),
    "iact": (hpac.hpac_bo_iact, 16, dict(table_size=8, threshold=0.05)),
    "taf": (hpac.hpac_bo_taf, 8, dict(history_size=4, prediction_size=4, rsd_threshold=0.01)),
    "perfo": (hpac.hpac_bo_perfo, 10, dict(kind="small", param=10)),
}

HYDRO_TECHS = {
    "exact": {},
    "eos_taf": dict(eos=(2, 2, 0.001, "thread")),
    "hg_perfo": dict(perfo=("small", 10, 1)),
}


def listed():
    return [
        # a portfolio priced for one user's request: 65,536 options from 1,024
        # contracts; a few microseconds of work behind each call
        dict(name="portfolio_64k", kind="techniques", n=65536, data="pool", dtype="f32", body="f32", calls="all"),
        # the whole book, sorted by spot: the four techniques over 2^24 options
        dict(name="sorted_16m", kind="techniques", n=BIG, data="sorted", dtype="f32", body="f32", calls="all"),
        # repeated pricing of the same contracts along each lane, the locality
        # output memoization needs; a ragged item count
        dict(name="taf_periodic_10m", kind="techniques", n=10000019, data="lane", dtype="f32", body="f32",
             calls="taf"),
        # half-precision columns and arithmetic
        dict(name="half_4m", kind="techniques", n=4194319, data="pool", dtype="f16", body="f16", calls="exact"),
        # call Greeks of a medium book, derivatives recomputed in the backward
        dict(name="greeks_exact_3m", kind="greeks", n=3000017, data="pool", technique="exact", upstream="call"),
        # Greeks of call and put positions with memoized derivatives
        dict(name="greeks_iact_16m", kind="greeks", n=BIG, data="wave", technique="iact", upstream="both"),
        # the network as a pricing engine, 5% of the options outside its box
        dict(name="surrogate_16m", kind="surrogate", n=BIG, outside=0.05),
        # the same on one request's worth of options
        dict(name="surrogate_20k", kind="surrogate", n=20011, outside=0.05),
        # one step of its training at the training's batch size
        dict(name="train_8k", kind="train", batch=8192),
        # the blast at the size of the published runs: the first phase of a run
        dict(name="hydro_90", kind="hydro", n=90, steps=48, tech="exact"),
        # a small mesh with output memoization of the equation of state
        dict(name="hydro_24_taf", kind="hydro", n=24, steps=60, tech="eos_taf"),
        # American options on 512-step trees
        dict(name="binomial_512", kind="binomial", n=65536, steps=512, technique="exact", american=True, data="pool"),
    ]


def draw(rng):
    def log_int(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi))))) | rng.randint(0, 1)

    kind = rng.choice(["techniques", "techniques", "greeks", "surrogate", "train", "hydro", "binomial", "binomial"])
    if kind == "techniques":
        calls = rng.choice(["all", "exact", "iact", "taf", "perfo"])
        dtype = rng.choice(["f32", "f32", "f16", "bf16"])
        body = "f16" if dtype == "f16" and rng.random() < 0.5 else "f32"
        return dict(kind=kind, n=log_int(1000, BIG // 2), data=rng.choice(["pool", "sorted", "lane", "wave"]),
                    dtype=dtype, body=body, calls=calls)
    if kind == "greeks":
        return dict(kind=kind, n=log_int(1000, BIG // 2), data=rng.choice(["pool", "wave"]),
                    technique=rng.choice(["exact", "iact"]), upstream=rng.choice(["call", "both"]))
    if kind == "surrogate":
        return dict(kind=kind, n=log_int(500, BIG // 2), outside=rng.choice([0.0, 0.05, 0.2]))
    if kind == "train":
        return dict(kind=kind, batch=log_int(500, 60000))
    if kind == "hydro":
        return dict(kind=kind, n=log_int(8, 80), steps=rng.randint(20, 48), tech=rng.choice(sorted(HYDRO_TECHS)))
    technique = rng.choice(["exact", "exact", "iact", "taf", "perfo"])
    # output memoization on repeating trees decides by computed prices, so that
    # one decision at its threshold moves whole runs of outputs: random order there
    return dict(kind=kind, n=log_int(200, 60000), steps=log_int(30, 500), technique=technique,
                american=rng.random() < 0.75, data="pool" if technique == "taf" else rng.choice(["pool", "unit"]))


# ------------------------------------------------------------------- inputs

def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed) * 7919 + 17)
    return g


def _box(n, g):
    lo, hi = (torch.tensor(v, dtype=torch.float64, device=DEV)[:, None] for v in (LO, HI))
    return lo + (hi - lo) * torch.rand(5, n, generator=g, dtype=torch.float64, device=DEV)


def _options(n, data, seed, period=None):
    """(5, n) FP32 columns: contracts of a pool with a little jitter, in random
    order ("pool"), sorted by spot ("sorted"), or repeating with a period."""
    g = _gen(seed)
    if data in ("pool", "sorted"):
        pool = _box(65536 if data == "sorted" else 1024, g)
        idx = torch.randint(0, pool.shape[1], (n,), generator=g, device=DEV)
    else:
        period = period or {"lane": 1024, "wave": 2}[data]
        pool = _box(period, g)
        idx = torch.arange(n, device=DEV) % period
    x = pool[:, idx].float()
    z = torch.randn(5, n, generator=g, device=DEV)
    z[3] = 0.0  # the rate is one number for all
    x = x * (1.0 + 1e-3 * z)
    if data == "sorted":
        x = x[:, torch.argsort(x[0], stable=True)]
    return x


def _columns(x, dtype=torch.float32):
    return [c.to(dtype).contiguous() for c in x]


def _dtype(case):
    return {"f32": torch.float32, "f16": torch.float16, "bf16": torch.bfloat16}[case.get("dtype", "f32")]


def _calls(case):
    return list(TECHS) if case["calls"] == "all" else [case["calls"]]


def _ipt(case, call):
    # the packed FP16 evaluation takes two items of a lane at a time
    return 2 if call == "exact" and case["body"] == "f16" else TECH_IPT[call]


def _net(seed):
    """Weights of the size training leaves them, biases included."""
    g = np.random.Generator(np.random.PCG64(int(seed) + 4242))
    w = surrogate.init_params(seed=int(seed) + 1)
    for a, b in ((320, 384), (4480, 4544), (4672, 4674)):
        w[a:b] = 0.1 * g.standard_normal(b - a)
    return w.astype(np.float32)


def _norm(logp):
    center = (np.array(LO) + np.array(HI)) / 2
    half = (np.array(HI) - np.array(LO)) / 2
    scale = np.where(half > 0, 1.0 / np.where(half > 0, half, 1.0), 0.0)
    return dict(in_center=center, in_scale=scale, out_mean=logp.mean(1).cpu().numpy(),
                out_scale=logp.std(1).cpu().numpy(), out_shift=np.array([surrogate.PRICE_SHIFT] * 2))


def _surrogate_inputs(case, seed):
    n, g = case["n"], _gen(seed)
    x = _box(n, g)
    out = torch.rand(n, generator=g, device=DEV) < case["outside"]
    which = torch.tensor([0, 1, 2, 4], device=DEV)[torch.randint(0, 4, (n,), generator=g, device=DEV)]
    far = 1.01 + 0.09 * torch.rand(n, generator=g, dtype=torch.float64, device=DEV)
    for j in (0, 1, 2, 4):
        x[j] = torch.where(out & (which == j), HI[j] * far, x[j])
    norm = _norm((_price(_box(65536, _gen(5))) + surrogate.PRICE_SHIFT).log())
    return x.float(), norm


def _train_inputs(case, seed):
    x = _box(case["batch"], _gen(seed)).float()
    t = _price(x.double()).float()
    return x, t, _norm((t.double() + surrogate.PRICE_SHIFT).log())


def _blast_energy(case, seed):
    return hydro.sedov_origin_energy(case["n"]) * (0.8 + 0.4 * np.random.Generator(np.random.PCG64(int(seed))).random())


def prepare(case, seed):
    kind = case["kind"]
    if kind == "techniques":
        x = _columns(_options(case["n"], case["data"], seed), _dtype(case))
        region = hpac.REGION_BS_PRICE_F16 if case["body"] == "f16" else hpac.REGION_BS_PRICE
        outs = {c: [torch.zeros_like(x[0]) for _ in range(2)] for c in _calls(case)}
        return dict(case=case, x=x, outs=outs, region=region)
    if kind == "greeks":
        n = case["n"]
        x = [c.requires_grad_() for c in _columns(_options(n, case["data"], seed))]
        w = [torch.randn(n, generator=_gen(seed + 1), device=DEV) for _ in range(2 if case["upstream"] == "both" else 1)]
        par = dict(table_size=16, threshold=0.05) if case["technique"] == "iact" else None
        return dict(case=case, x=x, w=w, params=par)
    if kind == "surrogate":
        x, norm = _surrogate_inputs(case, seed)
        x = _columns(x)
        return dict(case=case, x=x, net=surrogate.Surrogate(_net(seed), norm, LO, HI, device=DEV),
                    out=[torch.zeros_like(x[0]) for _ in range(2)])
    if kind == "train":
        x, t, norm = _train_inputs(case, seed)
        w = torch.from_numpy(_net(seed)).to(DEV)
        blocks = hpac.hpac_mlp_grad_blocks(case["batch"])
        return dict(case=case, x=_columns(x), t=_columns(t), norm=hpac.make_norm(**norm), w=w, m=torch.zeros_like(w),
                    v=torch.zeros_like(w), step=0, blocks=blocks, loss=torch.empty(blocks, device=DEV),
                    grad=torch.empty(blocks * hpac.MLP_NUM_PARAMS, device=DEV))
    if kind == "hydro":
        e0 = _blast_energy(case, seed)
        return dict(case=case, e0=e0, h=hydro.Hydro(case["n"], e_origin=e0, tech=hydro.Tech(**HYDRO_TECHS[case["tech"]]),
                                                    device=DEV))
    x = _columns(_binomial_options(case, seed))
    return dict(case=case, x=x, out=[torch.zeros_like(x[0]) for _ in range(2)])


def _binomial_options(case, seed):
    period = hpac.hpac_bo_units(case["n"], BO_TECHS[case["technique"]][1])
    return _options(case["n"], case["data"], seed, period=min(period, case["n"]))


# --------------------------------------------------------------------- runs

def run(s):
    case = s["case"]
    kind = case["kind"]
    if kind == "techniques":
        for call, out in s["outs"].items():
            fn, par = TECHS[call]
            fn(s["x"], out, items_per_lane=_ipt(case, call), region=s["region"], **par)
        return s["outs"]
    if kind == "greeks":
        prices = greeks.bs_prices(*s["x"], technique=case["technique"], params=s["params"],
                                  items_per_lane=1 if case["technique"] == "exact" else 16)
        grads = torch.autograd.grad(prices[:len(s["w"])], s["x"], s["w"])
        return dict(prices=[p.detach() for p in prices], grads=grads)
    if kind == "surrogate":
        return s["net"](s["x"], s["out"])
    if kind == "train":
        s["step"] += 1
        hpac.hpac_mlp_grad(s["x"], s["t"], s["w"], s["norm"], case["batch"], s["grad"], s["loss"])
        hpac.hpac_mlp_adam(s["grad"], s["blocks"], s["w"], s["m"], s["v"], 8e-3, 0.9, 0.999, 1e-8, s["step"])
        return dict(w=s["w"], m=s["m"], v=s["v"], loss=s["loss"])
    if kind == "hydro":
        h = s["h"]
        hpac.hpac_hydro_init(h.params, s["e0"], h.state)
        h.steps = 0
        h.run(case["steps"])
        return {f: getattr(h, f) for f in ("x", "u", "e", "p", "q", "c", "vol", "force")}
    fn, ipt, par = BO_TECHS[case["technique"]]
    fn(s["x"], s["out"], case["steps"], american=case["american"], items_per_lane=ipt, **par)
    return s["out"]


# --------------------------------------------------------------------- work

def work(case):
    kind, n = case["kind"], case.get("n", 0)
    if kind == "techniques":
        size = 4 if case["dtype"] == "f32" else 2
        items = {"exact": 1.0, "iact": 1.0, "taf": 1.0, "perfo": 0.9}
        b = sum(7 * size * n * items[c] for c in _calls(case))
        if case["data"] == "lane" and "taf" in _calls(case):
            b -= 5 * size * n * 0.6  # approximated items read no inputs
        return dict(bytes=b, flops=70.0 * n * len(_calls(case)))
    if kind == "greeks":
        # forward 5 columns in and 2 out; backward those 5 and the upstream in, 5 out
        return dict(bytes=4.0 * n * (7 + 10 + (2 if case["upstream"] == "both" else 1)), flops=180.0 * n)
    if kind == "surrogate":
        return dict(bytes=28.0 * n, flops=(2.0 * (5 * 64 + 64 * 64 + 2 * 64) + 128 * 8) * n)
    if kind == "train":
        return dict(bytes=28.0 * case["batch"] + 6 * 4.0 * hpac.MLP_NUM_PARAMS,
                    flops=3 * 2.0 * (5 * 64 + 64 * 64 + 2 * 64) * case["batch"])
    if kind == "hydro":
        # a step reads and writes the node positions and velocities and the
        # element energy, pressure, viscosity and sound speed; the masses are read
        return dict(bytes=case["steps"] * 4.0 * (13 * (n + 1) ** 3 + 9 * n ** 3), flops=case["steps"] * 1200.0 * n ** 3)
    nodes = case["steps"] * (case["steps"] + 1) / 2
    per = 8.0 if case["american"] else 6.0  # two values per node: product, multiply-add and, American, the exercise test
    kept = 0.9 if case["technique"] == "perfo" else 0.25 if case["technique"] == "iact" and case["data"] == "unit" else 1.0
    return dict(bytes=28.0 * n, flops=n * kept * nodes * per)


# ------------------------------------------------------------- 64-bit values

def _price(x):
    """Black-Scholes call and put of (5, n) columns, 64 bits."""
    S, K, T, r, v = x.double()
    vs = v * T.sqrt()
    d1 = ((S / K).log() + (r + 0.5 * v * v) * T) / vs
    d2 = d1 - vs
    D = K * (-r * T).exp()

    def N(d):
        return 0.5 * torch.special.erfc(-d / math.sqrt(2.0))

    return torch.stack([S * N(d1) - D * N(d2), D * N(-d2) - S * N(-d1)])


def _kept(case):
    """Items that small perforation with M = 10 computes."""
    n, ipt = case["n"], TECH_IPT["perfo"]
    L = 64 * (-(-(-(-n // ipt)) // 64))
    return (torch.arange(n, device=DEV) // L) % 10 != 9


def exact(case, seed):
    kind = case["kind"]
    if kind == "techniques":
        x = torch.stack(_columns(_options(case["n"], case["data"], seed), _dtype(case))).double()
        y = _price(x)
        memo = case["data"] not in ("pool", "sorted")  # reused outputs depend on FP32 decisions
        out = {}
        for c in _calls(case):
            if c in ("iact", "taf") and memo:
                out[c] = None
            else:
                out[c] = [torch.where(_kept(case), v, 0.0) if c == "perfo" else v for v in y]
        return out if any(v is not None for v in out.values()) else None
    if kind == "greeks":
        if case["technique"] == "iact" and case["data"] == "wave":
            return None
        s = prepare(case, seed)
        x = torch.stack([c.detach() for c in s["x"]]).double().requires_grad_()
        y = _price(x)
        w = torch.stack([c.double() for c in s["w"]])
        (g,) = torch.autograd.grad((y[:len(w)] * w).sum(), x)
        return dict(prices=list(y.detach()), grads=list(g))
    if kind == "surrogate":
        return _exact_surrogate(case, seed)
    if kind == "train":
        return _exact_train(case, seed)
    if kind == "hydro":
        return _exact_hydro(case, seed) if case["tech"] == "exact" else None
    if case["data"] == "unit" and case["technique"] == "iact":
        return None
    return _exact_binomial(case, seed)


def _unpack(w):
    return [w[a:b].reshape(s) for a, b, s in ((0, 320, (64, 5)), (320, 384, (64,)), (384, 4480, (64, 64)),
                                              (4480, 4544, (64,)), (4544, 4672, (2, 64)), (4672, 4674, (2,)))]


def _forward(w, xh):
    """The network on normalised inputs (5, n); weights rounded to BF16."""
    W1, b1, W2, b2, W3, b3 = (p + (p.detach().bfloat16().double() - p.detach()) if p.dim() == 2 else p
                              for p in _unpack(w))
    gelu = torch.nn.functional.gelu
    h = gelu(W1 @ xh + b1[:, None], approximate="tanh")
    h = gelu(W2 @ h + b2[:, None], approximate="tanh")
    return W3 @ h + b3[:, None]


def _f32(v):
    """The FP32 values the call is given, in 64 bits."""
    return torch.from_numpy(np.asarray(v, np.float64).astype(np.float32)).double().to(DEV)[:, None]


def _exact_surrogate(case, seed):
    x, norm = _surrogate_inputs(case, seed)
    w = torch.from_numpy(_net(seed)).to(DEV).double()
    lo, hi = _f32(LO), _f32(HI)
    outs = []
    for part in x.split(1 << 20, dim=1):
        p = part.double()
        y = _forward(w, (p - _f32(norm["in_center"])) * _f32(norm["in_scale"]))
        y = (y * _f32(norm["out_scale"]) + _f32(norm["out_mean"])).exp() - _f32(norm["out_shift"])
        inside = ((p >= lo) & (p <= hi)).all(0)
        outs.append(torch.where(inside, y, _price(p)))
    return list(torch.cat(outs, 1))


def _exact_train(case, seed):
    x, t, norm = _train_inputs(case, seed)
    n = case["batch"]
    w = torch.from_numpy(_net(seed)).to(DEV).double().requires_grad_()
    y = _forward(w, (x.double() - _f32(norm["in_center"])) * _f32(norm["in_scale"]))
    th = ((t.double() + _f32(norm["out_shift"])).log() - _f32(norm["out_mean"])) / _f32(norm["out_scale"])
    e2 = ((y - th) ** 2).sum(0)
    (g,) = torch.autograd.grad(0.5 * e2.sum() / n, w)
    m, v = 0.1 * g, 0.001 * g * g
    wn = w.detach() - 8e-3 * (m / 0.1) / ((v / 0.001).sqrt() + 1e-8)
    blocks = -(-n // 64)
    loss = torch.nn.functional.pad(e2.detach(), (0, blocks * 64 - n)).reshape(blocks, 64).sum(1)
    return dict(w=wn, m=m, v=v, loss=loss)


def _exact_binomial(case, seed):
    x = torch.stack(_columns(_binomial_options(case, seed))).double()
    n, N, dev = case["n"], case["steps"], DEV
    outs = []
    for part in x.split(16384, dim=1):
        S, K, T, r, v = (c[:, None] for c in part)
        dt = T / N
        u = (v * dt.sqrt()).exp()
        a = (r * dt).exp()
        p = (a - 1 / u) / (u - 1 / u)
        pu, pd = p / a, (1 - p) / a
        lu = u.log()
        i = torch.arange(N + 1, dtype=torch.float64, device=dev)[None]
        X = S * ((2 * i - N) * lu).exp()
        C, P = (X - K).clamp(min=0), (K - X).clamp(min=0)
        for k in range(N - 1, -1, -1):
            C = pu * C[:, 1:] + pd * C[:, :-1]
            P = pu * P[:, 1:] + pd * P[:, :-1]
            if case["american"]:
                X = S * ((2 * i[:, :k + 1] - k) * lu).exp()
                C, P = torch.maximum(C, X - K), torch.maximum(P, K - X)
        outs.append(torch.stack([C[:, 0], P[:, 0]]))
    y = torch.cat(outs, 1)
    if case["technique"] == "perfo":
        L = hpac.hpac_bo_units(n, BO_TECHS["perfo"][1])
        y = torch.where((torch.arange(n, device=dev) // L) % 10 != 9, y, 0.0)
    return list(y)


def _exact_hydro(case, seed):
    n, d64 = case["n"], dict(dtype=torch.float64, device=DEV)
    m, E = n + 1, n ** 3
    gamma, cq, cl, khg, cfl, growth, dvmax = (hydro.DEFAULTS[k] for k in ("gamma", "cq", "cl", "khg", "cfl", "growth",
                                                                          "dvmax"))
    k, j, i = torch.meshgrid(*[torch.arange(n, device=DEV)] * 3, indexing="ij")
    base = (i + m * (j + m * k)).reshape(-1)
    node = [base + (c & 1) + m * (((c >> 1) & 1) + m * (c >> 2)) for c in range(8)]
    sg = torch.tensor([[1.0 if (c >> d) & 1 else -1.0 for d in range(3)] for c in range(8)], **d64)
    G = torch.stack([sg[:, 1] * sg[:, 2], sg[:, 0] * sg[:, 2], sg[:, 0] * sg[:, 1], sg.prod(1)])
    kk, jj, ii = torch.meshgrid(*[torch.arange(m, device=DEV)] * 3, indexing="ij")
    x = torch.stack([ii, jj, kk]).reshape(3, -1).double() * (hydro.DEFAULTS["side"] / n)
    wall = torch.stack([ii, jj, kk]).reshape(3, -1) == 0
    u = torch.zeros_like(x)

    def corners(f):  # (8, 3, E)
        return torch.stack([f[:, v] for v in node])

    def volume(xc):
        """Volume by the 2x2x2 Gauss rule and its gradient."""
        xc = xc.detach().requires_grad_()
        g, V = 1.0 / math.sqrt(3.0), 0.0
        with torch.enable_grad():
            for q in range(8):
                xi = sg[q] * g
                J = []
                for a in range(3):
                    w = sg[:, a] / 8
                    for b in range(3):
                        if b != a:
                            w = w * (1 + sg[:, b] * xi[b])
                    J.append(torch.tensordot(w, xc, dims=1))
                V = V + (J[0] * torch.linalg.cross(J[1], J[2], dim=0)).sum(0)
            (B,) = torch.autograd.grad(V.sum(), xc)
        return V.detach(), B

    V, _ = volume(corners(x))
    mass = V.clone()
    M = torch.zeros(m ** 3, **d64)
    for v in node:
        M.index_add_(0, v, mass / 8)
    e = torch.zeros(E, **d64)
    e[0] = _blast_energy(case, seed)
    p = (gamma - 1) * e
    q = torch.zeros_like(e)
    c = (gamma * p).sqrt()
    dt = hydro.DEFAULTS["dt0"]
    for _ in range(case["steps"]):
        xc, uc = corners(x), corners(u)
        vol, B = volume(xc)
        gx = torch.tensordot(G, xc, dims=1)                              # (4, 3, E)
        gam = G[:, :, None] - (gx[:, None] * B).sum(2) / vol             # (4, 8, E)
        h = (gam[:, :, None] * uc).sum(1)                                # (4, 3, E)
        f = (gam[:, :, None] * h[:, None]).sum(0)                        # (8, 3, E)
        F = (p + q) * B - (khg / 8) * (mass / vol) * c * vol ** (2 / 3) * f
        ceff2 = gamma * (p + q).clamp(min=0) * vol / mass
        vdot = (B * uc).sum((0, 1))
        bound = torch.minimum(cfl * vol ** (1 / 3) / ceff2.sqrt(), dvmax * vol / vdot.abs())
        dt = min(float(bound.min()), growth * dt)
        Fn = torch.zeros_like(x)
        for a in range(8):
            Fn.index_add_(1, node[a], F[a])
        un = torch.where(wall, 0.0, u + dt * Fn / M)
        ub = 0.5 * (u + un)
        x = x + dt * ub
        ubc = corners(ub)
        V1, B1 = volume(corners(x))
        e = e - dt * (F * ubc).sum((0, 1)) / mass
        rho = mass / V1
        du = (B1 * ubc).sum((0, 1)) / V1 ** (2 / 3)
        q = torch.where(du < 0, rho * (cq * du * du + cl * c * du.abs()), 0.0)
        p = (gamma - 1) * rho * e
        c = (gamma * p.clamp(min=0) / rho).sqrt()
        u = un
    return dict(x=x, u=u, e=e, p=p, q=q, c=c, vol=vol, force=F.reshape(24, E))
