"""What the framework's speed is judged by: calls of its public entry points over the sizes a
user has, from one instance to full batches.

  sfft    SfftPricer.run: QTT build, zip-up, rounding and read-out of a batch of grids
  dense   cm_fft_price: the dense Carr-Madan transform, all 2^n strikes or a chosen set of them
  shots   SfftPricer.measure: the QFT-observable arm with emulated measurement
  query   Surrogate.predict: the pricing network and its gate
  train   MlpNet.train_step: one Adam step of the network

`exact` holds the same results from plain torch in 64 bits.
"""
import math

import numpy as np
import torch

import paper_2607_28435_amd as cm

DEV = "cuda"
C128 = torch.complex128

# The batched Heston box (kappa, theta, sigma_v, rho, v0, T) and the surrogate's log-moneyness.
BOX_LO = np.array([0.5, 0.01, 0.1, -0.9, 0.01, 0.1, -0.5])
BOX_HI = np.array([4.0, 0.1, 0.8, -0.1, 0.1, 2.0, 0.5])


def listed():
    return [
        # The headline workload: one batch of calibrated Heston surfaces priced overnight or on a
        # tick, 4096 near-money strikes each, with the launch widths the benchmark uses.
        dict(name="sfft heston batch", kind="sfft", model="heston", dtype="c64", batch=4096, n_lo=24, n_hi=24,
             strikes=4096, tol=1e-8, cap=32, grid="rule", slots="4096,1536,4096"),
        # A mixed book: grids of several resolutions in one batch, an odd number of them, library
        # default launch widths.
        dict(name="sfft heston ragged", kind="sfft", model="heston", dtype="c64", batch=777, n_lo=16, n_hi=28,
             strikes=1000, tol=1e-8, cap=32, grid="rule", slots=""),
        # Full-precision pricing of another model (slowly decaying transform) on a medium batch.
        dict(name="sfft vg fp64", kind="sfft", model="vg", dtype="c128", batch=256, n_lo=20, n_hi=20, strikes=513,
             tol=1e-10, cap=32, grid="rule", slots=""),
        # One grid at a time, as in the paper's run-time curves: pure latency.
        dict(name="sfft bs single", kind="sfft", model="bs", dtype="c128", batch=1, n_lo=30, n_hi=30, strikes=4096,
             tol=1e-10, cap=64, grid="paper", slots=""),
        # The dense transform the paper compares with, at the headline size, prices wanted in the
        # moneyness window (elsewhere the undamping amplifies rounding).
        dict(name="dense heston n24", kind="dense", model="heston", dtype="c64", batch=8, n=24, strikes=4096,
             grid="rule"),
        # The FP64 dense curve on the paper's symmetric grid.
        dict(name="dense bs fp64 n20", kind="dense", model="bs", dtype="c128", batch=16, n=20, strikes=4096,
             grid="paper"),
        # Many small grids: below the crossover the dense transform is the faster path.
        dict(name="dense merton n13", kind="dense", model="merton", dtype="c64", batch=1000, n=13, strikes=501,
             grid="rule"),
        # Every strike of one very large grid (a coarse frequency step keeps all of them meaningful).
        dict(name="dense heston n26 all", kind="dense", model="heston", dtype="c64", batch=1, n=26, strikes=0,
             grid="coarse"),
        # Emulated hardware runs: the paper's default of 4096 shots for a batch of instances.
        dict(name="shots heston", kind="shots", model="heston", dtype="c64", batch=512, n_lo=24, n_hi=24,
             strikes=4096, shots=4096, tol=1e-8, cap=32, grid="rule", slots=""),
        # The surrogate serving a large block of queries, and one request's worth of them.
        dict(name="query 1m", kind="query", rows=1 << 20),
        dict(name="query 777", kind="query", rows=777),
        # One training step at the recipe's minibatch.
        dict(name="train 8192", kind="train", rows=8192),
    ]


def _logint(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["sfft", "sfft", "sfft", "dense", "dense", "shots", "query", "train"])
    if kind == "sfft":
        dtype = rng.choice(["c64", "c64", "c128"])
        model = rng.choice(["heston", "heston", "merton", "bs", "vg"])
        n_lo = rng.randint(12, 20 if model == "vg" else 28)
        n_hi = min(n_lo + rng.choice([0, 0, 3, 7]), 20 if model == "vg" else 28)
        return dict(kind=kind, model=model, dtype=dtype, batch=_logint(rng, 1, 2048), n_lo=n_lo, n_hi=n_hi,
                    strikes=_logint(rng, 16, 4096), tol=1e-8 if dtype == "c64" else 1e-10,
                    cap=rng.choice([32, 32, 64]), grid="rule", slots="")
    if kind == "dense":
        n = rng.randint(9, 26)
        most = 1 << (26 - n)
        return dict(kind=kind, model=rng.choice(["heston", "merton", "bs", "vg"] if n <= 20 else ["heston", "bs"]),
                    dtype=rng.choice(["c64", "c64", "c128"] if n < 26 else ["c64"]), n=n,
                    batch=_logint(rng, 1, min(most, 4096)), grid="coarse" if (every := rng.random() < 0.4) else "rule",
                    strikes=0 if every else _logint(rng, 16, 4096))
    if kind == "shots":
        return dict(kind=kind, model=rng.choice(["heston", "bs"]), dtype=rng.choice(["c64", "c128"]),
                    batch=_logint(rng, 1, 256), n_lo=(n := rng.randint(10, 24)), n_hi=n,
                    strikes=_logint(rng, 64, 512), shots=_logint(rng, 100, 4096), tol=1e-8, cap=32, grid="rule",
                    slots="")
    if kind == "query":
        return dict(kind=kind, rows=_logint(rng, 1, 1 << 20))
    return dict(kind=kind, rows=_logint(rng, 256, 16384))


# ------------------------------------------------------------------ inputs

def _eta(n, grid):
    # rule: 40 / 2^(n/2), the batched grids; coarse: log-strikes within pi of the spot;
    # paper: the experiments' grid (N = 2^(n-1), log-strike step N^(-1/2))
    if grid == "rule":
        return 40.0 / 2.0 ** (n / 2.0)
    if grid == "coarse":
        return 1.0
    N = 2 ** (n - 1)
    return math.pi / (N * N ** -0.5)


def _problems(case, seed):
    """The batch's problems as numpy arrays: n, T, model parameters, grid."""
    g = np.random.Generator(np.random.Philox(seed))
    count, model = case["batch"], case["model"]
    n = g.integers(case["n_lo"], case["n_hi"] + 1, count) if "n_lo" in case else np.full(count, case["n"])
    r, q, alpha = 0.03, 0.0, 1.5
    if model == "heston":
        p = BOX_LO[:6] + (BOX_HI[:6] - BOX_LO[:6]) * g.random((count, 6))
        T, p = p[:, 5].copy(), p[:, :5].copy()
    elif model == "bs":
        T, p = g.uniform(0.25, 2.0, count), g.uniform(0.1, 0.5, (count, 1))
        if case["grid"] == "paper":
            T, p, r, alpha = g.uniform(0.4, 0.6, count), g.uniform(0.25, 0.35, (count, 1)), 0.05, 2.5
    elif model == "merton":
        T = g.uniform(0.5, 2.0, count)
        p = np.stack([g.uniform(0.1, 0.3, count), g.uniform(0.1, 1.0, count), g.uniform(-0.2, 0.1, count),
                      g.uniform(0.1, 0.3, count)], axis=1)
    else:   # Variance Gamma with a finite damping moment and a clock no shorter than its variance rate
        rows = []
        while len(rows) < count:
            sig, nu, th, t = g.uniform(0.08, 0.3), g.uniform(0.05, 0.5), g.uniform(-0.3, 0.05), g.uniform(0.1, 1.5)
            if 1.0 - 2.5 * th * nu - 0.5 * sig * sig * nu * 6.25 > 0.05 and t >= nu:
                rows.append((sig, nu, th, t))
        a = np.array(rows)
        T, p = a[:, 3].copy(), a[:, :3].copy()
    paper = case["grid"] == "paper"
    eta = np.array([_eta(int(v), case["grid"]) for v in n])
    k0 = None
    if paper:
        k0 = np.array([math.log(100.0) - 2.0 ** ((int(v) - 1) / 2.0) / 2.0 for v in n])
    return dict(model=model, quad="rect2" if paper else "simpson1", n=n, S0=100.0, r=r, q=q, T=T, alpha=alpha, eta=eta,
                p=p, k0=k0)


def _arrays(P):
    return cm.ProblemArrays(P["model"], P["quad"], P["n"], P["S0"], P["r"], P["q"], P["T"], P["alpha"], P["eta"],
                            P["p"], k0=P["k0"])


def _strikes(case, P):
    """[batch, strikes] increasing log-strike indices with one stride per row: consecutive ones about
    the money where that is what the batch wants, else spread over 0.5 <= K/S0 <= 1.5."""
    count, nk = len(P["T"]), case["strikes"]
    out = np.empty((count, nk), dtype=np.int64)
    start, step = np.empty(count, dtype=np.int64), np.empty(count, dtype=np.int64)
    for i in range(count):
        n, eta = int(P["n"][i]), float(P["eta"][i])
        M = 1 << n
        lam = 2.0 * math.pi / (M * eta)
        mid = M // 2 if P["k0"] is None else int(round((math.log(P["S0"]) - float(P["k0"][i])) / lam))
        if case["kind"] in ("sfft", "shots") and P["k0"] is None:
            g = max(1, min(1, M // nk))
        else:
            g = max(1, int((math.log(1.5) - math.log(0.5)) / lam) // nk)
        first = mid - g * (nk // 2)
        first = max(0, min(first, M - 1 - g * (nk - 1)))
        start[i], step[i] = first, g
        out[i] = first + g * np.arange(nk, dtype=np.int64)
    return out, start, step


def _sizes(case):
    """Cases smaller than the strikes they ask for get as many as fit."""
    n = case.get("n_lo", case.get("n"))
    return dict(case, strikes=min(case["strikes"], 1 << n)) if "strikes" in case else case


def _net(seed):
    """A network and its serving gate: the surrogate's own initial weights with the output centred
    on a mid-range price, and a calibrated error table."""
    s = cm.Surrogate(BOX_LO, BOX_HI, seed=seed, device=DEV)
    s.net.params[-1] = math.log(0.51)
    g = np.random.Generator(np.random.Philox(seed + 77))
    s.cell_err = torch.from_numpy(g.uniform(0.0, 6e-4, (16, 16)).astype(np.float32)).to(DEV)
    s.err_tol = 5e-4
    return s


def _queries(rows, seed):
    """Nine queries of ten in the trusted box, the others in the box widened by a fifth."""
    g = np.random.Generator(np.random.Philox(seed + 5001))
    u = g.random((rows, 7))
    w = (BOX_HI - BOX_LO) * np.where(g.random((rows, 1)) < 0.9, 0.0, 0.1)
    lo, hi = np.maximum(BOX_LO - w, [0.05, 0.001, 0.02, -0.98, 0.001, 0.02, -9.0]), BOX_HI + w
    return (lo + (hi - lo) * u).astype(np.float32)


def prepare(case, seed):
    case = _sizes(case)
    kind = case["kind"]
    if kind in ("sfft", "shots"):
        P = _problems(case, seed)
        dtype = cm.CM_C64 if case["dtype"] == "c64" else cm.CM_C128
        slots = dict(zip(("build", "apply", "round"), map(int, case["slots"].split(",")))) if case["slots"] else None
        # the operator table a pricing program keeps for the resolutions it serves
        mpo = cm.MpoCache(P["n"], case["tol"] / 10, case["cap"], dtype, DEV)
        pr = cm.SfftPricer(_arrays(P), dtype, tol=case["tol"], cap=case["cap"], mpo=mpo, device=DEV, slots=slots)
        state = dict(kind=kind, pr=pr, strikes=torch.from_numpy(_strikes(case, P)[0]).to(DEV))
        if kind == "shots":
            gen = torch.Generator(device=DEV)
            gen.manual_seed(seed)
            state["uniforms"] = torch.rand((case["batch"], int(P["n"].max()), case["shots"]), dtype=torch.float64,
                                           device=DEV, generator=gen)
        return state
    if kind == "dense":
        P = _problems(case, seed)
        c64 = case["dtype"] == "c64"
        M = 1 << case["n"]
        idx = torch.from_numpy(_strikes(case, P)[0]).to(DEV) if case["strikes"] else None
        return dict(kind=kind, prob=_arrays(P).pack(DEV), batch=case["batch"], n=case["n"],
                    dtype=cm.CM_C64 if c64 else cm.CM_C128, idx=idx, nk=case["strikes"],
                    prices=torch.empty((case["batch"], case["strikes"] or M),
                                       dtype=torch.float32 if c64 else torch.float64, device=DEV),
                    status=torch.zeros(case["batch"], dtype=torch.int32, device=DEV), ws=cm.Workspace(DEV))
    if kind == "query":
        s = _net(seed)
        return dict(kind=kind, s=s, q=torch.from_numpy(_queries(case["rows"], seed)).to(DEV))
    # a network in mid-training: Adam's moments at the size of the gradients they average
    net = _net(seed).net
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    net.m.copy_(1e-4 * torch.randn(net.m.shape, device=DEV, generator=g))
    net.v.copy_((1e-4 * (0.5 + torch.rand(net.v.shape, device=DEV, generator=g))) ** 2)
    net.t = 1000
    x, t = _training_rows(case["rows"], seed)
    return dict(kind=kind, net=net, x=x, t=t, loss=torch.zeros(1, dtype=torch.float32, device=DEV))


def _training_rows(rows, seed):
    q = _queries(rows, seed)
    # targets of the size of encoded call prices: log of the intrinsic value plus a time value
    k, T = q[:, 6].astype(np.float64), q[:, 5].astype(np.float64)
    c = np.maximum(0.0, 1.0 - np.exp(k - 0.03 * T)) + 0.08 * np.sqrt(T) * np.exp(-8.0 * k * k)
    return torch.from_numpy(q).to(DEV), torch.from_numpy(np.log(c + 0.01).astype(np.float32)).to(DEV)


def run(state):
    kind = state["kind"]
    if kind == "sfft":
        return state["pr"].run(state["strikes"])
    if kind == "shots":
        return state["pr"].measure(state["strikes"], state["uniforms"])
    if kind == "dense":
        cm.cm_fft_price(state["prob"], state["batch"], state["n"], state["dtype"], state["idx"], state["nk"],
                        state["prices"], state["status"], state["ws"])
        return dict(prices=state["prices"], status=state["status"])
    if kind == "query":
        return state["s"].predict(state["q"])
    net = state["net"]
    net.train_step(state["x"], state["t"], 1e-3, state["loss"])
    return dict(grad=net.grad, params=net.params, m=net.m, v=net.v)


def work(case):
    case = _sizes(case)
    kind = case["kind"]
    if kind in ("sfft", "shots"):
        # flops of one site (measured ranks at these tolerances): build 125 K, zip-up 470 K,
        # rounding 43 K; a read-out strike finishes from shared prefixes
        sites = case["batch"] * (case["n_lo"] + case["n_hi"]) / 2.0
        w = dict(bytes=case["batch"] * (128 + 16.0 * case["strikes"]),
                 flops=sites * 638e3 + 100.0 * case["batch"] * case["strikes"])
        if kind == "shots":   # 800 flops a shot and level; uniforms in, outcomes out
            w["bytes"] += case["batch"] * case["shots"] * (8.0 * case["n_hi"] + 8)
            w["flops"] += 800.0 * sites * case["shots"]
        return w
    if kind == "dense":
        M, es = 1 << case["n"], 4 if case["dtype"] == "c64" else 8
        out = case["strikes"] or M
        return dict(bytes=case["batch"] * (128 + out * (es + (8 if case["strikes"] else 0))),
                    flops=2.5 * case["batch"] * M * case["n"])
    mul = 2.0 * (7 * 256 + 3 * 65536 + 256)
    if kind == "query":
        return dict(bytes=case["rows"] * 36.0 + 4 * 199681, flops=case["rows"] * mul)
    return dict(bytes=case["rows"] * 32.0 + 28.0 * 199681, flops=3 * case["rows"] * mul)


# ------------------------------------------------------------------ the same results in 64 bits

def _h(P, rows, v):
    """psi(v) exp(-i v m_f) of the rows' problems: the damped transform without the forward's phase."""
    col = lambda a: torch.as_tensor(np.broadcast_to(np.asarray(a, dtype=np.float64), len(P["T"]))[rows].copy(),
                                    device=DEV)[:, None]
    T, al, r, q = col(P["T"]), P["alpha"], P["r"], P["q"]
    p = [col(P["p"][:, i]) for i in range(P["p"].shape[1])]
    v = v[None, :] if v.dim() == 1 else v
    u = torch.complex(v, torch.full_like(v, -(al + 1.0)))
    iu, u2 = 1j * u, u * u
    if P["model"] == "bs":
        L = -0.5 * p[0] * p[0] * T * (u2 + iu)
    elif P["model"] == "merton":
        kj = torch.exp(p[2] + 0.5 * p[3] * p[3]) - 1.0
        L = -0.5 * p[0] * p[0] * T * (u2 + iu) - p[1] * kj * T * iu
        L = L + p[1] * T * (torch.exp(iu * p[2] - 0.5 * p[3] * p[3] * u2) - 1.0)
    elif P["model"] == "vg":
        om = torch.log(1.0 - p[2] * p[1] - 0.5 * p[0] * p[0] * p[1]) / p[1]
        L = om * T * iu - T / p[1] * torch.log(1.0 - p[2] * p[1] * iu + 0.5 * p[0] * p[0] * p[1] * u2)
    else:
        ka, th, sv, rho, v0 = p
        b = ka - rho * sv * iu
        d = torch.sqrt(b * b + sv * sv * (iu + u2))
        g = (b - d) / (b + d)
        e = torch.exp(-T * d)
        L = ka * th / (sv * sv) * (T * (b - d) - 2.0 * torch.log((1.0 - g * e) / (1.0 - g)))
        L = L + v0 / (sv * sv) * (b - d) * (1.0 - e) / (1.0 - g * e)
    mf = math.log(P["S0"]) + (r - q) * T
    return torch.exp(L + (-r * T + (al + 1.0) * mf)) / (torch.complex(torch.full_like(v, al), v) *
                                                       torch.complex(torch.full_like(v, al + 1.0), v))


def _turn(m, frac):
    """exp(2 pi i m frac), m whole numbers below 2^30 in size, frac a long double in [0, 1)."""
    a = np.floor(frac * 2 ** 22) / 2 ** 22
    b = float(frac - a)
    f = m * float(a)
    f = (f - torch.floor(f)) + m * b
    return torch.exp(2j * math.pi * f)


def _terms(P, i, m):
    """w_m h(v_m) exp(i v_m (m_f - k0)) for the frequencies m eta of problem i."""
    eta, n = float(P["eta"][i]), int(P["n"][i])
    ld = np.longdouble
    x = _h(P, [i], m.double() * eta)[0]
    rq = ld(P["r"] - P["q"]) * ld(P["T"][i])
    two_pi = 2 * ld("3.14159265358979323846264338")
    if P["k0"] is None:   # k0 = ln S0 - pi / eta
        th = ld(eta) * rq / two_pi + ld(0.5)
    else:
        th = ld(eta) * (np.log(ld(P["S0"])) - ld(P["k0"][i]) + rq) / two_pi
    x = x * _turn(m.double(), th - np.floor(th))
    if P["quad"] == "simpson1":
        w = torch.where(m % 2 == 1, 4.0, 2.0)
        return x * torch.where(m == 0, 1.0, w) * (eta / 3.0)
    return x * eta


def _logk(P, i, u):
    """Log-strikes of the whole-number indices u (numpy)."""
    ld = np.longdouble
    n, eta = int(P["n"][i]), ld(P["eta"][i])
    lam = 2 * ld("3.14159265358979323846264338") / (ld(2) ** n * eta)
    if P["k0"] is None:
        return (np.log(ld(P["S0"])) + lam * (u - (1 << (n - 1))).astype(ld)).astype(np.float64)
    return (ld(P["k0"][i]) + lam * u.astype(ld)).astype(np.float64)


def _support(P, i):
    """Frequencies beyond which |h| stays under 1e-19 of |h(0)|, or the whole grid."""
    n, eta = int(P["n"][i]), float(P["eta"][i])
    most = (1 << n) if P["quad"] == "simpson1" else (1 << (n - 1))
    v = torch.exp2(torch.arange(0, 28 * 8, device=DEV) / 8.0 - 4.0)
    h = _h(P, [i], torch.cat([v * 0, v]))[0].abs()
    over = torch.nonzero(~(h[len(v):] < 1e-19 * h[0]))
    last = int(over[-1]) + 2 if len(over) else 0
    return most if last >= len(v) else min(most, int(float(v[last]) / eta) + 2)


def _frequencies(P, i):
    E = _support(P, i)
    return torch.arange(0 if P["quad"] == "simpson1" else -E, E, device=DEV)


def _scale(P, i, u):
    s = 1.0 if P["quad"] == "simpson1" else 2.0
    return torch.from_numpy(np.exp(-P["alpha"] * _logk(P, i, u)) / (s * math.pi)).to(DEV)


def _window_prices(P, i, start, step, nk):
    """Prices at start + step s, s < nk: the sum over the support by Bluestein's identity
    m s = (m^2 + s^2 - (s - m)^2) / 2, every phase a whole multiple of step / 2^(n+1) turns."""
    m = _frequencies(P, i)
    n, lo, E = int(P["n"][i]), int(m[0]), m.numel()
    M2 = 1 << (n + 1)
    ph = lambda e: torch.exp(2j * math.pi * ((e * step) % M2).double() / M2)
    j = torch.arange(E, device=DEV)
    # exp(-2 pi i m start / M), start reduced exactly
    a = _terms(P, i, m) * torch.exp(-2j * math.pi * (((m % (M2 >> 1)) * start) % (M2 >> 1)).double() / (M2 >> 1))
    N = 1 << (E + nk - 1).bit_length()
    s = torch.arange(nk, device=DEV)
    c = torch.zeros(N, dtype=C128, device=DEV)
    c[:nk] = ph(s * s)
    c[N - E + 1:] = ph((j * j)[1:]).flip(0)
    f = torch.zeros(N, dtype=C128, device=DEV)
    f[:E] = a * ph(-(j * j))
    y = torch.fft.ifft(torch.fft.fft(f) * torch.fft.fft(c))[:nk] * ph(-(s * s))
    y = y * torch.exp(-2j * math.pi * ((lo * step * s) % (M2 >> 1)).double() / (M2 >> 1))
    return _scale(P, i, start + step * np.arange(nk, dtype=np.int64)) * y.real


def _all_prices(P, i):
    n = int(P["n"][i])
    M = 1 << n
    m = _frequencies(P, i)
    x = torch.zeros(M, dtype=C128, device=DEV)
    x[m % M] = _terms(P, i, m)
    y = torch.fft.fft(x).real
    del x
    out = torch.empty(M, dtype=torch.float64, device=DEV)
    for a in range(0, M, 1 << 22):
        u = np.arange(a, min(M, a + (1 << 22)), dtype=np.int64)
        out[a:a + len(u)] = _scale(P, i, u) * y[a:a + len(u)]
    return out


def _net64(net):
    """The network's parameters in 64 bits, hidden weights as their BF16 copies hold them."""
    p = net.params.double()
    W, b, o = [], [], 0
    for out, inp in ((256, 7), (256, 256), (256, 256), (256, 256), (1, 256)):
        w = net.params[o:o + out * inp].reshape(out, inp)
        W.append((w.bfloat16() if inp == 256 and out == 256 else w).double())
        o += out * inp
        b.append(p[o:o + out])
        o += out
    return W, b


def _forward64(W, b, x):
    scale = (2.0 / (_TRAIN_HI - _TRAIN_LO)).astype(np.float32)
    shift = ((_TRAIN_LO + _TRAIN_HI) / 2).astype(np.float32)
    a = (x.double() - torch.from_numpy(shift.astype(np.float64)).to(DEV)) * torch.from_numpy(
        scale.astype(np.float64)).to(DEV)
    acts, zs = [a], []
    for k in range(4):
        z = a @ W[k].T + b[k]
        a = z * torch.sigmoid(z)
        zs.append(z)
        acts.append(a)
    return (a @ W[4].T + b[4])[:, 0], acts, zs


# The box the surrogate trains on: the trusted one widened by a fifth where the model allows it.
_W = (BOX_HI - BOX_LO) * 0.1
_TRAIN_LO = np.maximum(BOX_LO - _W, [0.05, 0.001, 0.02, -0.98, 0.001, 0.02, -np.inf])
_TRAIN_HI = np.minimum(BOX_HI + _W, [np.inf, np.inf, np.inf, 0.98, np.inf, np.inf, np.inf])


def exact(case, seed):
    case = _sizes(case)
    kind = case["kind"]
    if kind in ("sfft", "dense", "shots"):
        P = _problems(case, seed)
        if kind == "shots":   # outcomes are whole numbers; the squared norm is the integrand's
            norm = [float((_terms(P, i, _frequencies(P, i)).abs() ** 2).sum()) for i in range(case["batch"])]
            return None, None, None, np.array(norm)
        if not case["strikes"]:
            out = torch.stack([_all_prices(P, i) for i in range(case["batch"])])
        else:
            _, start, step = _strikes(case, P)
            out = torch.stack([_window_prices(P, i, int(start[i]), int(step[i]), case["strikes"])
                               for i in range(case["batch"])])
        return out if kind == "sfft" else dict(prices=out, status=None)
    if kind == "query":
        W, b = _net64(_net(seed).net)
        z = _forward64(W, b, torch.from_numpy(_queries(case["rows"], seed)).to(DEV))[0]
        return torch.exp(z) - 0.01, None
    state = prepare(case, seed)
    net = state["net"]
    W, b = _net64(net)
    x, t = state["x"], state["t"].double()
    z, acts, zs = _forward64(W, b, x)
    d = (2.0 * (z - t) / len(t))[:, None]
    grads = [None] * 5
    for k in range(4, -1, -1):
        grads[k] = torch.cat([(d.T @ acts[k]).reshape(-1), d.sum(0)])
        if k:
            s = torch.sigmoid(zs[k - 1])
            d = (d @ W[k]) * s * (1.0 + zs[k - 1] * (1.0 - s))
    g = torch.cat(grads)
    m = 0.9 * net.m.double() + 0.1 * g
    v = 0.999 * net.v.double() + 0.001 * g * g
    t1 = net.t + 1
    p = net.params.double() - 1e-3 * (m / (1.0 - 0.9 ** t1)) / (torch.sqrt(v / (1.0 - 0.999 ** t1)) + 1e-8)
    return dict(grad=g, params=p, m=m, v=v)
