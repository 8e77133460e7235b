"""The work this library is timed on: completions of synthetic traffic tensors (OD pairs x
time slots x days, and the other layouts), through the Python binding's public calls.

Kinds of a case:
  step      a completion under way: `iters` more iterations of a kept context, then W
  watch     the same in single iterations with the objective read after each, then W, Z, X, Y
  resume    a saved state restored into a kept context, one more iteration, then W and Z
  complete  the one-call form: a new problem completed from scratch (W and f0)
  unroll    a held-out error differentiated through the unrolled iterations
  batch     `count` uneven completions advanced together, then every W

Inputs follow the recipe of the seeded workloads: a low-tubal-rank core with unit-mean
factors, log-normal OD scales, diurnal and weekly profiles, noise, clipping at 0 and a
uniformly random mask; X0 = 0 and Y0 ~ N(0, 1).
"""
import math
import random

import numpy as np
import torch

from paper_2005_09838_amd import Batch, Completion, complete
from paper_2005_09838_amd.autodiff import unrolled_completion

DEV = "cuda:0"


def _step(name, n1, n2, n3, r, p, iters, rho1=1e-2):
    return {"name": name, "kind": "step", "n1": n1, "n2": n2, "n3": n3, "r": r, "p": p, "iters": iters,
            "precision": "fp32", "rho1": rho1}


def listed():
    return [
        # the smallest workload: 36 OD pairs, half-hour slots, one week; launches and latency
        _step("small_36x48x7", 36, 48, 7, 3, 0.3, 20),
        # five-minute slots over four weeks: the ordinary size
        _step("mid_144x288x28", 144, 288, 28, 8, 0.4, 20),
        # quarter-hour slots over 112 days, the benchmark's workload
        _step("large_529x96x112", 529, 96, 112, 16, 0.4, 20),
        # the same in mixed precision, from a checkpoint.  One iteration: stochastic BF16
        # rounding turns a difference in the last FP32 bit into BF16-sized ones in the next
        {"name": "mixed_529x96x112", "kind": "resume", "n1": 529, "n2": 96, "n3": 112, "r": 16, "p": 0.4, "iters": 1,
         "precision": "mixed", "rho1": 1e-2},
        # the mid-size data as slot x day x OD pair (the model's layout): the tube is the OD pair
        _step("slot_day_od_288x28x144", 288, 28, 144, 8, 0.4, 10),
        # and as origin x destination x time: few, very long tubes
        _step("router_pairs_12x12x8064", 12, 12, 8064, 8, 0.4, 2),
        # a rank past 16 with strong temporal smoothing (the separate solve along mode 1)
        _step("rank24_300x120x24", 300, 120, 24, 24, 0.5, 20, rho1=0.3),
        # a ragged size with an odd tube, followed iteration by iteration
        {"name": "watch_70x50x9", "kind": "watch", "n1": 70, "n2": 50, "n3": 9, "r": 5, "p": 0.4, "iters": 8},
        # a new problem from scratch to its completed tensor
        {"name": "complete_144x288x28", "kind": "complete", "n1": 144, "n2": 288, "n3": 28, "r": 8, "p": 0.4,
         "iters": 50},
        # weights tuned by gradient: the held-out error through the unrolled iterations
        {"name": "unroll_144x288x28", "kind": "unroll", "n1": 144, "n2": 288, "n3": 28, "r": 8, "p": 0.4,
         "iters": 6, "every": 3},
        # many networks at once
        {"name": "batch_16_uneven", "kind": "batch", "count": 16, "sizes": 1, "iters": 10},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


FAST_TUBES = tuple(range(1, 17)) + (20, 24, 28, 32, 40, 48, 56, 64, 84, 96, 112, 128)


def draw(rng):
    kind = rng.choice(("step", "step", "step", "step", "tubes", "routers", "watch", "resume", "complete", "unroll",
                       "batch"))
    p = round(rng.uniform(0.1, 0.8), 3)
    if kind == "batch":
        return {"kind": "batch", "count": rng.randint(4, 16), "sizes": rng.randint(2, 1 << 20), "iters": 10}
    if kind == "routers":
        # N x N router pairs over slots x days
        n = rng.randint(9, 12)
        n3 = rng.choice((24, 48, 96, 144, 288)) * rng.randint(7, 28)
        return {"kind": "step", "n1": n, "n2": n, "n3": n3, "r": rng.randint(2, 8), "p": p, "iters": 2,
                "precision": "fp32", "rho1": 1e-2}
    n1, n2 = _log_int(rng, 12, 529), _log_int(rng, 12, 288)
    if kind == "tubes":
        # any tube length: OD pairs or odd numbers of days along the tube
        n3, most = _log_int(rng, 17, 400), 1_200_000
    else:
        n3, most = rng.choice(FAST_TUBES[4:] + (7, 28, 112)), 5_600_000
    if kind == "unroll":
        most = 1_100_000
    while n1 * n2 * n3 > most:
        if n1 >= n2:
            n1 = max(12, n1 * 2 // 3)
        else:
            n2 = max(12, n2 * 2 // 3)
    r = rng.randint(2, min(n1, n2, 24 if rng.random() < 0.2 else 16))
    if kind == "watch":
        return {"kind": "watch", "n1": n1, "n2": n2, "n3": n3, "r": r, "p": p, "iters": 8}
    if kind == "resume":
        return {"kind": "resume", "n1": n1, "n2": n2, "n3": n3, "r": r, "p": p, "iters": 1,
                "precision": rng.choice(("mixed", "mixed", "fp32")), "rho1": 1e-2}
    if kind == "complete":
        return {"kind": "complete", "n1": n1, "n2": n2, "n3": n3, "r": r, "p": p, "iters": rng.randint(10, 50)}
    if kind == "unroll":
        r = min(r, 8)
        return {"kind": "unroll", "n1": n1, "n2": n2, "n3": n3, "r": r, "p": max(p, 0.2), "iters": rng.randint(2, 6),
                "every": rng.randint(1, 4)}
    return {"kind": "step", "n1": n1, "n2": n2, "n3": n3, "r": r, "p": p, "iters": 10, "precision": "fp32",
            "rho1": rng.choice((0.0, 1e-2, 1e-2, 0.1, 0.3))}


def _inputs(n1, n2, n3, r, p, seed):
    g = torch.Generator(device=DEV).manual_seed(seed)
    normal = lambda *s: torch.randn(*s, generator=g, device=DEV, dtype=torch.float64)
    xf = torch.fft.rfft(1.0 + normal(n3, n1, r), dim=0)
    yf = torch.fft.rfft(1.0 + normal(n3, r, n2), dim=0)
    core = torch.fft.irfft(torch.matmul(xf, yf), n=n3, dim=0).permute(1, 2, 0)
    core = core * torch.exp(normal(n1))[:, None, None]
    j = torch.arange(n2, device=DEV, dtype=torch.float64)
    k = torch.arange(n3, device=DEV, dtype=torch.float64)
    core = core * (1.0 + 0.3 * torch.sin(2.0 * math.pi * j / n2))[None, :, None]
    core = core * (1.0 + 0.3 * torch.sin(2.0 * math.pi * k / 7.0))[None, None, :]
    rms = core.square().mean().sqrt()
    m = (core + 0.02 * rms * normal(n1, n2, n3)).clamp_min(0.0).float().contiguous()
    u = torch.rand(n1, n2, n3, generator=g, device=DEV)
    omega = u < p
    hold = (u >= p) & (u < p + 0.1)
    return {"M": m, "omega": omega.to(torch.uint8).contiguous(), "hold": hold,
            "G": torch.where(omega, m, torch.zeros_like(m)).contiguous(),
            "X0": torch.zeros(n1, r, n3, device=DEV), "Y0": normal(r, n2, n3).float().contiguous()}


def _batch_sizes(case):
    """Uneven sizes as in the batch workload, from the case's own number."""
    rng = random.Random(case["sizes"])
    return [(rng.choice((36, 144, 529)), rng.choice((48, 96, 288)), rng.choice((7, 28, 112)), rng.randint(2, 16),
             rng.uniform(0.2, 0.6)) for _ in range(case["count"])]


def prepare(case, seed):
    if case["kind"] == "batch":
        probs = []
        for t, (n1, n2, n3, r, p) in enumerate(_batch_sizes(case)):
            d = _inputs(n1, n2, n3, r, p, seed * 100 + t)
            probs.append({"G": d["G"], "omega": d["omega"], "r": r, "X0": d["X0"], "Y0": d["Y0"]})
        return {"case": case, "batch": Batch(probs)}
    d = _inputs(case["n1"], case["n2"], case["n3"], case["r"], case["p"], seed)
    state = {"case": case, "in": d}
    if case["kind"] in ("step", "watch", "resume"):
        state["ctx"] = Completion(d["G"], d["omega"], case["r"], rho1=case.get("rho1", 1e-2),
                                  precision=case.get("precision", "fp32"), X0=d["X0"], Y0=d["Y0"])
        if case["kind"] == "resume":
            state["saved"] = state["ctx"].get_state()
    elif case["kind"] == "unroll":
        state["theta"] = torch.tensor([1e-2, 1e-2, 1e-2], device=DEV, requires_grad=True)
        state["Y0"] = d["Y0"].clone().requires_grad_(True)
        hold = d["hold"].double()
        state["hold"] = hold
        state["target"] = d["M"].double() * hold
        state["norm"] = torch.linalg.vector_norm(state["target"])
    return state


def run(state):
    case = state["case"]
    kind = case["kind"]
    if kind == "step":
        c = state["ctx"]
        c.step(case["iters"])
        return c.result()
    if kind == "watch":
        c = state["ctx"]
        f0 = []
        for _ in range(case["iters"]):
            c.step(1)
            f0.append(c.objective())
        return {"f0": f0, **c.result(W=True, Z=True, X=True, Y=True)}
    if kind == "resume":
        c = state["ctx"]
        c.set_state(state["saved"])
        c.step(case["iters"])
        return c.result(W=True, Z=True)
    if kind == "complete":
        d = state["in"]
        w, info = complete(d["G"], d["omega"], case["r"], iters=case["iters"], X0=d["X0"], Y0=d["Y0"])
        return {"W": w, "f0": info["f0"]}
    if kind == "unroll":
        d = state["in"]
        w = unrolled_completion(state["theta"], d["X0"], state["Y0"], d["G"], d["omega"], case["r"], case["iters"],
                                case["every"])
        loss = torch.linalg.vector_norm(w * state["hold"] - state["target"]) / state["norm"]
        theta_bar, y0_bar = torch.autograd.grad(loss, (state["theta"], state["Y0"]))
        return {"W": w.detach().float(), "loss": loss.detach().float(), "theta_bar": theta_bar, "Y0_bar": y0_bar}
    b = state["batch"]
    b.step(case["iters"])
    return [b[k].result()["W"] for k in range(len(b))]


def _iteration_work(n1, n2, n3, r, precision="fp32"):
    """One iteration: read G once, write W~ once and read it once, read and write the factors;
    three complex products, two tube transforms and the row solves."""
    nb = n3 // 2 + 1
    n, nh = n1 * n2 * n3, n1 * n2 * nb
    sw = 4 if precision == "mixed" else 8
    nbytes = 4 * n + 2 * sw * nh + 5 * 8 * nb * r * n1 + 4 * 8 * nb * r * n2
    flops = 3 * 8 * nh * r + 5.0 * n * math.log2(max(n3, 2)) + 10.0 * n
    return nbytes, flops


def work(case):
    if case["kind"] == "batch":
        parts = [_iteration_work(n1, n2, n3, r) + (n1 * n2 * n3,) for n1, n2, n3, r, _ in _batch_sizes(case)]
        return {"bytes": sum(case["iters"] * b + 4 * n for b, _, n in parts),
                "flops": case["iters"] * sum(f for _, f, _ in parts)}
    n = case["n1"] * case["n2"] * case["n3"]
    b, f = _iteration_work(case["n1"], case["n2"], case["n3"], case["r"], case.get("precision", "fp32"))
    out = 4 * n
    if case["kind"] == "watch":
        out = 4 * (2 * n + (case["n1"] + case["n2"]) * case["r"] * case["n3"])
    if case["kind"] == "resume":
        # the restored state is read and written, W and Z written
        nh, fac = case["n1"] * case["n2"] * (case["n3"] // 2 + 1), (case["n1"] + case["n2"]) * case["r"] * (case["n3"] // 2 + 1)
        out = 8 * n + 2 * ((4 if case["precision"] == "mixed" else 8) * nh + 8 * fac)
    if case["kind"] == "complete":
        out += 5 * n                   # G and the mask
    if case["kind"] == "unroll":
        # forward, and backward about twice it in FP64 (twice the bytes), W_bar in
        b, f, out = 5 * b, 3 * f, 5 * n + 8 * n + 8 * n
    return {"bytes": case["iters"] * b + out, "flops": case["iters"] * f}


# ---- the same in 64 bits with plain torch

def _pinv(g):
    """Inverse of Hermitian Grams [nb][r][r], eigenvalues up to r eps lambda_max dropped."""
    r = g.shape[-1]
    lam, v = np.linalg.eigh(g.detach().cpu().numpy())
    keep = lam > np.maximum(r * np.finfo(np.float64).eps * lam[:, -1:], 0.0)
    inv = np.where(keep, 1.0 / np.where(keep, lam, 1.0), 0.0)
    return torch.from_numpy((v * inv[:, None, :]) @ v.conj().transpose(0, 2, 1)).to(g.device)


def _second_difference(n):
    """D^T D of the first differences along n entries."""
    a = torch.zeros(n, n, device=DEV, dtype=torch.float64)
    if n > 1:
        d = torch.eye(n, device=DEV, dtype=torch.float64)
        d = d[1:] - d[:-1]
        a = d.t().contiguous() @ d
    return a


def _w_step(z, g, obs, mu, rho2):
    """w = g on observed entries; elsewhere the tridiagonal equations along mode 2.
    z, g, obs: [n2][rows]."""
    n2 = z.shape[0]
    cs, ds = [], []
    c = torch.zeros_like(z[0])
    d = torch.zeros_like(z[0])
    zero = torch.zeros_like(z[0])
    for j in range(n2):
        deg = 0.0 if n2 == 1 else (1.0 if j in (0, n2 - 1) else 2.0)
        lo = rho2 if j > 0 else 0.0
        up = rho2 if j + 1 < n2 else 0.0
        piv = 1.0 + mu + rho2 * deg - lo * c
        d = torch.where(obs[j], g[j], (z[j] + lo * d) / piv)
        c = torch.where(obs[j], zero, up / piv + zero)
        cs.append(c)
        ds.append(d)
    w = [None] * n2
    nxt = torch.zeros_like(z[0])
    for j in range(n2 - 1, -1, -1):
        nxt = ds[j] + cs[j] * nxt
        w[j] = nxt
    return torch.stack(w)


def _solve_h(h, a):
    """h^{-1} a for real h [n1][n1] and complex a [nb][n1][r]."""
    nb, n1, r = a.shape
    flat = a.permute(1, 0, 2).reshape(n1, nb * r)
    both = torch.linalg.solve(h, torch.cat((flat.real, flat.imag), dim=1))
    out = torch.complex(both[:, : nb * r].contiguous(), both[:, nb * r:].contiguous())
    return out.reshape(n1, nb, r).permute(1, 0, 2).contiguous()


class _Exact:
    """The iteration on stored frequencies: X [nb][n1][r], Y [nb][r][n2], W~ [nb][n1][n2]."""

    def __init__(self, d, mu, rho1, rho2, differentiable=False):
        self.n1, self.n2, self.n3 = d["G"].shape
        self.mu, self.rho1, self.rho2, self.diff = mu, rho1, rho2, differentiable
        self.h = torch.eye(self.n1, device=DEV, dtype=torch.float64) + rho1 * _second_difference(self.n1)
        self.obs = d["omega"].bool().permute(1, 0, 2).reshape(self.n2, -1).contiguous()
        self.g = d["G"].double().permute(1, 0, 2).reshape(self.n2, -1).contiguous()
        self.w = torch.where(d["omega"].bool(), d["G"].double(), torch.zeros((), device=DEV, dtype=torch.float64))
        self.wt = self.dft(self.w)
        self.x = self.dft(d["X0"].double())
        self.y = self.dft(d["Y0"].double())

    def dft(self, a):
        # root exp(+2 pi i / n3): the conjugate of torch's
        return torch.fft.rfft(a, dim=2).conj().resolve_conj().permute(2, 0, 1).contiguous()

    def idft(self, a):
        return torch.fft.irfft(a.permute(1, 2, 0).conj().resolve_conj().contiguous(), n=self.n3, dim=2)

    def inverse(self, g):
        return torch.linalg.inv(g) if self.diff else _pinv(g)

    def iterate(self):
        t = lambda a: a.conj().transpose(1, 2).resolve_conj().contiguous()
        yh = t(self.y)
        self.x = _solve_h(self.h, self.wt @ yh @ self.inverse(self.y @ yh))
        hc = self.h.to(torch.complex128)
        xh = t(self.x)
        self.y = self.inverse(xh @ torch.matmul(hc, self.x)) @ (xh @ self.wt)
        z = self.idft(self.x @ self.y)
        w = _w_step(z.permute(1, 0, 2).reshape(self.n2, -1), self.g, self.obs, self.mu, self.rho2)
        self.z, self.w = z, w.reshape(self.n2, self.n1, self.n3).permute(1, 0, 2)
        self.wt = self.dft(self.w)

    def objective(self):
        f = 0.5 * (self.z - self.w).square().sum() + 0.5 * self.mu * self.w.square().sum()
        f = f + 0.5 * self.rho1 * (self.z[1:] - self.z[:-1]).square().sum()
        return f + 0.5 * self.rho2 * (self.w[:, 1:] - self.w[:, :-1]).square().sum()


def exact(case, seed):
    if case["kind"] == "batch":
        out = []
        for t, (n1, n2, n3, r, p) in enumerate(_batch_sizes(case)):
            if n1 * n2 * n3 > 1_500_000:
                out.append(None)
                continue
            e = _Exact(_inputs(n1, n2, n3, r, p, seed * 100 + t), 1e-2, 1e-2, 1e-2)
            for _ in range(case["iters"]):
                e.iterate()
            out.append(e.w.contiguous())
        return out
    d = _inputs(case["n1"], case["n2"], case["n3"], case["r"], case["p"], seed)
    kind = case["kind"]
    if kind == "unroll":
        w32 = torch.tensor([1e-2, 1e-2, 1e-2], device=DEV).double()
        theta = w32.clone().requires_grad_(True)
        y0 = d["Y0"].double().requires_grad_(True)
        e = _Exact({**d, "Y0": y0}, theta[0], theta[1], theta[2], differentiable=True)
        for _ in range(case["iters"]):
            e.iterate()
        hold = d["hold"].double()
        target = d["M"].double() * hold
        loss = torch.linalg.vector_norm(e.w * hold - target) / torch.linalg.vector_norm(target)
        theta_bar, y0_bar = torch.autograd.grad(loss, (theta, y0))
        return {"W": e.w.detach().contiguous(), "loss": loss.detach(), "theta_bar": theta_bar, "Y0_bar": y0_bar}
    e = _Exact(d, 1e-2, case.get("rho1", 1e-2), 1e-2)
    f0 = []
    for _ in range(case["iters"]):
        e.iterate()
        if kind == "watch":
            f0.append(float(e.objective()))
    if kind == "watch":
        return {"f0": f0, "W": e.w.contiguous(), "Z": e.z.contiguous(), "X": e.idft(e.x).contiguous(),
                "Y": e.idft(e.y).contiguous()}
    if kind == "resume":
        return {"W": e.w.contiguous(), "Z": e.z.contiguous()}
    if kind == "complete":
        return {"W": e.w.contiguous(), "f0": float(e.objective())}
    return {"W": e.w.contiguous()}
