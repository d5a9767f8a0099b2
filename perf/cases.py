"""The workloads whose speed this library is judged by: what a program that
uses it has it do, through the public entry points, over the range of sizes,
types and options that such programs have.

    listed()             the named cases
    draw(rng)            one more case of the same ranges
    prepare(case, seed)  what the program has in hand before the call
    run(state)           one pass, returning its outputs
    work(case)           the bytes and operations a pass cannot do without
    exact(case, seed)    the outputs in binary64, without the library
"""

import math

import numpy as np
import torch

from paper_2312_02756_amd import autograd, glv

DEV = "cuda"
DTYPES = {"f64": torch.float64, "f32": torch.float32}
TARGET = 91.1876  # GeV: the resonance the best pair is chosen for
HIST = (0.0, 400.0, 1000)  # GeV, GeV, bins


def listed():
    return [
        # The smallest calls: one batch of a loop over small files or of an
        # interactive session.  Latency and launches count.
        {"name": "mass_small", "op": "mass", "n": 4096, "dtype": "f64", "coords": "PtEtaPhiM", "mode": "plain",
         "layout": "columns"},
        {"name": "events_small", "op": "events", "ne": 1000, "mean": 8.0, "shape": 0.0, "cap": 64, "dtype": "f64",
         "coords": "PtEtaPhiM", "mode": "plain"},
        # Pair masses in a fit or a training step: forward and backward.
        {"name": "mass_grad", "op": "mass_grad", "n": 1 << 24, "dtype": "f64", "coords": "PtEtaPhiM", "mode": "plain",
         "layout": "columns"},
        # The largest: light, nearly collinear pairs in FP32 with the
        # cancellation-free mass (the precision stress).
        {"name": "mass_comp", "op": "mass", "n": 1 << 26, "dtype": "f32", "coords": "PtEtaPhiM",
         "mode": "compensated", "layout": "columns"},
        # The analysis step: a spectrum of pair masses, never stored.
        {"name": "mass_hist", "op": "mass_hist", "n": 1 << 24, "dtype": "f64", "coords": "PtEtaPhiM", "mode": "plain",
         "layout": "columns"},
        # Boosts with one velocity per vector, forward and backward, on the
        # rows of one (k, n) block with odd n, as a ragged batch leaves them.
        {"name": "boost_grad", "op": "boost_grad", "n": 10000019, "dtype": "f32", "layout": "rows"},
        # A change of frame: detector coordinates to Cartesian, one Lorentz
        # matrix for all vectors, and back.
        {"name": "frame", "op": "frame", "n": 5000003, "dtype": "f64", "layout": "columns"},
        # Jagged collider events: pair offsets, then totals, event masses and
        # all pair masses; FP64 and the FP32 cancellation-free mode.
        {"name": "events", "op": "events", "ne": 1 << 20, "mean": 8.0, "shape": 0.0, "cap": 64, "dtype": "f64",
         "coords": "PtEtaPhiM", "mode": "plain"},
        {"name": "events_comp", "op": "events", "ne": 1 << 20, "mean": 8.0, "shape": 0.0, "cap": 64, "dtype": "f32",
         "coords": "PtEtaPhiM", "mode": "compensated"},
        # The same reduction inside a training step.
        {"name": "events_grad", "op": "events_grad", "ne": 1 << 19, "mean": 8.0, "shape": 0.0, "cap": 64,
         "dtype": "f64", "coords": "PtEtaPhiM", "mode": "plain"},
        # Events of many objects (clusters, subjets), sizes widely spread:
        # negative binomial with a mean of 96.
        {"name": "events_dense", "op": "events_grad", "ne": 4096, "mean": 96.0, "shape": 2.0, "cap": 1024,
         "dtype": "f32", "coords": "PtEtaPhiM", "mode": "plain"},
        # Selection: each event's pair closest to a resonance.
        {"name": "events_best", "op": "events_best", "ne": 1 << 20, "mean": 8.0, "shape": 0.0, "cap": 64,
         "dtype": "f64", "coords": "PtEtaPhiM", "mode": "plain"},
    ]


def draw(rng):
    op = rng.choice(["mass", "mass_grad", "mass_hist", "boost_grad", "frame", "events", "events", "events_grad",
                     "events_grad", "events_best"])
    case = {"op": op, "dtype": rng.choice(["f64", "f32"])}
    if op.startswith("events"):
        mean = math.exp(rng.uniform(math.log(2.0), math.log(128.0)))
        shape = rng.choice([0.0, 0.0, 2.0, 5.0])  # 0: Poisson
        # E[n (n - 1) / 2] = mean^2 (1 + 1/shape) / 2 pairs per event
        pairs = 0.5 * mean * mean * (1.0 + (1.0 / shape if shape else 0.0))
        most = min(1 << 20, int((1 << 24) / (pairs + mean)))
        if op == "events_grad":
            most //= 2
        case["ne"] = int(math.exp(rng.uniform(math.log(50.0), math.log(max(most, 100)))))
        case.update(mean=round(mean, 3), shape=shape, cap=rng.choice([64, 256, 1024]))
        case["mode"] = "plain" if op == "events_grad" else rng.choice(["plain", "compensated"])
        case["coords"] = "PtEtaPhiM" if case["mode"] == "compensated" else rng.choice(["PtEtaPhiM", "PxPyPzE"])
        return case
    most = 1 << (26 if op == "mass" and case["dtype"] == "f32" else 24)
    n = int(math.exp(rng.uniform(math.log(1000.0), math.log(most))))
    case["n"] = n - n % 16 if rng.random() < 0.4 else n
    case["layout"] = rng.choice(["columns", "columns", "rows"])
    if op.startswith("mass"):
        case["mode"] = rng.choice(["plain", "compensated"])
        case["coords"] = ("PtEtaPhiM" if case["mode"] == "compensated"
                          else rng.choice(["PtEtaPhiM", "PtEtaPhiM", "PxPyPzE", "PtEtaPhiE", "PxPyPzM"]))
    return case


# ------------------------------------------------------------------ inputs

def _uniform(g, n, lo, hi):
    return torch.rand(n, dtype=torch.float64, device=DEV, generator=g).mul_(hi - lo).add_(lo)


def _normal(g, n):
    return torch.randn(n, dtype=torch.float64, device=DEV, generator=g)


def _leg(g, n, kind="generic"):
    """(pt, eta, phi, M) of n particles: generic collider legs, light ones over
    a wide range of pt, or jets with a mass of their own (the plain form's
    FP32 gradients mean little for nearly massless collinear legs)."""
    if kind == "light":
        pt = torch.exp(_uniform(g, n, 0.0, math.log(2000.0)))
        return [pt, _uniform(g, n, -4.0, 4.0), _uniform(g, n, -math.pi, math.pi), _uniform(g, n, 0.0, 0.14)]
    pt = torch.empty(n, dtype=torch.float64, device=DEV).exponential_(1.0 / 30.0, generator=g).add_(5.0)
    lo, hi = (2.0, 20.0) if kind == "jets" else (0.0, 0.2)
    return [pt, _uniform(g, n, -2.5, 2.5), _uniform(g, n, -math.pi, math.pi), _uniform(g, n, lo, hi)]


def _kind(case):
    if case["mode"] == "compensated":
        return "light"
    return "jets" if case["op"].endswith("_grad") and case["dtype"] == "f32" else "generic"


def _cart(c):
    pt, eta, phi, m = c
    return [pt * torch.cos(phi), pt * torch.sin(phi), pt * torch.sinh(eta), torch.hypot(pt * torch.cosh(eta), m)]


def _in_coords(c, coords):
    if coords == "PtEtaPhiM":
        return c
    v = _cart(c)
    return {"PxPyPzE": v, "PtEtaPhiE": [*c[:3], v[3]], "PxPyPzM": [*v[:3], c[3]]}[coords]


def _lay(cols, dtype, layout):
    """Columns of their own, or the rows of one (k, n) block."""
    if layout == "rows":
        block = torch.empty(len(cols), cols[0].numel(), dtype=dtype, device=DEV)
        for row, c in zip(block, cols):
            row.copy_(c)
        return tuple(block[k] for k in range(len(cols)))
    return tuple(c.to(dtype) for c in cols)


def _lorentz_matrix():
    """A rotation about z followed by a boost: 16 row-major numbers."""
    c, s = math.cos(0.7), math.sin(0.7)
    rot = np.array([[c, -s, 0, 0], [s, c, 0, 0], [0, 0, 1, 0], [0, 0, 0, 1.0]])
    b = np.array([0.2, -0.1, 0.5])
    g = 1.0 / math.sqrt(1.0 - b @ b)
    boost = np.eye(4)
    boost[:3, :3] += g * g / (1.0 + g) * np.outer(b, b)
    boost[:3, 3] = boost[3, :3] = g * b
    boost[3, 3] = g
    return (boost @ rot).reshape(-1)


def _inputs(case, seed):
    """The inputs of a case, in its types and layout."""
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    op, dt = case["op"], DTYPES[case["dtype"]]
    s = {"case": case}
    if op.startswith("events"):
        # the sizes belong to the case, their order to the seed: every seed has as many pairs
        gs = torch.Generator(device=DEV)
        gs.manual_seed(2312)
        rate = torch.full((case["ne"],), case["mean"], dtype=torch.float64, device=DEV)
        if case["shape"]:  # negative binomial: Poisson of a gamma-distributed rate
            k = int(case["shape"])
            e = torch.empty(k, case["ne"], dtype=torch.float64, device=DEV).exponential_(1.0, generator=gs)
            rate *= e.sum(0) / k
        cnt = torch.poisson(rate, generator=gs).clamp_(max=case["cap"]).to(torch.int64)
        cnt = cnt[torch.randperm(case["ne"], device=DEV, generator=g)]
        off = torch.zeros(case["ne"] + 1, dtype=torch.int64, device=DEV)
        torch.cumsum(cnt, 0, out=off[1:])
        s["offsets"] = off
        s["n_pairs"] = int((cnt * (cnt - 1) // 2).sum().item())
        n = int(off[-1].item())
        s["p"] = _lay(_in_coords(_leg(g, n, _kind(case)), case["coords"]), dt, "columns")
        if op == "events_grad":
            s["up"] = tuple(_normal(g, m).to(dt) for m in [case["ne"]] * 5 + [s["n_pairs"]])
        return s
    n, layout = case["n"], case["layout"]
    if op.startswith("mass"):
        a, b = _leg(g, n, _kind(case)), _leg(g, n, _kind(case))
        if case["mode"] == "compensated":  # a tenth of the pairs nearly collinear
            near = _uniform(g, n, 0.0, 1.0) < 0.1
            for k, most in ((1, 4.0), (2, math.pi)):
                b[k] = torch.where(near, (a[k] + _uniform(g, n, -1e-3, 1e-3)).clamp_(-most, most), b[k])
        s["a"] = _lay(_in_coords(a, case["coords"]), dt, layout)
        s["b"] = _lay(_in_coords(b, case["coords"]), dt, layout)
        if op == "mass_grad":
            s["up"] = (_normal(g, n).to(dt),)
    elif op == "boost_grad":
        x = [_normal(g, n) * 50.0 for _ in range(3)]
        m = _uniform(g, n, 0.0, 100.0)
        x.append(torch.sqrt(x[0] ** 2 + x[1] ** 2 + x[2] ** 2 + m * m))
        cth, az, mag = _uniform(g, n, -1.0, 1.0), _uniform(g, n, -math.pi, math.pi), _uniform(g, n, 0.0, 0.99)
        sth = torch.sqrt(1.0 - cth * cth)
        s["x"] = _lay(x, dt, layout)
        s["beta"] = _lay([mag * sth * torch.cos(az), mag * sth * torch.sin(az), mag * cth], dt, layout)
        s["up"] = _lay([_normal(g, n) for _ in range(4)], dt, layout)
    else:  # frame
        s["x"] = _lay(_leg(g, n), dt, layout)
        s["L"] = tuple(torch.tensor([v], dtype=torch.float64, device=DEV).to(dt) for v in _lorentz_matrix())
    return s


def prepare(case, seed):
    s = _inputs(case, seed)
    if case["op"].endswith("_grad"):
        for key in ("a", "b", "x", "beta", "p"):
            for c in s.get(key, ()):
                c.requires_grad_(True)
    return s


def run(state):
    case = state["case"]
    op, mode, coords = case["op"], case.get("mode"), case.get("coords")
    if op == "mass":
        return glv.glv_invariant_mass(state["a"], state["b"], coords=coords, mode=mode)
    if op == "mass_grad":
        m = autograd.invariant_mass(state["a"], state["b"], coords=coords, mode=mode)
        return (m.detach(), *torch.autograd.grad(m, (*state["a"], *state["b"]), state["up"][0]))
    if op == "mass_hist":
        return glv.glv_invariant_mass_histogram(state["a"], state["b"], *HIST, coords=coords, mode=mode)
    if op == "boost_grad":
        y = autograd.boost(state["x"], state["beta"])
        return (*(c.detach() for c in y), *torch.autograd.grad(y, (*state["x"], *state["beta"]), state["up"]))
    if op == "frame":
        v = glv.glv_convert(state["x"], "PtEtaPhiM", "PxPyPzE")
        w = glv.glv_lorentz_transform(v, state["L"])
        return (*v, *w, *glv.glv_convert(w, "PxPyPzE", "PtEtaPhiM"))
    if op == "events":
        po = glv.glv_pair_offsets(state["offsets"])
        total, em, pm = glv.glv_event_reduce(state["p"], state["offsets"], po, coords=coords, mode=mode,
                                             n_pairs=state["n_pairs"])
        return (po, *total, em, pm)
    if op == "events_grad":
        total, em, pm = autograd.event_reduce(state["p"], state["offsets"], coords=coords)
        out = (*total, em, pm)
        return (*(c.detach() for c in out), *torch.autograd.grad(out, state["p"], state["up"]))
    rank, bm = glv.glv_event_reduce_best_pair(state["p"], state["offsets"], TARGET, coords=coords, mode=mode)
    return rank, bm


def work(case):
    es = 8 if case["dtype"] == "f64" else 4
    op = case["op"]
    if op.startswith("events"):
        ne, mean = case["ne"], case["mean"]
        parts = ne * mean
        pairs = 0.5 * ne * mean * mean * (1.0 + (1.0 / case["shape"] if case["shape"] else 0.0))
        b = 4 * es * parts + 8 * ne  # particles, offsets
        if op == "events_best":
            return {"bytes": b + (8 + es) * ne, "flops": 60 * parts + 25 * pairs}
        comp = case["mode"] == "compensated"
        b += 5 * es * ne + es * pairs + (8 * ne if op == "events" else 0)
        f = (100 if comp else 60) * parts + (50 if comp else 20) * pairs
        if op == "events_grad":
            b += 5 * es * ne + es * pairs + 4 * es * parts
            f += 100 * parts + 45 * pairs
        return {"bytes": b, "flops": f}
    n = case["n"]
    cols, flops = {"mass": (9, 130), "mass_grad": (18, 320), "mass_hist": (8, 140), "boost_grad": (22, 130),
                   "frame": (16, 230)}[op]
    return {"bytes": cols * es * n, "flops": flops * n}


# ------------------------------------------------------- binary64 reference

def _pair_mass2(a, b, coords):
    """m^2 of pairs of legs.  PtEtaPhiM: the cancellation-free form; otherwise
    E^2 - |P|^2 of the sum.  Returns (m^2, E_a E_b - p_a.p_b or None)."""
    if coords != "PtEtaPhiM":
        v = [x + y for x, y in zip(_to_cart(a, coords), _to_cart(b, coords))]
        return v[3] * v[3] - v[0] * v[0] - v[1] * v[1] - v[2] * v[2]

    def parts(c):
        pt, eta, _, m = c
        mt = torch.sqrt(pt * pt + m * m)
        pc = pt * torch.cosh(eta)
        delta = -torch.asinh(m * m * torch.sinh(eta) / (mt * (pc + torch.sqrt(pc * pc + m * m))))
        return mt, delta, m * m / (mt + pt)

    mta, da, ca = parts(a)
    mtb, db, cb = parts(b)
    dy = (a[1] - b[1]) + (da - db)
    dphi = torch.remainder(a[2] - b[2] + math.pi, 2 * math.pi) - math.pi
    dphi = torch.where((a[2] - b[2]).abs() < math.pi, a[2] - b[2], dphi)
    k = (2 * mta * mtb * torch.sinh(0.5 * dy) ** 2 + 2 * a[0] * b[0] * torch.sin(0.5 * dphi) ** 2
         + ca * mtb + a[0] * cb)
    return a[3] ** 2 + b[3] ** 2 + 2 * k


def _to_cart(c, coords):
    if coords == "PxPyPzE":
        return list(c)
    if coords == "PxPyPzM":
        return [*c[:3], torch.sqrt(c[0] ** 2 + c[1] ** 2 + c[2] ** 2 + c[3] ** 2)]
    v = _cart(c)
    return v if coords == "PtEtaPhiM" else [*v[:3], c[3]]


def _signed_sqrt(q):
    return torch.sign(q) * torch.sqrt(q.abs())


def _wide(cols, grad=False):
    return [c.detach().to(torch.float64).clone().requires_grad_(grad) for c in cols]


def _pair_index(off):
    """The two particles of every pair, events in order, i < j lexicographic."""
    n = int(off[-1].item())
    cnt = off[1:] - off[:-1]
    end = torch.repeat_interleave(off[1:], cnt)
    left = end - torch.arange(n, device=DEV) - 1  # partners after each particle
    i = torch.repeat_interleave(torch.arange(n, device=DEV), left)
    start = torch.cumsum(left, 0) - left
    j = i + 1 + torch.arange(i.numel(), device=DEV) - start[i]
    return i, j, torch.repeat_interleave(torch.arange(cnt.numel(), device=DEV), cnt)


def _exact_events(case, s):
    grad = case["op"] == "events_grad"
    off, coords = s["offsets"], case["coords"]
    p = _wide(s["p"], grad)
    i, j, ev = _pair_index(off)
    ne = case["ne"]
    zero = torch.zeros(ne, dtype=torch.float64, device=DEV)
    total = [zero.index_add(0, ev, v) for v in _to_cart(p, coords)]
    q = _pair_mass2([c[i] for c in p], [c[j] for c in p], coords)
    pm = _signed_sqrt(q)
    if coords == "PtEtaPhiM":  # sum of M^2 plus twice the sum of E_i E_j - p_i.p_j
        m2 = p[3] * p[3]
        em2 = zero.index_add(0, ev, m2).index_add(0, ev[i], q - m2[i] - m2[j])
    else:
        em2 = total[3] ** 2 - total[0] ** 2 - total[1] ** 2 - total[2] ** 2
    em = _signed_sqrt(em2)
    if case["op"] == "events_best":
        po = torch.zeros(ne + 1, dtype=torch.int64, device=DEV)
        cnt = off[1:] - off[:-1]
        torch.cumsum(cnt * (cnt - 1) // 2, 0, out=po[1:])
        d = (pm - TARGET).abs()
        best = torch.full((ne,), math.inf, dtype=torch.float64, device=DEV).index_reduce(0, ev[i], d, "amin")
        hit = d == best[ev[i]]
        bm = torch.full((ne,), math.nan, dtype=torch.float64, device=DEV)
        bm[ev[i][hit]] = pm[hit]
        return (None, bm)
    out = (*total, em, pm)
    if grad:
        return (*(c.detach() for c in out),
                *torch.autograd.grad(out, p, [u.to(torch.float64) for u in s["up"]]))
    return (None, *out)


def exact(case, seed):
    s = _inputs(case, seed)
    op = case["op"]
    if op == "mass_hist":
        return None  # counts
    if op.startswith("events"):
        return _exact_events(case, s)
    if op.startswith("mass"):
        grad = op == "mass_grad"
        a, b = _wide(s["a"], grad), _wide(s["b"], grad)
        m = _signed_sqrt(_pair_mass2(a, b, case["coords"]))
        if not grad:
            return m
        return (m.detach(), *torch.autograd.grad(m, (*a, *b), s["up"][0].to(torch.float64)))
    if op == "boost_grad":
        x, beta = _wide(s["x"], True), _wide(s["beta"], True)
        g = 1.0 / torch.sqrt(1.0 - (beta[0] ** 2 + beta[1] ** 2 + beta[2] ** 2))
        sdot = beta[0] * x[0] + beta[1] * x[1] + beta[2] * x[2]
        c = g * g / (1.0 + g) * sdot + g * x[3]
        y = [*(x[k] + c * beta[k] for k in range(3)), g * (x[3] + sdot)]
        return (*(c.detach() for c in y),
                *torch.autograd.grad(y, (*x, *beta), [u.to(torch.float64) for u in s["up"]]))
    x, lm = _wide(s["x"]), [v.to(torch.float64) for v in s["L"]]
    v = _to_cart(x, "PtEtaPhiM")
    w = [lm[4 * r] * v[0] + lm[4 * r + 1] * v[1] + lm[4 * r + 2] * v[2] + lm[4 * r + 3] * v[3] for r in range(4)]
    pt = torch.hypot(w[0], w[1])
    back = [pt, torch.asinh(w[2] / pt), torch.atan2(w[1], w[0]), None]  # M: the input's, lost to cancellation
    return (*v, *w, *back)
