"""The calls whose speed is followed from one version of the library to the next.

A case is one call (or one iteration) that a program using this library makes:

* ``step``      one iteration of the exact gradient descent with P stored;
* ``implicit``  the same with P recomputed in every pass;
* ``fit``       the start of a run on new points: affinities, then the first gradient;
* ``dissim``    the same from a given matrix of dissimilarities;
* ``batch``     one sweep of the batched iteration over many independent problems;
* ``ptsne``     one epoch of the parallel scheme;
* ``predict``   the surrogate network on new points;
* ``train``     one training step of the surrogate (gradient and Adam);
* ``pakde``     the density raster of a finished map, bandwidths included.

Inputs are Gaussian mixtures (the inputs of the benchmark and of the tests),
drawn on the GPU from the seed alone. Maps in mid-run are drawn as clusters,
as in ``synth.clustered_state``, so that a state depends on no optimiser.
"""
import math

import numpy as np
import torch

from paper_1812_09869_amd import _lib
from paper_1812_09869_amd.surrogate import Surrogate
from paper_1812_09869_amd.tsne import ExactTSNE, PTSNE, Schedule, pakde


def listed():
    return [
        # The smallest problems of the tests and of interactive use: an
        # iteration is a few launches and nothing else.
        {"name": "step_n300", "kind": "step", "n": 300, "d": 10, "k": 4, "perp": 20.0, "t": 400},
        # The 2,000-point workload whose whole run the oracle holds: the size
        # of most published example sets.
        {"name": "step_n2000", "kind": "step", "n": 2000, "d": 10, "k": 8, "perp": 30.0, "t": 10},
        # An ordinary set, not a multiple of anything (the batch's own range
        # is 1,000 to 20,000 points).
        {"name": "step_n12345", "kind": "step", "n": 12345, "d": 50, "k": 10, "perp": 30.0,
         "t": 400},
        # The benchmark's iteration.
        {"name": "step_n65536", "kind": "step", "n": 65536, "d": 50, "k": 32, "perp": 50.0,
         "t": 400},
        # The start of a run on a small set, distances in FP64 (the default).
        {"name": "fit_n2000", "kind": "fit", "n": 2000, "d": 10, "k": 8, "perp": 30.0,
         "mode": "fp64", "t": 0},
        # The start of the benchmark's run, in the distance mode it uses.
        {"name": "fit_n65536_x3", "kind": "fit", "n": 65536, "d": 50, "k": 32, "perp": 50.0,
         "mode": "bf16x3", "t": 0},
        # The benchmark's batch: 64 problems of 1,000 to 20,000 points.
        {"name": "batch_64", "kind": "batch", "count": 64, "lo": 1000, "hi": 20000, "t": 400,
         "pick": 7},
        # The paper's rounds figure: 60,000 points in 30 dimensions, 120
        # partial problems of two layers, perplexity 400.
        {"name": "ptsne_n60000", "kind": "ptsne", "n": 60000, "d": 30, "k": 10, "threads": 120,
         "layers": 2, "perp": 400.0},
        # P recomputed (sets beyond what a stored P fits), at the benchmark's
        # size and in its distance mode.
        {"name": "implicit_n65536_x3", "kind": "implicit", "n": 65536, "d": 50, "k": 32,
         "perp": 50.0, "mode": "bf16x3", "t": 400},
        # Mapping a million new points with the trained network.
        {"name": "predict_1m", "kind": "predict", "n": 1048576, "d": 50, "hidden": 256},
        # Training that network: one minibatch.
        {"name": "train_b1024", "kind": "train", "n": 65536, "d": 50, "hidden": 256,
         "batch": 1024},
        # The density raster of a finished map of the benchmark's size.
        {"name": "pakde_n65536", "kind": "pakde", "n": 65536, "k": 32, "perp": 100.0, "gx": 512,
         "gy": 512},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["step", "step", "step", "fit", "fit", "dissim", "batch", "ptsne",
                       "implicit", "predict", "train", "pakde"])
    if kind in ("step", "fit", "implicit"):
        n = _log_int(rng, 300, 65536)
        c = {"kind": kind, "n": n, "d": rng.choice([3, 10, 30, 50, 64, 128]),
             "k": rng.randint(4, 32), "perp": float(rng.randint(8, 50)),
             "t": rng.choice([10, 400])}
        if kind != "step":
            # FP64 is the library's default, BF16x3 the benchmark's choice; the
            # other modes trade precision for speed
            c["mode"] = rng.choice(["fp64", "fp64", "bf16x3", "bf16x3", "fp16x3", "fp32",
                                    "bf16"])
        return c
    if kind == "dissim":
        n = _log_int(rng, 300, 16384)
        return {"kind": kind, "n": n, "d": rng.choice([3, 10, 50]), "k": rng.randint(4, 32),
                "perp": float(rng.randint(8, 50)), "t": 0}
    if kind == "batch":
        return {"kind": kind, "count": _log_int(rng, 2, 64), "lo": 1000,
                "hi": _log_int(rng, 2000, 20000), "t": rng.choice([10, 400]),
                "pick": rng.randint(0, 1 << 20)}
    if kind == "ptsne":
        threads = _log_int(rng, 4, 120)
        layers = rng.randint(1, 3)
        size = _log_int(rng, 150, 1000)  # points of one partial problem
        n = max(threads * 60, min(60000, size * threads // layers))
        least = layers * (n // threads)
        return {"kind": kind, "n": n, "d": rng.choice([10, 30, 50]), "k": 10,
                "threads": threads, "layers": layers, "perp": float(int(least * 0.25))}
    if kind == "predict":
        return {"kind": kind, "n": _log_int(rng, 100, 1048576), "d": rng.choice([2, 10, 30, 50, 64]),
                "hidden": rng.choice([64, 128, 192, 256, 256])}
    if kind == "train":
        return {"kind": kind, "n": 65536, "d": rng.choice([10, 30, 50, 64]),
                "hidden": rng.choice([64, 128, 256, 256]),
                "batch": rng.choice([300, 512, 1000, 1024, 2048, 4096])}
    return {"kind": "pakde", "n": _log_int(rng, 1000, 65536), "k": rng.randint(4, 32),
            "perp": float(rng.randint(20, 100)), "gx": _log_int(rng, 64, 512),
            "gy": _log_int(rng, 64, 512)}


# ---------------------------------------------------------------------------
# Inputs
# ---------------------------------------------------------------------------

def _gen(seed):
    return torch.Generator(device="cuda").manual_seed(int(seed) * 1000003 + 17)


def _randn(g, *shape):
    return torch.randn(*shape, generator=g, device="cuda", dtype=torch.float32)


def _rand(g, *shape):
    return torch.rand(*shape, generator=g, device="cuda", dtype=torch.float32)


def _mixture(g, n, d, k):
    """n points of k Gaussian components (means ~ N(0, 25 I), a spread of its
    own for each coordinate of each component, variances in [0.1, 10])."""
    lab = torch.randint(0, k, (n,), generator=g, device="cuda")
    means = 5.0 * _randn(g, k, d)
    scale = torch.exp(0.5 * (math.log(0.1) + math.log(100.0) * _rand(g, k, d)))
    return (means[lab] + scale[lab] * _randn(g, n, d)).contiguous(), lab


def _map(g, lab, k):
    """A map in mid-run: clusters at random centres."""
    centres = 8.0 * _randn(g, k, 2)
    return (centres[lab] + _randn(g, lab.shape[0], 2)).contiguous()


def _momentum(g, n):
    return (0.05 * _randn(g, n, 2)).contiguous()


def _gains(g, n):
    return (0.05 + 1.5 * _rand(g, n, 2)).contiguous()


def _points_case(case, seed):
    g = _gen(seed)
    x, lab = _mixture(g, case["n"], case["d"], case["k"])
    y = _map(g, lab, case["k"])
    return x, y, _momentum(g, case["n"]), _gains(g, case["n"])


def _batch_sizes(case):
    # the sizes of a batch belong to the case; its points come from the seed
    r = np.random.Generator(np.random.PCG64(case["pick"]))
    return [(int(r.integers(case["lo"], case["hi"] + 1)), int(r.choice([10, 50])),
             int(r.integers(4, 17))) for _ in range(case["count"])]


def _batch_inputs(case, seed):
    g = _gen(seed)
    xs, ys = [], []
    for n, d, k in _batch_sizes(case):
        lab = torch.randint(0, k, (n,), generator=g, device="cuda")
        xs.append((5.0 * _randn(g, k, d)[lab] + _randn(g, n, d)).contiguous())
        ys.append(_map(g, lab, k))
    y = torch.cat(ys).contiguous()
    return xs, y, _momentum(g, y.shape[0]), _gains(g, y.shape[0])


def _pt_inputs(case, seed):
    g = _gen(seed)
    n = case["n"]
    x, _ = _mixture(g, n, case["d"], case["k"])
    r, a = torch.sqrt(_rand(g, n)), 2.0 * math.pi * _rand(g, n)
    y0 = torch.stack([r * torch.cos(a), r * torch.sin(a)], dim=1).contiguous()
    order = torch.randperm(n, generator=g, device="cuda").to(torch.int32)
    return x, y0, order


def _net_inputs(case, seed):
    """Points, standardisation and He-normal weights as the surrogate has them."""
    g = _gen(seed)
    d, h = case["d"], case["hidden"]
    x, lab = _mixture(g, case["n"], d, 32)
    mean = x.mean(dim=0).contiguous()
    invstd = (1.0 / x.std(dim=0)).contiguous()
    params = torch.cat([(_randn(g, h * d) * math.sqrt(2.0 / d)), 0.1 * _randn(g, h),
                        (_randn(g, h * h) * math.sqrt(2.0 / h)), 0.1 * _randn(g, h),
                        (_randn(g, 2 * h) * math.sqrt(1.0 / h)), 0.1 * _randn(g, 2)])
    return x, lab, mean, invstd, params.contiguous(), g


def _train_inputs(case, seed):
    x, lab, mean, invstd, params, g = _net_inputs(case, seed)
    y = _map(g, lab, 32)
    y = ((y - y.mean(dim=0)) / y.std()).contiguous()
    idx = torch.randperm(case["n"], generator=g, device="cuda").to(torch.int32)[:case["batch"]]
    # Adam's moments in mid-training
    m = (1e-3 * _randn(g, params.shape[0])).contiguous()
    v = (1e-6 * (0.25 + _rand(g, params.shape[0]))).contiguous()
    return x, y, idx.contiguous(), mean, invstd, params, m, v


ADAM = (1e-3, 0.9, 0.999, 1e-8)
ADAM_T = 500  # steps taken before the measured one


def _kde_inputs(case, seed):
    g = _gen(seed)
    lab = torch.randint(0, case["k"], (case["n"],), generator=g, device="cuda")
    y = (10.0 * _randn(g, case["k"], 2)[lab] + 2.5 * _randn(g, case["n"], 2)).contiguous()
    # the raster of a case is fixed and covers every map that it draws
    side = 90.0
    return y, -side / 2, -side / 2, side / case["gx"], side / case["gy"]


def prepare(case, seed):
    kind = case["kind"]
    if kind in ("step", "implicit"):
        x, y, u, g = _points_case(case, seed)
        model = ExactTSNE(x, case["perp"], dist_mode=case.get("mode", "fp64"),
                          implicit=kind == "implicit")
        return {"kind": kind, "model": model, "state": (y, u, g), "t": case["t"],
                "sched": Schedule()}
    if kind == "fit":
        x, y, _, _ = _points_case(case, seed)
        return {"kind": kind, "x": x, "y": y, "case": case,
                "ws": _lib.new_workspace(case["n"], case["d"], case["mode"])}
    if kind == "dissim":
        x, y, _, _ = _points_case(case, seed)
        return {"kind": kind, "dis": _dissim(x), "y": y, "case": case}
    if kind == "batch":
        xs, y, u, g = _batch_inputs(case, seed)
        models = [ExactTSNE(x, 30.0) for x in xs]
        rows, at = [], 0
        for m in models:
            rows.append((m.ws, m.n, y[at:at + m.n], u[at:at + m.n], g[at:at + m.n]))
            at += m.n
        arr = _lib.batch_problems(rows)
        return {"kind": kind, "models": models, "rows": rows, "arr": arr,
                "bws": _lib.batch_plan(arr), "state": (y, u, g), "t": case["t"],
                "sched": Schedule()}
    if kind == "ptsne":
        x, y0, order = _pt_inputs(case, seed)
        model = PTSNE(x, case["threads"], case["layers"], case["perp"])
        model.init_maps(y0)
        return {"kind": kind, "model": model, "order": order}
    if kind == "predict":
        x, _, mean, invstd, params, _ = _net_inputs(case, seed)
        net = Surrogate(case["d"], case["hidden"])
        net.mean, net.invstd, net.params = mean, invstd, params
        return {"kind": kind, "net": net, "x": x,
                "out": torch.empty(case["n"], 2, device="cuda")}
    if kind == "train":
        x, y, idx, mean, invstd, params, m, v = _train_inputs(case, seed)
        return {"kind": kind, "x": x, "y": y, "idx": idx, "mean": mean, "invstd": invstd,
                "params": params, "m": m, "v": v, "grad": torch.empty_like(params),
                "loss": torch.zeros(1, dtype=torch.float64, device="cuda"), "t": ADAM_T,
                "d": case["d"], "hidden": case["hidden"], "batch": case["batch"],
                "ws": _lib.mlp_new_workspace(case["d"], case["hidden"], case["batch"], True)}
    y, x0, y0, cx, cy = _kde_inputs(case, seed)
    return {"kind": kind, "y": y, "perp": case["perp"],
            "raster": (x0, y0, cx, cy, case["gx"], case["gy"])}


def run(state):
    kind = state["kind"]
    if kind in ("step", "implicit"):
        state["model"].step(state["t"], state["state"], state["sched"])
        return state["state"]
    if kind == "fit":
        c = state["case"]
        model = ExactTSNE(state["x"], c["perp"], dist_mode=c["mode"], ws=state["ws"])
        return model.gradient(state["y"], Schedule()(c["t"])[0])[0]
    if kind == "dissim":
        c = state["case"]
        model = ExactTSNE.from_dissimilarities(state["dis"], c["perp"])
        return model.gradient(state["y"], Schedule()(c["t"])[0])[0]
    if kind == "batch":
        alpha, mu, eta = state["sched"](state["t"])
        _lib.batch_step(state["arr"], state["bws"], alpha, mu, eta, state["sched"].min_gain)
        return state["state"]
    if kind == "ptsne":
        monitors = state["model"].epoch(state["order"])
        # the maps go on to the next epoch; the monitors are logged in single
        # precision
        return state["model"].maps, monitors.float()
    if kind == "predict":
        return state["net"].predict(state["x"], state["out"])
    if kind == "train":
        s = state
        _lib.mlp_gradient(s["params"], s["d"], s["hidden"], s["mean"], s["invstd"], s["x"],
                          s["y"], s["idx"], s["batch"], s["grad"], s["loss"], s["ws"])
        s["t"] += 1
        _lib.mlp_adam(s["params"], s["grad"], s["m"], s["v"], *ADAM, s["t"])
        return s["params"], s["m"], s["v"], s["grad"], s["loss"].float()
    return pakde(state["y"], state["perp"], *state["raster"])


# ---------------------------------------------------------------------------
# Work that a pass cannot do without
# ---------------------------------------------------------------------------

def work(case):
    """Inputs read once, outputs written once. A stored P counts the pairs of
    one mixture component (those of two components underflow to zero), and a
    pair costs 17 operations of repulsion, 9 more of attraction where P holds
    something."""
    kind = case["kind"]
    if kind == "batch":
        sizes = _batch_sizes(case)
        pairs = sum(n * (n - 1) / 2 for n, _, _ in sizes)
        held = sum(n * (n - 1) / 2 / k for n, _, k in sizes)
        return {"bytes": 4 * held + 48 * sum(n for n, _, _ in sizes),
                "flops": 17 * pairs + 9 * held}
    n = case["n"]
    pairs = n * (n - 1) / 2
    held = pairs / case.get("k", 1)
    if kind == "step":
        return {"bytes": 4 * held + 48 * n, "flops": 17 * pairs + 9 * held}
    if kind == "implicit":
        return {"bytes": 4 * n * case["d"] + 48 * n,
                "flops": 17 * pairs + 9 * held + 2 * case["d"] * held}
    if kind == "fit":
        # P is written and read once; the distances, about four passes of the
        # search (two operations and an exponential for each ordered pair)
        return {"bytes": 4 * n * case["d"] + 8 * held + 16 * n,
                "flops": 2 * case["d"] * pairs + 24 * pairs + 17 * pairs + 9 * held}
    if kind == "dissim":
        return {"bytes": 4 * n * n + 8 * held + 16 * n, "flops": 24 * pairs + 17 * pairs + 9 * held}
    if kind == "ptsne":
        z = case["n"] * case["layers"] / case["threads"]
        p = case["threads"] * z * (z - 1) / 2
        iters = math.ceil(math.sqrt(z))
        return {"bytes": 4 * n * case["d"] + 16 * n * case["layers"] + 4 * n + 4 * p * iters,
                "flops": 2 * case["d"] * p + 24 * p + iters * 26 * p}
    d = case.get("d", 2)
    if kind == "predict":
        h = case["hidden"]
        return {"bytes": 4 * n * d + 8 * n, "flops": 2.0 * n * (d * h + h * h + 2 * h)}
    if kind == "train":
        h, b = case["hidden"], case["batch"]
        w = d * h + h * h + 2 * h
        return {"bytes": 4 * b * (d + 2) + 32 * w, "flops": 6.0 * b * w}
    cells = case["gx"] * case["gy"]
    return {"bytes": 8 * n + 8 * n + 4 * cells, "flops": 4.0 * n * n + 24 * n * n + 2.0 * n * cells}


# ---------------------------------------------------------------------------
# The same in plain FP64 torch
# ---------------------------------------------------------------------------

F64 = torch.float64


def _dissim(x):
    """Euclidean distances in FP64, rounded once, exactly symmetric."""
    xd = x.double()
    out = torch.empty(x.shape[0], x.shape[0], device=x.device)
    for r in range(0, x.shape[0], 1024):
        out[r:r + 1024] = torch.cdist(xd[r:r + 1024], xd,
                                      compute_mode="donot_use_mm_for_euclid_dist").float()
    out = torch.triu(out, 1)
    return (out + out.t()).contiguous()


def _sq_points(x):
    c = x.double() - x.double().mean(dim=0)
    nrm = (c * c).sum(dim=1)
    return lambda r0, r1: (nrm[r0:r1, None] + nrm[None, :] - 2.0 * (c[r0:r1] @ c.t())).clamp_min_(0)


def _chunk(n):
    return max(1, min(n, (1 << 26) // n))


def _search(sq, n, perp):
    """beta, m and S of every row: the entropy of its conditional is ln(perp)."""
    target, step = math.log(perp), _chunk(n)
    beta_all, m_all, s_all = (torch.empty(n, dtype=F64, device="cuda") for _ in range(3))
    for r0 in range(0, n, step):
        r1 = min(n, r0 + step)
        d = sq(r0, r1)
        at = torch.arange(r0, r1, device="cuda")
        d[at - r0, at] = math.inf
        m = d.min(dim=1).values
        d -= m[:, None]
        d[at - r0, at] = 1e300  # its weight is zero at every beta
        lo = torch.zeros(r1 - r0, dtype=F64, device="cuda")
        hi = torch.full_like(lo, math.inf)
        beta = torch.ones_like(lo)
        for it in range(120):
            e = torch.exp(-beta[:, None] * d)
            s = e.sum(dim=1)
            e *= d
            e[at - r0, at] = 0.0
            t = e.sum(dim=1) / s
            e *= d
            e[at - r0, at] = 0.0
            var = (e.sum(dim=1) / s - t * t).clamp_min(0)
            off = torch.log(s) + beta * t - target
            if it % 4 == 3 and float(off.abs().max()) < 1e-12:
                break
            lo = torch.where(off > 0, beta, lo)
            hi = torch.where(off > 0, hi, beta)
            new = beta + off / (beta * var)
            bad = ~torch.isfinite(new) | (new <= lo) | (new >= hi)
            mid = torch.where(torch.isinf(hi), 2.0 * beta, 0.5 * (lo + hi))
            new = torch.where(bad, mid, new)
            beta = torch.where(off.abs() < 1e-14, beta, new)
        e = torch.exp(-beta[:, None] * d)
        beta_all[r0:r1], m_all[r0:r1], s_all[r0:r1] = beta, m, e.sum(dim=1)
    return beta_all, m_all, s_all


def _gradient(sq, n, stats, y, alpha):
    """4 (alpha A - R / Z) of Eq. 6 for P from the rows' statistics."""
    beta, m, s = stats
    yd, step = y.double(), _chunk(n)
    a, r = (torch.empty(n, 2, dtype=F64, device="cuda") for _ in range(2))
    z = torch.zeros((), dtype=F64, device="cuda")
    for r0 in range(0, n, step):
        r1 = min(n, r0 + step)
        d = sq(r0, r1)
        p = torch.exp(-beta[r0:r1, None] * (d - m[r0:r1, None])) / s[r0:r1, None]
        p += torch.exp(-beta[None, :] * (d - m[None, :])) / s[None, :]
        p /= 2.0 * n
        dx = yd[r0:r1, None, 0] - yd[None, :, 0]
        dy = yd[r0:r1, None, 1] - yd[None, :, 1]
        w = 1.0 / (1.0 + dx * dx + dy * dy)
        at = torch.arange(r0, r1, device="cuda")
        w[at - r0, at] = 0.0
        z += w.sum()
        p *= w
        a[r0:r1, 0], a[r0:r1, 1] = (p * dx).sum(dim=1), (p * dy).sum(dim=1)
        w *= w
        r[r0:r1, 0], r[r0:r1, 1] = (w * dx).sum(dim=1), (w * dy).sum(dim=1)
    return 4.0 * (alpha * a - r / z)


def _step(grad, y, u, g, mu, eta, min_gain):
    y, u, g = y.double(), u.double(), g.double()
    g = torch.where((grad > 0) != (u > 0), g + 0.2, g * 0.8).clamp_min(min_gain)
    u = mu * u - eta * g * grad
    y = y + u
    return y - y.mean(dim=0), u, g


def _exact_step(x, perp, y, u, g, t):
    n = x.shape[0]
    sq = _sq_points(x)
    alpha, mu, eta = Schedule()(t)
    grad = _gradient(sq, n, _search(sq, n, perp), y, alpha)
    return _step(grad, y, u, g, mu, eta, Schedule().min_gain)


def _exact_ptsne(case, seed):
    x, y0, order = _pt_inputs(case, seed)
    n, threads, layers = case["n"], case["threads"], case["layers"]
    maps = y0.double().unsqueeze(0).repeat(layers, 1, 1)
    out = maps.clone()
    base, extra = divmod(n, threads)
    ends = np.cumsum([0] + [base + (1 if c < extra else 0) for c in range(threads)])
    order = order.long()
    iters = math.ceil(math.sqrt(n * layers / threads))
    costs = []
    for k in range(threads):
        rows, lay = [], []
        for l in range(layers):
            c = (k + l) % threads
            rows.append(order[ends[c]:ends[c + 1]])
            lay += [l] * int(ends[c + 1] - ends[c])
        rows, lay = torch.cat(rows), torch.tensor(lay, device="cuda")
        z = rows.shape[0]
        sq = _sq_points(x[rows])(0, z)
        beta, m, s = _search(lambda r0, r1: sq[r0:r1].clone(), z, case["perp"])
        p = torch.exp(-beta[:, None] * (sq - m[:, None])) / s[:, None]
        p = (p + p.t()) / (2.0 * z)
        p.fill_diagonal_(0.0)
        y = maps[lay, rows]
        u = torch.zeros_like(y)
        for _ in range(iters):
            dx = y[:, None, :] - y[None, :, :]
            w = 1.0 / (1.0 + (dx * dx).sum(dim=2))
            w.fill_diagonal_(0.0)
            c = p * w - w * w / w.sum()
            grad = 4.0 * (c.sum(dim=1, keepdim=True) * y - c @ y)
            ext = (y.max(dim=0).values - y.min(dim=0).values).max()
            u = 0.8 * u - (math.log(z - 1) * ext / 2) * grad
            y = y + u
        dx = y[:, None, :] - y[None, :, :]
        q = 1.0 + (dx * dx).sum(dim=2)
        w = 1.0 / q
        w.fill_diagonal_(0.0)
        cross = (p * torch.log(q)).sum() + p.sum() * torch.log(w.sum())
        costs.append(cross / math.log(z * (z - 1)))
        out[lay, rows] = y
    ext = out.max(dim=1).values - out.min(dim=1).values
    size = (ext * ext).sum(dim=1).sqrt().mean()
    return out, torch.stack([torch.stack(costs).mean(), size])


def _layers(case, params):
    d, h = case["d"], case["hidden"]
    cut = torch.split(params.double(), [h * d, h, h * h, h, 2 * h, 2])
    return (cut[0].view(h, d), cut[1], cut[2].view(h, h), cut[3], cut[4].view(2, h), cut[5])


def _exact_predict(case, seed):
    x, _, mean, invstd, params, _ = _net_inputs(case, seed)
    w1, b1, w2, b2, w3, b3 = _layers(case, params)
    out = torch.empty(case["n"], 2, dtype=F64, device="cuda")
    for r in range(0, case["n"], 65536):
        v = (x[r:r + 65536].double() - mean.double()) * invstd.double()
        v = torch.relu(torch.relu(v @ w1.t() + b1) @ w2.t() + b2)
        out[r:r + 65536] = v @ w3.t() + b3
    return out


def _exact_train(case, seed):
    x, y, idx, mean, invstd, params, m, v = _train_inputs(case, seed)
    w1, b1, w2, b2, w3, b3 = _layers(case, params)
    i, b = idx.long(), case["batch"]
    h0 = (x[i].double() - mean.double()) * invstd.double()
    h1 = torch.relu(h0 @ w1.t() + b1)
    h2 = torch.relu(h1 @ w2.t() + b2)
    e = h2 @ w3.t() + b3 - y[i].double()
    loss = (e * e).sum() / (2 * b)
    e = e / b
    d2 = (e @ w3) * (h2 > 0)
    d1 = (d2 @ w2) * (h1 > 0)
    grad = torch.cat([(d1.t() @ h0).reshape(-1), d1.sum(dim=0), (d2.t() @ h1).reshape(-1),
                      d2.sum(dim=0), (e.t() @ h2).reshape(-1), e.sum(dim=0)])
    lr, c1, c2, eps = ADAM
    t = ADAM_T + 1
    m, v = c1 * m.double() + (1 - c1) * grad, c2 * v.double() + (1 - c2) * grad * grad
    p = params.double() - lr * (m / (1 - c1 ** t)) / (torch.sqrt(v / (1 - c2 ** t)) + eps)
    return p, m, v, grad, loss.reshape(1)


def _exact_pakde(case, seed):
    y, x0, y0, cx, cy = _kde_inputs(case, seed)
    n, yd = case["n"], y.double()

    def sq(r0, r1):
        d = (yd[r0:r1, None, 0] - yd[None, :, 0]) ** 2
        return d.add_((yd[r0:r1, None, 1] - yd[None, :, 1]) ** 2)

    beta = _search(sq, n, case["perp"])[0]
    # the library takes the raster's corner and cells in FP32
    x0, y0, cx, cy = (float(np.float32(v)) for v in (x0, y0, cx, cy))
    u = x0 + (torch.arange(case["gx"], device="cuda", dtype=F64) + 0.5) * cx
    v = y0 + (torch.arange(case["gy"], device="cuda", dtype=F64) + 0.5) * cy
    f = torch.zeros(case["gy"], case["gx"], dtype=F64, device="cuda")
    for r in range(0, n, 16384):
        b = beta[r:r + 16384, None]
        ex = torch.exp(-b * (u[None, :] - yd[r:r + 16384, 0:1]) ** 2)
        ey = torch.exp(-b * (v[None, :] - yd[r:r + 16384, 1:2]) ** 2) * (b / math.pi)
        f += ey.t() @ ex
    return beta, f * (cx * cy / n)


def exact(case, seed):
    kind = case["kind"]
    if kind in ("step", "implicit"):
        x, y, u, g = _points_case(case, seed)
        return _exact_step(x, case["perp"], y, u, g, case["t"])
    if kind in ("fit", "dissim"):
        x, y, _, _ = _points_case(case, seed)
        if kind == "fit":
            sq = _sq_points(x)
        else:
            dis = _dissim(x).double()
            sq = lambda r0, r1: dis[r0:r1] ** 2  # noqa: E731
        return _gradient(sq, case["n"], _search(sq, case["n"], case["perp"]), y,
                         Schedule()(case["t"])[0])
    if kind == "batch":
        xs, y, u, g = _batch_inputs(case, seed)
        parts, at = [], 0
        for x in xs:
            s = slice(at, at + x.shape[0])
            parts.append(_exact_step(x, 30.0, y[s], u[s], g[s], case["t"]))
            at += x.shape[0]
        return tuple(torch.cat([p[q] for p in parts]) for q in range(3))
    if kind == "ptsne":
        return _exact_ptsne(case, seed)
    if kind == "predict":
        return _exact_predict(case, seed)
    if kind == "train":
        return _exact_train(case, seed)
    return _exact_pakde(case, seed)
