"""Performance cases of the Newman-Ziff sweep: the work that programs built on
this package have it do, through its public entry points.

A case is a dict of plain values.  Kinds:

  sweep      nz_sweep: host arrays in and out, the library's own workspace
  batch      nz_sweep_batch on a kept workspace, as bench.py runs it: the plan
             of every pass comes from the prefill MLP ("learned": bulk prefill,
             "plain": a plain sweep with the learned key band)
  static     nz_sweep_batch_static: small batches in a serving loop that
             allocates nothing
  pmax       fss.pmax_curve: P_max(p) from the largest-cluster window
  train      one training step of the prefill MLP (forward, loss, backward,
             Adam), as learned.train runs it
  canonical  nz_canonical: the binomial convolution of an n* histogram

n* and masses are integers fixed by (L, mask, seed, sample), whatever the plan.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2607_18991_amd import autotune, fss, learned, nz

COMPACT = "1,3,7,15,31,63,127"
ZONE_SIZES = (10, 40, 80, 90, 112, 240, 320)
# the p grid of the threshold estimate (fss.py's default grid)
P_LO, P_HI, P_STEP = 0.1375, 0.1440, 0.0001


def listed():
    return [
        # the smallest call: one small lattice through the host entry point,
        # where latency and launches count
        dict(name="sweep_L4_zone1", kind="sweep", L="4", masks="1", samples=1000, boundary=0),
        # a serving loop's request: an odd lattice, a non-compact neighbourhood,
        # a handful of samples, nothing allocated
        dict(name="static_L13_0x2b", kind="static", L="13", masks="43", samples=37, plan="learned", boundary=0),
        # the L = 8 table, a tenth of its samples
        dict(name="batch_L8_compact", kind="batch", L="8", masks=COMPACT, samples=1000, plan="learned", boundary=0),
        # the uneven batch: five lattice sizes in one call
        dict(name="batch_L8-20_compact", kind="batch", L="8,10,12,16,20", masks=COMPACT, samples=100, plan="learned",
             boundary=0),
        # the benchmark's batch, learned and plain
        dict(name="batch_L16_compact", kind="batch", L="16", masks=COMPACT, samples=1000, plan="learned", boundary=0),
        dict(name="batch_L16_compact_plain", kind="batch", L="16", masks=COMPACT, samples=1000, plan="plain",
             boundary=0),
        # every neighbourhood at L = 16 with few samples each
        dict(name="batch_L16_127masks", kind="batch", L="16", masks=",".join(str(m) for m in range(1, 128)),
             samples=24, plan="learned", boundary=0),
        # the largest tabulated lattice
        dict(name="batch_L24_compact", kind="batch", L="24", masks=COMPACT, samples=200, plan="learned", boundary=0),
        # first wrapping under periodic boundaries (the mass fit)
        dict(name="batch_L12_periodic", kind="batch", L="12", masks=COMPACT, samples=100, plan="learned", boundary=1),
        # one lattice of the threshold estimate by finite-size scaling
        dict(name="pmax_L12_zone1", kind="pmax", L="12", masks="1", samples=1000, boundary=1),
        # one step of the MLP's training on its 170 lattices
        dict(name="train_170", kind="train", rows=170),
        # R_L(p) on 101 points from an n* histogram at L = 16
        dict(name="canonical_L16", kind="canonical", L="16", points=101, samples=1000),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["batch"] * 7 + ["sweep", "sweep", "static", "pmax", "train", "canonical"])
    if kind == "train":
        return dict(kind="train", rows=_log_int(rng, 7, 600))
    if kind == "canonical":
        return dict(kind="canonical", L=str(rng.randint(4, 20)), points=rng.randint(11, 151),
                    samples=_log_int(rng, 100, 10000))
    if kind == "pmax":
        return dict(kind="pmax", L=str(rng.randint(6, 16)), masks="1", samples=_log_int(rng, 50, 800),
                    boundary=rng.randint(0, 1))
    if kind == "static":
        return dict(kind="static", L=str(rng.randint(5, 20)), masks=str(rng.randint(1, 127)),
                    samples=rng.randint(1, 60), plan=rng.choice(["learned", "plain"]), boundary=0)
    if kind == "sweep":
        L = rng.randint(4, 14)
        return dict(kind="sweep", L=str(L), masks=str(rng.randint(1, 127)),
                    samples=min(2000, max(1, int(_log_int(rng, 1e7, 2e8) / L**5))),
                    boundary=1 if L >= 5 and rng.random() < 0.3 else 0)
    Ls = sorted({rng.randint(5, 25) for _ in range(rng.choice([1, 1, 2, 3]))})
    masks = sorted({rng.choice([int(m) for m in COMPACT.split(",")]) if rng.random() < 0.4 else rng.randint(1, 127)
                    for _ in range(rng.randint(1, 9))})
    plan = rng.choice(["learned", "learned", "learned", "plain"])
    boundary = 1 if rng.random() < 0.15 else 0
    # total sites over samples, well inside the largest listed batch's
    budget = _log_int(rng, 2e7, 3e9) / ((4 if plan == "plain" else 1) * (4 if boundary else 1))
    per_sample = sum(L**5 for L in Ls) * len(masks)
    samples = min(3000, max(1, int(budget / per_sample)))
    return dict(kind="batch", L=",".join(map(str, Ls)), masks=",".join(map(str, masks)), samples=samples, plan=plan,
                boundary=boundary)


def _ints(text):
    return [int(v) for v in text.split(",")]


def _jobs(case, seed):
    """One job per (L, mask); every L has its own Philox seed."""
    return [dict(L=L, zone_mask=m, seed=0x5EED_0000_0000 + 4096 * int(seed) + L, nsamples=int(case["samples"]),
                 boundary=int(case["boundary"])) for L in _ints(case["L"]) for m in _ints(case["masks"])]


def _plan(state):
    if state["plan"] == "learned":
        return state["model"].plan(state["jobs"], **state["depth"])
    return learned.plan_band_only(state["model"], state["jobs"])


def prepare(case, seed):
    kind = case["kind"]
    if kind == "sweep":
        return dict(kind=kind, L=int(case["L"]), mask=int(case["masks"]), samples=int(case["samples"]),
                    seed=0x5EED_0000_0000 + int(seed), boundary=int(case["boundary"]))
    if kind in ("batch", "static"):
        jobs = _jobs(case, seed)
        total = sum(j["nsamples"] for j in jobs)
        state = dict(kind=kind, jobs=jobs, plan=case["plan"], model=learned.PrefillModel.load(), depth={},
                     nstar=torch.zeros(total, dtype=torch.int32, device="cuda"),
                     mass=torch.zeros(total, dtype=torch.int32, device="cuda"))
        planned = _plan(state)
        if kind == "batch":
            if case["plan"] == "learned":
                # the tuned prefill depth, if this batch has one
                state["depth"] = autotune.plan_for(planned)
                planned = _plan(state)
            state["tune"] = autotune.for_jobs(planned) or None
            state["ws"] = torch.empty(nz.nz_batch_workspace_bytes(planned, state["tune"]), dtype=torch.uint8,
                                      device="cuda")
        return state
    if kind == "pmax":
        return dict(kind=kind, L=int(case["L"]), mask=int(case["masks"]), samples=int(case["samples"]),
                    seed=0xF55 + 4096 * int(seed), boundary=int(case["boundary"]),
                    p=np.arange(P_LO, P_HI + P_STEP / 2, P_STEP))
    if kind == "train":
        d = _train_inputs(case, seed)
        n = nz.NZ_MLP_NPARAM
        rows = int(case["rows"])
        dev = lambda a: torch.from_numpy(a).cuda()  # noqa: E731
        empty = lambda *s: torch.empty(s, dtype=torch.float32, device="cuda")  # noqa: E731
        return dict(kind=kind, x=dev(d["x"]), target=dev(d["target"]), weight=dev(d["weight"]), w=dev(d["w"]),
                    wb=dev(learned.to_bf16_bits(d["w"]).view(np.int16)), m=dev(d["m"]), v=dev(d["v"]), g=empty(n),
                    y=empty(rows, 2), act=empty(rows, nz.NZ_MLP_NACT), dy=empty(rows, 2), loss=empty(1),
                    hyper=_HYPER, step=_FIRST_STEP)
    if kind == "canonical":
        hist, p = _histogram(case, seed)
        return dict(kind=kind, hist=hist, p=p)
    raise ValueError(kind)


_HYPER = [3e-3, 0.9, 0.999, 1e-8, 0.0]
_FIRST_STEP = 20


def _train_inputs(case, seed):
    """A state some steps into training: the lattices' features, targets near
    the threshold fit, Glorot weights, Adam moments of gradients of this size."""
    rng = np.random.default_rng(int(seed))
    rows = int(case["rows"])
    masks = rng.integers(1, 128, size=rows).astype(np.uint32)
    Ls = rng.choice([4, 8, 10, 12, 16, 20], size=rows).astype(np.int32)
    mean, std = nz.nz_mlp_size_stats(Ls)
    z = np.array([_z(int(m)) for m in masks], dtype=np.float64)
    lm = np.log(1.553 / (z + 1.01)) + 0.05 * rng.standard_normal(rows)
    ls = lm - 3.0 + 0.1 * rng.standard_normal(rows)
    n = nz.NZ_MLP_NPARAM
    return dict(x=nz.nz_mlp_features(masks, Ls, mean, std), target=np.stack([lm, ls], 1).astype(np.float32),
                weight=np.sqrt(rng.choice([500.0, 1000.0, 10000.0], size=rows)).astype(np.float32),
                w=learned.init_params(int(seed)), m=(0.01 * rng.standard_normal(n)).astype(np.float32),
                v=(1e-4 * rng.random(n) + 1e-8).astype(np.float32))


def _histogram(case, seed):
    """n* histogram of a zone-1 run (spread a few percent of the mean) and a
    uniform p grid."""
    rng = np.random.default_rng(int(seed))
    N = int(case["L"]) ** 5
    ns = np.clip(np.rint((0.145 + 0.004 * rng.standard_normal(int(case["samples"]))) * N), 1, N).astype(np.int64)
    return np.bincount(ns, minlength=N + 1).astype(np.uint64), np.linspace(0.0, 1.0, int(case["points"]))


def run(state):
    kind = state["kind"]
    if kind == "sweep":
        return nz.nz_sweep(state["L"], state["mask"], state["samples"], state["seed"], boundary=state["boundary"])
    if kind == "batch":
        back = nz.nz_sweep_batch(_plan(state), state["ws"], state["nstar"], state["mass"], tune=state["tune"])
        return dict(nstar=state["nstar"], mass=state["mass"], backoffs=back)
    if kind == "static":
        back = nz.nz_sweep_batch_static(_plan(state), state["nstar"], state["mass"])
        return dict(nstar=state["nstar"], mass=state["mass"], backoffs=back)
    if kind == "pmax":
        P, cover, _ = fss.pmax_curve(state["L"], state["mask"], state["seed"], state["samples"], state["p"],
                                     boundary=state["boundary"])
        return dict(P=P, cover=cover)
    if kind == "train":
        s = state
        nz.nz_mlp_forward(s["wb"], s["x"], s["y"], s["act"])
        nz.nz_mlp_loss(s["y"], s["target"], s["weight"], s["dy"], s["loss"])
        nz.nz_mlp_backward(s["wb"], s["x"], s["act"], s["dy"], s["g"])
        nz.nz_mlp_adam(s["w"], s["wb"], s["g"], s["m"], s["v"], s["hyper"], s["step"])
        s["step"] += 1
        return dict(y=s["y"], act=s["act"], loss=s["loss"], dy=s["dy"], grad=s["g"], w=s["w"],
                    w_bf16=s["wb"].view(torch.bfloat16), m=s["m"], v=s["v"])
    return dict(R=nz.nz_canonical(state["hist"], state["p"]))


def _z(mask):
    return sum(s for k, s in enumerate(ZONE_SIZES) if mask >> k & 1)


def work(case):
    """What a pass cannot do without.  A sample: every site's key (ten Philox
    rounds of two products and two three-way XORs for each pair of sites), half
    of the neighbour checks of the sites up to the threshold (a load's worth of
    address and bit arithmetic each: 2), the occupancy bitset, one order entry
    and one union-find entry of every site up to the threshold, and the two
    results.  Operations of the sweeps are integer ones."""
    kind = case["kind"]
    if kind == "train":
        rows, n = int(case["rows"]), nz.NZ_MLP_NPARAM
        return dict(bytes=rows * 4.0 * (8 + 2 + 1 + 2 + 2 + 128) + n * (4.0 * 7 + 2), flops=6.0 * rows * n + 12.0 * n)
    if kind == "canonical":
        N, points = int(case["L"]) ** 5, int(case["points"])
        # the binomial weights within 9 standard deviations of every p
        terms = sum(min(N, 18.0 * math.sqrt(N * p * (1 - p))) for p in np.linspace(0, 1, points))
        return dict(bytes=8.0 * N + 16.0 * points, flops=5.0 * terms + N)
    total = dict(bytes=0.0, flops=0.0)
    for L in _ints(case["L"]):
        N = float(L**5)
        for m in _ints(case["masks"]):
            z = _z(m)
            f = min(1.0, (P_HI if kind == "pmax" else 1.553 / (z + 1.01)))
            S = int(case["samples"])
            total["bytes"] += S * (N / 8 + f * N * 8 + 8)
            total["flops"] += S * (20 * N + f * N * z)
    return total


def exact(case, seed):
    """Outputs in 64 bits by plain numpy: the training step and the canonical
    convolution (n*, masses and window sums are integers)."""
    if case["kind"] == "canonical":
        hist, p = _histogram(case, seed)
        F = np.cumsum(hist, dtype=np.uint64).astype(np.longdouble) / np.longdouble(hist.sum())
        N = len(hist) - 1
        return dict(R=np.array([_convolve(F, N, float(q)) for q in p], dtype=np.float64))
    if case["kind"] != "train":
        return None
    d = _train_inputs(case, seed)
    rows = int(case["rows"])
    f64 = lambda a: np.asarray(a, dtype=np.float64)  # noqa: E731
    bits = learned.to_bf16_bits(d["w"]).astype(np.uint32) << 16
    p = f64(bits.view(np.float32))
    W1, b1, W2, b2, W3, b3 = (p[a:b].reshape(s) for a, b, s in _layout())
    x, t, wt = f64(d["x"]), f64(d["target"]), f64(d["weight"])
    h1 = np.tanh(x @ W1 + b1)
    h2 = np.tanh(h1 @ W2 + b2)
    y = h2 @ W3 + b3
    wn = (wt / wt.sum())[:, None]
    dy = 2 * wn * (y - t)
    dz2 = (dy @ W3.T) * (1 - h2 * h2)
    dz1 = (dz2 @ W2.T) * (1 - h1 * h1)
    g = np.concatenate([a.reshape(-1) for a in (x.T @ dz1, dz1.sum(0), h1.T @ dz2, dz2.sum(0), h2.T @ dy, dy.sum(0))])
    lr, b1_, b2_, eps, wd = f64(np.array(_HYPER, dtype=np.float32))
    m = b1_ * f64(d["m"]) + (1 - b1_) * g
    v = b2_ * f64(d["v"]) + (1 - b2_) * g * g
    mh, vh = m / (1 - b1_**_FIRST_STEP), v / (1 - b2_**_FIRST_STEP)
    w = f64(d["w"]) - lr * (mh / (np.sqrt(vh) + eps) + wd * f64(d["w"]))
    return dict(y=y, act=np.concatenate([h1, h2], 1).reshape(rows, -1), loss=np.array([(wn * (y - t) ** 2).sum()]),
                dy=dy, grad=g, w=w, w_bf16=w, m=m, v=v)


def _layout():
    at, out = 0, []
    for shape in ((8, 64), (64,), (64, 64), (64,), (64, 2), (2,)):
        n = math.prod(shape)
        out.append((at, at + n, shape))
        at += n
    return out


def _convolve(F, N, p):
    """sum_n C(N, n) p^n (1 - p)^(N - n) F[n], weights from the mode outward in
    extended precision."""
    if p <= 0.0 or p >= 1.0:
        return float(F[0] if p <= 0.0 else F[N])
    mode = min(N, int(math.floor((N + 1) * p)))
    half = int(40 * math.sqrt(N * p * (1 - p))) + 60
    lo, hi = max(0, mode - half), min(N, mode + half)
    pl = np.longdouble(p)
    up = pl / (1 - pl)
    n = np.arange(mode, hi, dtype=np.int64).astype(np.longdouble)
    right = np.cumprod((N - n) / (n + 1) * up)
    n = np.arange(mode, lo, -1, dtype=np.int64).astype(np.longdouble)
    left = np.cumprod(n / (N - n + 1) / up)
    w = np.concatenate([left[::-1], [np.longdouble(1)], right])
    return float((w * F[lo:hi + 1]).sum() / w.sum())
