"""Workloads that a user of the detector runs, for timing one version of the
library against another.

A case is one pass through the public entry points of
paper_1803_11449_amd.ddhf, by kind:

  window   one window of one link: reset, the window's pairs in `calls`
           updates, restore at theta (or restore_noalloc)
  links    several links' windows that close together: resets, one batched
           update, one batched restore
  plan     the same cycle as a captured plan: one run, one results call
  merge    two monitors' halves of a window, each in its own sketch, merged
           (router merge) and restored
  sweep    a stored sketch (a loaded snapshot) restored at several thresholds

Traffic is the repository's synthetic windows (traffic.py): Zipf sources,
uniform destinations, planted super points. Sketch shapes follow the sizing
rule: the smallest k >= 14 with n / (g 2^k) <= 0.45 and
alpha = ceil((32 - k) / (r - 2)).
"""
import math

import numpy as np
import torch

from paper_1803_11449_amd import ddhf, traffic

DEVICE = "cuda:0"
LOAD = 0.45


def _shape(n, g, r):
    """(k, alpha) of the sizing rule for an n-pair window (r = 3 needs
    k >= 16 to cover the 32 address bits)."""
    k = 16 if r == 3 else 14
    while n / (g * 2 ** k) > LOAD:
        k += 1
    return k, math.ceil((32 - k) / (r - 2))


def _window(name, n, **more):
    """A window case with the defaults of the paper's sketch."""
    return {"kind": "window", "name": name, "n": n, "calls": 1, "theta": 1024.0, "zipf": 1.0,
            "planted": 0, "g": 1024, "r": 5, "noalloc": False, **more}


def listed():
    return [
        # a quiet link polled often: one small capture buffer, then the list
        _window("window_3k", 3_001, theta=512.0, zipf=1.3),
        # a slow link's window, just past the size where updates get batched
        # into passes; a host that may not allocate while it runs
        _window("window_60k", 60_013, theta=512.0, zipf=1.2, noalloc=True),
        # the 1M-pair window on the paper's default sketch
        _window("window_1m", 1_000_000, zipf=1.1, planted=20),
        # a window that arrives in capture buffers of 16,667 pairs
        _window("buffers_1m", 1_000_003, calls=60, zipf=1.1, planted=20),
        # a 10 Gb/s link, low threshold, flat traffic: many near-threshold hosts
        _window("window_9m_theta512", 8_999_999, theta=512.0, zipf=0.9, planted=200),
        # a shorter hash group with smaller estimators (accuracy study shapes)
        _window("window_4m_g512_r4", 4_000_037, theta=700.0, zipf=1.1, planted=50, g=512, r=4),
        # the 100M-pair window of a core link
        _window("window_100m", 100_000_000, planted=500),
        # the largest link of a batch: a 320 MiB sketch
        _window("window_190m", 189_999_991, zipf=1.1, planted=500),
        # links of uneven size whose windows close together
        {"kind": "links", "name": "links_12", "links": 12, "lo": 100_000, "hi": 20_000_000,
         "theta": 1024.0, "g": 1024, "r": 5},
        # a fixed set of links, each with its own staging buffer, every period
        {"kind": "plan", "name": "plan_12", "links": 12, "lo": 300_000, "hi": 50_000_000,
         "theta": 512.0, "g": 1024, "r": 5},
        # two routers see one network's traffic
        {"kind": "merge", "name": "merge_30m", "n": 30_000_001, "theta": 1024.0, "zipf": 1.0,
         "planted": 200, "g": 1024, "r": 5},
        # an analyst tries thresholds on a stored window
        {"kind": "sweep", "name": "sweep_60m", "n": 60_000_000, "thetas": "512 1024 2048",
         "zipf": 0.9, "planted": 200, "g": 1024, "r": 5},
    ]


def _log(rng, lo, hi):
    return int(math.exp(rng.uniform(math.log(lo), math.log(hi))))


def draw(rng):
    kind = rng.choice(["window"] * 7 + ["links", "plan", "merge", "sweep"])
    r = rng.choice([5, 5, 5, 4, 6])
    g = rng.choice([1024, 1024, 512, 2048]) if r == 5 else rng.choice([512, 1024])
    theta = round(g * rng.choice([0.6, 0.75, 1.0, 1.3]) + rng.uniform(0, 20), 3)
    zipf = round(rng.uniform(0.8, 1.3), 2)
    if kind == "window":
        n = _log(rng, 2_000, 190_000_000) | 1
        return {"kind": kind, "n": n, "calls": rng.choice([1, 1, 1, 2, 7, 40]), "theta": theta,
                "zipf": zipf, "planted": min(500, n // 8000), "g": g, "r": r,
                "noalloc": rng.random() < 0.2}
    if kind in ("links", "plan"):
        lo = _log(rng, 50_000, 2_000_000)
        return {"kind": kind, "links": rng.randint(3, 12), "lo": lo, "hi": lo * rng.randint(2, 20),
                "theta": theta, "g": 1024, "r": 5}
    n = _log(rng, 200_000, 60_000_000) | 1
    case = {"kind": kind, "n": n, "zipf": zipf, "planted": min(300, n // 8000), "g": g, "r": r}
    if kind == "merge":
        return {**case, "theta": theta}
    return {**case, "thetas": " ".join(str(round(g * x, 2)) for x in (0.61, 1.03, 1.97))}


# ------------------------------------------------------------------- inputs

def _spec(n, zipf, planted, key):
    """One link's window; a window below 100k pairs has no room for a
    planted source of up to 50,000 destinations."""
    if planted and n >= 100_000:
        return traffic.spec_link_window(n, zipf, planted, key)
    return traffic.WindowSpec(n_pairs=n, n_sources=max(1000, n // 25), zipf_s=zipf,
                              planted_card=[])


def _pairs(n, zipf, planted, seed):
    """int32 [n, 2] (src, dst) on the GPU, from the seed alone."""
    return traffic.generate(_spec(n, zipf, planted, seed + 77), seed, device=DEVICE).pairs


def _thetas(case):
    return [float(t) for t in case["thetas"].split()] if "thetas" in case else [case["theta"]]


def _links(case, seed):
    """Per link: (pairs in its window, zipf exponent, planted sources). The
    sizes are spread over the case's range; the traffic is the seed's."""
    u = np.random.default_rng(seed).uniform(size=case["links"])
    sizes = [int(case["lo"] * (case["hi"] / case["lo"]) ** ((i + 0.5) / case["links"])) | 1
             for i in range(case["links"])]
    return [(n, 0.8 + 0.5 * float(x), max(1, min(300, n // 8000))) for n, x in zip(sizes, u)]


def _inputs(case, seed):
    """The case's windows: a list of (pairs tensor, k, alpha)."""
    g, r = case["g"], case["r"]
    if case["kind"] in ("links", "plan"):
        return [(_pairs(n, z, p, seed * 64 + i), *_shape(n, g, r))
                for i, (n, z, p) in enumerate(_links(case, seed))]
    return [(_pairs(case["n"], case["zipf"], case["planted"], seed), *_shape(case["n"], g, r))]


def _split(pairs, parts):
    """Consecutive buffers of about equal length (views)."""
    step = -(-pairs.shape[0] // parts)
    return [pairs[i:i + step] for i in range(0, pairs.shape[0], step)]


def _sketch(case, k, alpha):
    return ddhf.Sketch(case["g"], k, case["r"], alpha, traffic.HASH_SEED, device=0)


def prepare(case, seed):
    wins = _inputs(case, seed)
    state = {"case": case, "kind": case["kind"],
             "sketches": [_sketch(case, k, a) for _, k, a in wins],
             "reports": [Report(_rows(p.shape[0], t)) for p, _, _ in wins for t in _thetas(case)]}
    if case["kind"] == "window":
        state["buffers"] = _split(wins[0][0], case["calls"])
    elif case["kind"] == "merge":
        state["sketches"].append(_sketch(case, *wins[0][1:]))
        state["buffers"] = _split(wins[0][0], 2)
    elif case["kind"] == "sweep":
        # the sketch as a snapshot of it is loaded: its words uploaded
        sk = state["sketches"][0]
        sk.update(wins[0][0])
        sk.upload(sk.download())
        state["thetas"] = _thetas(case)
    else:
        state["buffers"] = [p for p, _, _ in wins]
        if case["kind"] == "plan":
            state["plan"] = ddhf.Plan([(sk, p, case["theta"]) for sk, p in
                                       zip(state["sketches"], state["buffers"])])
    return state


# --------------------------------------------------------------------- pass

class Report:
    """A link's report table, kept by the program: the list's columns from
    row 0, zeros below, and the window's counts and scalars."""

    def __init__(self, rows):
        self.ip = np.zeros(rows, dtype=np.uint32)
        self.sz = np.zeros(rows, dtype=np.uint32)
        self.est = np.zeros(rows, dtype=np.float64)
        self.used = 0

    def fill(self, recs, info):
        n = len(recs)
        for name in ("ip", "sz", "est"):
            col = getattr(self, name)
            col[:n] = recs[name]
            col[n:self.used] = 0
        self.used = n
        return {"ip": self.ip, "sz": self.sz, "est": self.est,
                "counts": np.array(info["zr"] + info["he_count"] +
                                   [info["n_candidates"], info["n_reported"]], dtype=np.int64),
                "scalars": np.array([info["psi"], info["d"], info["trep"]])}


def _rows(n, theta):
    """Report rows: more than the hosts that can reach theta in n pairs."""
    return 64 + int(1.5 * n / theta)


def run(state):
    kind, sks, reports = state["kind"], state["sketches"], state["reports"]
    theta = state["case"].get("theta")
    if kind == "window":
        sk = sks[0]
        sk.reset()
        for b in state["buffers"]:
            sk.update(b)
        return reports[0].fill(*(sk.restore_noalloc(theta) if state["case"]["noalloc"]
                                 else sk.restore(theta)))
    if kind == "links":
        for sk in sks:
            sk.reset()
        ddhf.update_batch(list(zip(sks, state["buffers"])))
        lists = ddhf.restore_batch([(sk, theta) for sk in sks])
        return [t.fill(*x) for t, x in zip(reports, lists)]
    if kind == "plan":
        state["plan"].run()
        return [t.fill(*x) for t, x in zip(reports, state["plan"].results())]
    if kind == "merge":
        for sk, b in zip(sks, state["buffers"]):
            sk.reset()
            sk.update(b)
        sks[0].merge(sks[1])
        return reports[0].fill(*sks[0].restore(theta))
    return [t.fill(*sks[0].restore(th)) for t, th in zip(reports, state["thetas"])]


# --------------------------------------------------------------------- work

def _sketch_bytes(n, g, r):
    return (r << _shape(n, g, r)[0]) * g // 8


def work(case):
    """A window reads its pairs (8 bytes each) and leaves its sketch; a
    stored sketch is read by each restore. The lists themselves are small."""
    g, r = case["g"], case["r"]
    if case["kind"] in ("links", "plan"):
        ns = [n for n, _, _ in _links(case, 0)]
        return {"bytes": sum(8 * n + _sketch_bytes(n, g, r) for n in ns), "flops": 0}
    sk = _sketch_bytes(case["n"], g, r)
    if case["kind"] == "sweep":
        return {"bytes": sk * len(case["thetas"].split()), "flops": 0}
    # a merge leaves two sketches, reads both and writes one of them again
    return {"bytes": 8 * case["n"] + (5 * sk if case["kind"] == "merge" else sk), "flops": 0}


# -------------------------------------------------------------------- exact

def _splitmix(seed, count):
    m = (1 << 64) - 1
    out, s = [], seed
    for _ in range(count):
        s = (s + 0x9E3779B97F4A7C15) & m
        z = s
        z = ((z ^ (z >> 30)) * 0xBF58476D1CE4E5B9) & m
        z = ((z ^ (z >> 27)) * 0x94D049BB133111EB) & m
        out.append(z ^ (z >> 31))
    return out


def _s64(x):
    return x - (1 << 64) if x >> 63 else x


def _hash(mul, add, x, bits):
    """Top `bits` bits of mul * x + add mod 2^64 (int64 tensors wrap)."""
    return ((x * _s64(mul) + _s64(add)) >> (64 - bits)) & ((1 << bits) - 1)


def _cells(a, k, r, alpha, coef):
    """The estimator of each address in each row."""
    c0 = _hash(coef[0], coef[1], a, k)
    m = (1 << k) - 1
    return [c0] + [c0 ^ ((a >> min((i - 1) * alpha, 32)) & m) for i in range(1, r)]


def _exact_window(pairs, k, alpha, case, thetas):
    g, r = case["g"], case["r"]
    c = _splitmix(traffic.HASH_SEED, 4)
    coef = (c[0] | 1, c[1], c[2] | 1, c[3])
    bits = torch.zeros((r, 1 << k, g), dtype=torch.bool, device=pairs.device)
    flat = bits.view(-1)
    for part in torch.split(pairs, 1 << 24):
        p = part.to(torch.int64) & 0xFFFFFFFF
        h = _hash(coef[2], coef[3], p[:, 1], int(math.log2(g)))
        for i, cell in enumerate(_cells(p[:, 0], k, r, alpha, coef)):
            flat[((i << k) + cell) * g + h] = True
    z0 = torch.stack([g - bits[i].sum(-1) for i in range(r)])
    zr = z0.sum(-1).cpu().numpy().astype(np.int64)
    psi = 1.0 - math.exp(sum(math.log(float(z) / (g * 2.0 ** k)) for z in zr) / r)
    d = g * (1.0 - psi ** r)
    outs = []
    for theta in thetas:
        hot = z0 < g * math.exp(-theta / g)
        found = []
        for lo in range(0, 1 << 32, 1 << 26):
            a = torch.arange(lo, lo + (1 << 26), dtype=torch.int64, device=pairs.device)
            a = a[hot[0][_hash(coef[0], coef[1], a, k)]]
            for i in range(1, r):
                a = a[hot[i][_cells(a, k, r, alpha, coef)[i]]]
            found.append(a)
        a = torch.cat(found)
        sz = torch.empty_like(a)
        for j in range(0, len(a), 4096):
            cells = _cells(a[j:j + 4096], k, r, alpha, coef)
            both = bits[0][cells[0]]
            for i in range(1, r):
                both = both & bits[i][cells[i]]
            sz[j:j + 4096] = g - both.sum(-1)
        trep = d * math.exp(-theta / g)
        keep = sz <= math.floor(trep)
        s = sz[keep].cpu().numpy()
        with np.errstate(divide="ignore"):
            est = -float(g) * np.log(s / d)
        he = hot.sum(-1).cpu().numpy().astype(np.int64)
        pad = np.zeros(8 - r, dtype=np.int64)
        table = Report(_rows(pairs.shape[0], theta))
        recs = {"ip": a[keep].cpu().numpy(), "sz": s, "est": est}
        for name, v in recs.items():
            getattr(table, name)[:len(s)] = v
        outs.append({"ip": table.ip, "sz": table.sz, "est": table.est,
                     "counts": np.concatenate([zr, pad, he, pad, [len(a), len(s)]]),
                     "scalars": np.array([psi, d, trep])})
    return outs


def exact(case, seed):
    outs = [o for p, k, a in _inputs(case, seed) for o in _exact_window(p, k, a, case,
                                                                       _thetas(case))]
    return outs if case["kind"] in ("links", "plan", "sweep") else outs[0]
