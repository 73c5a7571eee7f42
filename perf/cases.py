"""The work that a program using this library has it do, as measurable cases.

Five kinds of work, each through the package's public entry points:

  resample  one filter: RESAMPLE(x, w) by Megopolis, Metropolis, C1 or C2,
            with B from the bias bound, and the particle copy either fused
            ("fused"), a separate gather ("separate") or left out ("none");
  prefix    one filter by multinomial or systematic resampling;
  batch     many uneven filters in one graph launch;
  sir       the SIR filter of many runs, T steps per pass;
  serve     a burst of requests through the continuous-batching server.

Weights are the Gaussian-likelihood weights of the package's own experiments:
x ~ N(0, 1), w = exp(-(x - y)^2 / 2), y from 0 (mild) to 4 (degenerate).
"""
import math

import numpy as np
import torch

from paper_2109_13504_amd import inputs, mgp

EPS = 0.01        # bias bound of the resampling experiments
SIR_EPS = 0.1     # bias bound of the SIR experiments
N_MAX = 1 << 24   # the benchmark's largest filter


# ---------------------------------------------------------------------------
# The cases
# ---------------------------------------------------------------------------

def listed():
    return [
        # the smallest useful filter, ancestors only: launch latency and host path
        {"name": "mego_1k", "kind": "resample", "variant": "megopolis", "n": 1000, "y": 2.0, "d": 0, "copy": "none",
         "segment": 32},
        # a ragged mid-size filter with degenerate weights (B about 355) and rows of three floats
        {"name": "mego_20k_y4_d3", "kind": "resample", "variant": "megopolis", "n": 20011, "y": 4.0, "d": 3,
         "copy": "fused", "segment": 32},
        # an odd size above the small-filter paths, the copy as a call of its own, rows of five floats
        {"name": "mego_100k_y1_d5", "kind": "resample", "variant": "megopolis", "n": 100003, "y": 1.0, "d": 5,
         "copy": "separate", "segment": 32},
        # the ordinary filter: 2^20 particles, moderate weights (B = 16), rows of four floats
        {"name": "mego_1m_y2_d4", "kind": "resample", "variant": "megopolis", "n": 1 << 20, "y": 2.0, "d": 4,
         "copy": "fused", "segment": 32},
        # the headline filter: 2^24 particles, B = 354, rows of eight floats
        {"name": "mego_16m_y4_d8", "kind": "resample", "variant": "megopolis", "n": 1 << 24, "y": 4.0, "d": 8,
         "copy": "fused", "segment": 32},
        # the comparison resamplers of the same experiments
        {"name": "metropolis_1m_y2", "kind": "resample", "variant": "metropolis", "n": 1 << 20, "y": 2.0, "d": 0,
         "copy": "none", "segment": 32},
        {"name": "c2_4m_y3", "kind": "resample", "variant": "c2", "n": 1 << 22, "y": 3.0, "d": 0, "copy": "none",
         "segment": 32},
        # the unbiased methods: an ordinary filter, and a large one of a size that is no power of two
        {"name": "multinomial_1m_y2", "kind": "prefix", "method": "multinomial", "n": 1 << 20, "y": 2.0},
        {"name": "systematic_10m_y1", "kind": "prefix", "method": "systematic", "n": 10000000, "y": 1.0},
        # 512 uneven filters of 2^10 to 2^18 particles with their copies, one graph launch
        {"name": "batch_512", "kind": "batch", "count": 512, "lo": 10.0, "hi": 18.0, "d": 4, "mix": 777},
        # the SIR experiment: 64 runs of 2^20 particles, ten steps
        {"name": "sir_64x1m", "kind": "sir", "variant": "megopolis", "runs": 64, "n": 1 << 20, "steps": 10, "B": 16},
        # a burst of mixed requests at the server
        {"name": "serve_24", "kind": "serve", "count": 24, "lo": 12.0, "hi": 20.0, "d": 8, "mix": 999},
    ]


def _size(rng, lo, hi):
    """A size between lo and hi, spread over its logarithm; a third are powers of two, the rest as they fall."""
    n = int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))
    if rng.random() < 1.0 / 3.0:
        n = 1 << int(round(math.log2(n)))
    return max(lo, min(hi, n))


def draw(rng):
    kind = rng.choices(["megopolis", "other", "prefix", "batch", "sir", "serve"], [8, 4, 3, 2, 2, 1])[0]
    y = round(rng.uniform(0.0, 4.0), 2)
    if kind == "megopolis":
        d = rng.choice([0, 1, 2, 3, 4, 5, 8, 8, 16])
        n = _size(rng, 500, N_MAX >> (1 if d > 8 else 0))
        return {"kind": "resample", "variant": "megopolis", "n": n, "y": y, "d": d,
                "copy": rng.choice(["fused", "fused", "separate"]) if d else "none",
                "segment": 64 if rng.random() < 0.15 else 32}
    if kind == "other":
        d = rng.choice([0, 0, 1, 4, 8])
        return {"kind": "resample", "variant": rng.choice(["metropolis", "c1", "c2"]), "n": _size(rng, 500, 1 << 22),
                "y": round(rng.uniform(0.0, 3.0), 2), "d": d, "copy": rng.choice(["fused", "separate"]) if d else "none",
                "segment": 32}
    if kind == "prefix":
        return {"kind": "prefix", "method": rng.choice(["multinomial", "systematic"]), "n": _size(rng, 500, N_MAX),
                "y": y}
    if kind == "batch":
        lo = rng.uniform(8.0, 12.0)
        return {"kind": "batch", "count": rng.randint(16, 640), "lo": round(lo, 2), "hi": round(lo + rng.uniform(1.0, 6.0), 2),
                "d": rng.choice([0, 3, 4, 8]), "mix": rng.randint(1, 9999)}
    if kind == "sir":
        runs = _size(rng, 1, 64)
        n = _size(rng, 1 << 10, 1 << 20)
        steps = 1 if rng.random() < 0.5 else rng.randint(2, 10)
        return {"kind": "sir", "variant": rng.choice(["megopolis", "megopolis", "c2", "multinomial", "systematic"]),
                "runs": runs, "n": n, "steps": min(steps, 3) if runs * n > 1 << 25 else steps,
                "B": rng.choice([0, 16, 16, 32])}
    lo = rng.uniform(10.0, 14.0)
    return {"kind": "serve", "count": rng.randint(4, 32), "lo": round(lo, 2), "hi": round(lo + rng.uniform(2.0, 6.0), 2),
            "d": rng.choice([0, 4, 8]), "mix": rng.randint(1, 9999)}


# ---------------------------------------------------------------------------
# Inputs
# ---------------------------------------------------------------------------

def _gen(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(1000003 * int(seed) + 17)
    return g


def _likelihood(x, y):
    return torch.exp(-0.5 * (x - y) ** 2)


def _weights(n, y, g):
    """x ~ N(0, 1) and the fp32 weights of y."""
    x = torch.randn(n, generator=g, device="cuda", dtype=torch.float32)
    return x, _likelihood(x, y)


def _states(x, d, g):
    st = torch.randn((x.numel(), d), generator=g, device="cuda", dtype=torch.float32)
    st[:, 0] = x
    return st


def _round_up(n, k):
    return (n + k - 1) // k * k


def _uneven(case):
    """Sizes, y and starts (in one buffer, each filter 512-byte aligned) of a batch's or a burst's filters: the mix
    belongs to the case, the particles to the seed."""
    rng = np.random.Generator(np.random.PCG64(case["mix"]))
    n = np.rint(2.0 ** rng.uniform(case["lo"], case["hi"], case["count"])).astype(np.int64)
    y = rng.uniform(0.0, 4.0, case["count"])
    starts = np.concatenate([[0], np.cumsum((n + 127) // 128 * 128)])
    return n, y, starts


def _many(case, seed):
    """The filters of a batch or burst: slices of one weight, ancestor, state and output buffer."""
    g = _gen(seed)
    n, y, starts = _uneven(case)
    total, d = int(starts[-1]), case["d"]
    x = torch.randn(total, generator=g, device="cuda", dtype=torch.float32)
    yy = torch.from_numpy(np.repeat(y, np.diff(starts)).astype(np.float32)).cuda()
    w = _likelihood(x, yy)
    st = _states(x, d, g) if d else None
    anc = torch.zeros(total, dtype=torch.int32, device="cuda")
    out = torch.zeros((total, d), dtype=torch.float32, device="cuda") if d else None
    cuts = [slice(int(a), int(a) + int(k)) for a, k in zip(starts, n)]
    return n, cuts, w, st, anc, out


def _sir_x0(case, seed):
    x = torch.randn((case["runs"], case["n"]), generator=_gen(seed), device="cuda", dtype=torch.float32)
    return x.mul_(math.sqrt(5.0))


def _sir_z(case, seed):
    """Measurements: four runs to a trajectory of the model."""
    _, z = inputs.sir_truth(case["steps"], (case["runs"] + 3) // 4, seed=2021 + int(seed))
    return np.repeat(z, 4, axis=0)[: case["runs"]]


def prepare(case, seed):
    kind = case["kind"]
    s = {"case": case, "seed": 7 + 13 * int(seed)}
    if kind == "resample":
        g = _gen(seed)
        x, s["w"] = _weights(case["n"], case["y"], g)
        s["states"] = _states(x, case["d"], g) if case["d"] else None
        s["r"] = mgp.Resampler(case["n"])
        s["sums"] = s["r"].stats.view(torch.float64)[:3]
    elif kind == "prefix":
        _, s["w"] = _weights(case["n"], case["y"], _gen(seed))
        s["r"] = mgp.PrefixResampler(case["n"])
        s["sums"] = s["r"].stats.view(torch.float64)[:2]
    elif kind == "batch":
        n, cuts, w, st, s["anc"], s["out"] = _many(case, seed)
        filters = [{"w": w[c], "anc": s["anc"][c], "epsilon": EPS, "seed": s["seed"] + f, "stream_id": f,
                    "states": st[c] if case["d"] else None, "out": s["out"][c] if case["d"] else None}
                   for f, c in enumerate(cuts)]
        s["plan"] = mgp.BatchPlan(filters, "megopolis", d=case["d"])
    elif kind == "sir":
        s["x0"] = _sir_x0(case, seed)
        s["f"] = mgp.SirFilter(case["runs"], case["n"], case["steps"], case["variant"], B=case["B"], epsilon=SIR_EPS,
                               seed=s["seed"])
        s["f"].set_measurements(_sir_z(case, seed))
    else:
        s["n"], s["cuts"], s["w"], s["states"], s["anc"], s["out"] = _many(case, seed)
        s["server"] = mgp.Server("megopolis", d=case["d"], hbm_budget=1 << 30, streams=4, max_batch=8,
                                 max_batch_particles=1 << 22)
    return s


# ---------------------------------------------------------------------------
# One pass
# ---------------------------------------------------------------------------

def run(s):
    case, kind = s["case"], s["case"]["kind"]
    if kind == "resample":
        r, w = s["r"], s["w"]
        if case["copy"] == "fused":
            out, anc = r.resample_gather(w, s["states"], case["variant"], epsilon=EPS, seed=s["seed"],
                                         segment=case["segment"])
            return {"anc": anc, "out": out, "sums": s["sums"]}
        anc = r.resample(w, case["variant"], epsilon=EPS, seed=s["seed"], segment=case["segment"])
        if case["copy"] == "separate":
            return {"anc": anc, "out": mgp.gather(s["states"], anc), "sums": s["sums"]}
        return {"anc": anc, "sums": s["sums"]}
    if kind == "prefix":
        return {"anc": s["r"].resample(s["w"], case["method"], seed=s["seed"]), "sums": s["sums"]}
    if kind == "batch":
        s["plan"].run()
        return {"anc": s["anc"], "out": s["out"]} if case["d"] else {"anc": s["anc"]}
    if kind == "sir":
        f = s["f"]
        f.reset(s["x0"])
        f.run()
        est, B, status = f.results()
        got = {"est": est, "B": B, "status": status, "xbar": f.copy("xbar")}
        if case["steps"] == 1:  # a program that steps the filter by hand looks at the particles and weights too
            got.update(x=f.copy("x"), w=f.copy("w"), anc=f.copy("ancestors"))
        return got
    # serve: submit the burst, wait for every request, take the outputs, give the memory back
    server, stream = s["server"], torch.cuda.current_stream()
    tickets = [server.submit(s["w"][c], epsilon=EPS, seed=s["seed"] + f, stream_id=f,
                             states=s["states"][c] if case["d"] else None) for f, c in enumerate(s["cuts"])]
    for t, c in zip(tickets, s["cuts"]):
        server.wait(t)
        mgp.mgp_server_copy_outputs(server.handle, t, s["anc"][c].data_ptr(),
                                    s["out"][c].data_ptr() if case["d"] else 0, stream.cuda_stream)
    stream.synchronize()
    for t in tickets:
        server.release(t)
    return {"anc": s["anc"], "out": s["out"]} if case["d"] else {"anc": s["anc"]}


# ---------------------------------------------------------------------------
# What a pass cannot do without
# ---------------------------------------------------------------------------

def _steps(y, eps=EPS):
    """B of the bias bound for Gaussian-likelihood weights: mean exp(-y^2/4)/sqrt(2), maximum 1."""
    return max(1.0, math.ceil(math.log(eps) / math.log1p(-math.exp(-0.25 * y * y) / math.sqrt(2.0))))


def work(case):
    """Bytes: each weight, state row and initial particle read once, each output written once. Operations: a product
    and a comparison per particle and step; for the prefix methods an addition per weight and a binary search per
    output; for the SIR model about 60 per particle and step besides."""
    kind = case["kind"]
    if kind == "resample":
        n, d = case["n"], case["d"]
        return {"bytes": n * (8.0 + 8.0 * d), "flops": 2.0 * n * _steps(case["y"])}
    if kind == "prefix":
        n = case["n"]
        return {"bytes": 8.0 * n, "flops": n * (1.0 + (math.log2(n) if case["method"] == "multinomial" else 1.0))}
    if kind == "sir":
        p = float(case["runs"]) * case["n"]
        B = case["B"] or 28
        B = {"multinomial": 10, "systematic": 1}.get(case["variant"], B)
        return {"bytes": 8.0 * p, "flops": p * case["steps"] * (60.0 + 2.0 * B)}
    n, y, _ = _uneven(case)
    return {"bytes": float(n.sum()) * (8.0 + 8.0 * case["d"]), "flops": float(sum(2.0 * k * _steps(v) for k, v in zip(n, y)))}


# ---------------------------------------------------------------------------
# The computed numbers in 64 bits (ancestors, and rows copied by them, are whole numbers and copies: None)
# ---------------------------------------------------------------------------

def _philox(c0, c1, c2, c3, k0, k1):
    """Philox4x32-10 on arrays of uint64 counter words."""
    m = np.uint64(0xFFFFFFFF)
    c0, c1, c2, c3 = (np.asarray(c, dtype=np.uint64) for c in (c0, c1, c2, c3))
    for _ in range(10):
        p0, p1 = np.uint64(0xD2511F53) * c0, np.uint64(0xCD9E8D57) * c2
        c0, c1, c2, c3 = ((p1 >> np.uint64(32)) ^ c1 ^ np.uint64(k0), p1 & m,
                          (p0 >> np.uint64(32)) ^ c3 ^ np.uint64(k1), p0 & m)
        k0, k1 = (k0 + 0x9E3779B9) & 0xFFFFFFFF, (k1 + 0xBB67AE85) & 0xFFFFFFFF
    return c0, c1, c2, c3


def _sir_step(case, seed):
    """Step 1 of the model for every run: x_1, and the likelihood of x_1 as stored in 32 bits."""
    runs, n, key = case["runs"], case["n"], 7 + 13 * int(seed)
    x0, z = _sir_x0(case, seed).cpu().numpy().astype(np.float64), _sir_z(case, seed)
    x, w = np.empty((runs, n)), np.empty((runs, n))
    quads = np.arange((n + 3) // 4)
    for r in range(runs):
        a = _philox(np.full(quads.size, 1), np.full(quads.size, 5), np.full(quads.size, r), quads, key & 0xFFFFFFFF,
                    key >> 32)
        a = [v.astype(np.float64) for v in a]
        noise = np.empty((quads.size, 4))
        for k in (0, 2):
            radius, angle = np.sqrt(-2.0 * np.log((a[k] + 1.0) * 2.0 ** -32)), 2.0 * np.pi * (a[k + 1] * 2.0 ** -32)
            noise[:, k], noise[:, k + 1] = radius * np.cos(angle), radius * np.sin(angle)
        p = x0[r]
        x[r] = p / 2.0 + 25.0 * p / (1.0 + p * p) + 8.0 * math.cos(1.2) + math.sqrt(10.0) * noise.reshape(-1)[:n]
        stored = x[r].astype(np.float32).astype(np.float64)
        w[r] = np.exp(-0.5 * (z[r, 1] - stored * stored / 20.0) ** 2)
    return x, w


def exact(case, seed):
    kind = case["kind"]
    if kind in ("resample", "prefix"):
        w = _weights(case["n"], case["y"], _gen(seed))[1].double()
        total = w.sum().item()
        ratio = total / case["n"] / w.max().item()
        if kind == "prefix":
            return {"anc": None, "sums": np.array([total, ratio])}
        sums = np.array([total, ratio, math.log(EPS) / math.log1p(-ratio)])
        return {"anc": None, "out": None, "sums": sums} if case["copy"] != "none" else {"anc": None, "sums": sums}
    if kind == "sir" and case["steps"] == 1 and case["runs"] * case["n"] <= 1 << 22:
        x, w = _sir_step(case, seed)
        return {"est": None, "B": None, "status": None, "xbar": None, "x": x, "w": w, "anc": None}
    return None
