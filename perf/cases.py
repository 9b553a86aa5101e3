"""Performance cases of the library: the calls that a rescheduler makes, at the
sizes of the repository's workloads and over the ranges around them.

Kinds of case, each one pass through the public entry points of
``paper_2510_13668_amd.star``:

* ``predict``: the binned length head on one decode batch, with the EMA of
  continuous prediction where ``alpha`` > 0.
* ``overlap``: the same head over ``steps`` consecutive decode batches, one
  batch's head beside the next batch's product.
* ``mlp4``: the 4-layer regression head.
* ``schedule``: load projection, migration scores and their ranking.
* ``variance``: load projection, then every migration's exact variance gain.
* ``plan``: Algorithm 1 repeated, from a crowded placement.
"""
import math

import torch

from paper_2510_13668_amd import star

DEV = "cuda"
DTYPES = {"bf16": torch.bfloat16, "f32": torch.float32}
CODES = {"bf16": star.BF16, "f32": star.F32}
ACTS = {"relu": star.ACT_RELU, "gelu": star.ACT_GELU}
LARGEST_FLOPS = 2.0 * 32768 * 8192 * 1024     # first layer of the rebalancing scan


def listed():
    return [
        # the smallest predictor call: the fp32 head of a 64-request cluster
        dict(name="predict_tiny_f32", kind="predict", n_req=64, d=1024, m=256, nb=32, dtype="f32",
             act="relu", alpha=0.0, bias=False, len_max=4096),
        # a ragged batch (odd row count, bins no multiple of 16) of the
        # regression head's hidden width, with biases and smoothing
        dict(name="predict_ragged", kind="predict", n_req=777, d=3584, m=512, nb=50, dtype="bf16",
             act="gelu", alpha=0.2, bias=True, len_max=32768),
        # one decode step of continuous mode: the headline batch
        dict(name="predict_continuous", kind="predict", n_req=1024, d=4096, m=512, nb=64,
             dtype="bf16", act="gelu", alpha=0.2, bias=False, len_max=16384),
        # the long-reasoning batch
        dict(name="predict_long_mix", kind="predict", n_req=4096, d=5120, m=512, nb=64,
             dtype="bf16", act="gelu", alpha=0.0, bias=False, len_max=32768),
        # the largest predictor call: 64 instances x 512 requests
        dict(name="predict_rebalance", kind="predict", n_req=32768, d=8192, m=1024, nb=128,
             dtype="bf16", act="gelu", alpha=0.0, bias=False, len_max=65536),
        # continuous mode as a serving loop runs it: 16 decode steps in a row
        dict(name="overlap_continuous", kind="overlap", steps=16, n_req=1024, d=4096, m=512,
             nb=64, dtype="bf16", act="gelu", alpha=0.2, bias=False, len_max=16384),
        # the regression head on ten requests: a latency figure
        dict(name="mlp4_batch10", kind="mlp4", n_req=10, d=3584, m1=2048, m2=512, m3=64,
             dtype="bf16", alpha=0.0, bias=False, len_max=32768),
        # and on a whole decode batch
        dict(name="mlp4_batch1024", kind="mlp4", n_req=1024, d=3584, m1=2048, m2=512, m3=64,
             dtype="bf16", alpha=0.2, bias=True, len_max=32768),
        # scheduling of the headline batch: curves on-chip
        dict(name="schedule_continuous", kind="schedule", n_req=1024, n_inst=8, bucket=64,
             n_buckets=256, top_k=256, law="lognormal"),
        # the largest scheduling call: 2 M candidates
        dict(name="schedule_rebalance", kind="schedule", n_req=32768, n_inst=64, bucket=64,
             n_buckets=1024, top_k=256, law="pareto"),
        # exact variance gains of the same 2 M candidates
        dict(name="variance_rebalance", kind="variance", n_req=32768, n_inst=64, bucket=64,
             n_buckets=1024, law="pareto"),
        # a plan of up to 16 moves that relieves one crowded instance of 64
        dict(name="plan_rebalance", kind="plan", n_req=32768, n_inst=64, bucket=64,
             n_buckets=1024, moves=16, law="pareto"),
    ]


# ---------------------------------------------------------------------------
# more cases of the same ranges
# ---------------------------------------------------------------------------
def _log(rng, lo, hi):
    """A whole number between lo and hi, spread over its logarithm."""
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def _mult(rng, lo, hi, q):
    """A multiple of q between lo and hi, spread over its logarithm."""
    return q * _log(rng, lo // q, hi // q)


def _draw_head(rng, kind):
    f32 = kind == "predict" and rng.random() < 0.25
    while True:
        # overlapped prediction is a continuous-mode call: batches of a few
        # hundred to a few thousand requests
        n = _log(rng, 128, 4096) if kind == "overlap" else _log(rng, 1, 2048 if f32 else 32768)
        d = _mult(rng, 1024, 4096 if f32 else 8192, 4 if f32 else 8)
        m = _mult(rng, 256, 512 if f32 else 1024, 4 if f32 else 8)
        steps = rng.randint(4, 16) if kind == "overlap" else 1
        if 2.0 * n * d * m * steps <= LARGEST_FLOPS / 2:
            break
    c = dict(kind=kind, n_req=n, d=d, m=m, nb=rng.randint(16, 128),
             dtype="f32" if f32 else "bf16", act=rng.choice(["relu", "gelu", "gelu"]),
             alpha=0.2 if kind == "overlap" else rng.choice([0.0, 0.2]),
             bias=rng.random() < 0.5, len_max=1 << rng.randint(12, 16))
    if kind == "overlap":
        c["steps"] = steps
    return c


def _draw_requests(rng, kind):
    return dict(kind=kind, n_req=_log(rng, 64, 32768), n_inst=_log(rng, 3, 64),
                bucket=rng.choice([1, 16, 64, 100]), n_buckets=_log(rng, 100, 1024),
                law=rng.choice(["lognormal", "mixture", "pareto"]))


def draw(rng):
    kind = rng.choice(["predict", "predict", "predict", "overlap", "mlp4", "schedule", "schedule",
                       "variance", "plan"])
    if kind in ("predict", "overlap"):
        return _draw_head(rng, kind)
    if kind == "mlp4":
        return dict(kind=kind, n_req=_log(rng, 1, 4096), d=_mult(rng, 1024, 4096, 8),
                    m1=_mult(rng, 1024, 2048, 8), m2=_mult(rng, 256, 512, 8),
                    m3=rng.randint(32, 64), dtype="bf16", alpha=rng.choice([0.0, 0.2]),
                    bias=rng.random() < 0.5, len_max=32768)
    c = _draw_requests(rng, kind)
    if kind == "schedule":
        c["top_k"] = rng.choice([0, 16, 100, 256])
    if kind == "plan":
        c["moves"] = rng.randint(4, 16)
    return c


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------
def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    return g


def _normal(g, shape, scale=1.0):
    return torch.randn(shape, generator=g, device=DEV, dtype=torch.float32) * scale


def _uniform(g, n):
    return torch.rand(n, generator=g, device=DEV, dtype=torch.float64)


def _bins(nb, hi):
    """Log-spaced lengths from 1 to hi."""
    k = torch.arange(nb, dtype=torch.float64)
    v = torch.exp(math.log(hi) * k / max(nb - 1, 1))
    return v.to(torch.float32).to(DEV)


def _head_inputs(c, seed):
    """hidden ~ N(0, 1) (an AR(1) chain over decode steps), W ~ N(0, 1/fan_in),
    b ~ N(0, 0.1^2), and the smoothed lengths of the step before."""
    g = _gen(seed)
    dt = DTYPES[c["dtype"]]
    n, d, m, nb = c["n_req"], c["d"], c["m"], c["nb"]
    x = {"w1": _normal(g, (m, d), d ** -0.5).to(dt), "w2": _normal(g, (nb, m), m ** -0.5).to(dt),
         "b1": _normal(g, m, 0.1) if c["bias"] else None,
         "b2": _normal(g, nb, 0.1) if c["bias"] else None, "bins": _bins(nb, c["len_max"]),
         "ema0": torch.exp(_normal(g, n) + 7.0).clamp(1.0, float(c["len_max"]))}
    hidden, h = [], _normal(g, (n, d))
    for s in range(c.get("steps", 1)):
        if s:
            h = 0.95 * h + (1 - 0.95 ** 2) ** 0.5 * _normal(g, (n, d))
        hidden.append(h.to(dt))
    x["hidden"] = hidden
    return x


def _mlp4_inputs(c, seed):
    """W1..W3 ~ N(0, 2/fan_in) for ReLU; w4 and b4 put the outputs at
    remaining lengths of 1100 +- 400 tokens."""
    g = _gen(seed)
    dt = DTYPES[c["dtype"]]
    n, d, m1, m2, m3 = c["n_req"], c["d"], c["m1"], c["m2"], c["m3"]
    return {"hidden": _normal(g, (n, d)).to(dt), "w1": _normal(g, (m1, d), (2 / d) ** 0.5).to(dt),
            "w2": _normal(g, (m2, m1), (2 / m1) ** 0.5).to(dt),
            "w3": _normal(g, (m3, m2), (2 / m2) ** 0.5).to(dt),
            "w4": _normal(g, m3, 400.0 * m3 ** -0.5),
            "b1": _normal(g, m1, 0.1) if c["bias"] else None,
            "b2": _normal(g, m2, 0.1) if c["bias"] else None,
            "b3": _normal(g, m3, 0.1) if c["bias"] else None, "b4": 1100.0,
            "ema0": torch.exp(_normal(g, n) + 7.0).clamp(1.0, float(c["len_max"]))}


def _request_inputs(c, seed):
    """Requests in blocks over the instances; current lengths uniform over
    half the horizon, remaining lengths of the workloads' laws."""
    g = _gen(seed)
    n, ni, H = c["n_req"], c["n_inst"], c["bucket"] * c["n_buckets"]
    cur = 1 + torch.floor(_uniform(g, n) * max(H // 2, 2))
    if c["law"] == "lognormal":
        rem = torch.exp(_normal(g, n).double() + 7.0)
    elif c["law"] == "mixture":
        z, pick = _normal(g, n).double(), _uniform(g, n) < 0.7
        rem = torch.where(pick, torch.exp(6.0 + 0.8 * z), torch.exp(9.0 + 0.5 * z))
    else:
        rem = 64.0 * (1.0 - _uniform(g, n)) ** (-1.0 / 1.5)
    rem = torch.round(rem.clamp(1.0, float(H)))
    inst = (torch.arange(n, device=DEV, dtype=torch.int64) * ni) // n
    if c["kind"] == "plan":     # a quarter of the requests crowded onto one instance
        inst[: n // 4] = ni // 2
    return cur.to(torch.int32), rem.to(torch.int32), inst.to(torch.int32)


def _weights(K):
    """Bucket weights that halve eight times over the horizon (uint16 bits)."""
    w = torch.round(65535.0 * torch.exp2(-8.0 * torch.arange(K, dtype=torch.float64) / K))
    return w.clamp(min=1.0).to(torch.int32).to(torch.int16).to(DEV)


def _empty(shape, dt):
    return torch.zeros(shape, dtype=dt, device=DEV)


def prepare(case, seed):
    c, kind = case, case["kind"]
    s = {"kind": kind}
    if kind in ("predict", "overlap"):
        x = _head_inputs(c, seed)
        n, steps = c["n_req"], c.get("steps", 1)
        p = star.predict_params(n, c["d"], c["m"], c["nb"], CODES[c["dtype"]], ACTS[c["act"]],
                                c["alpha"], False, c["len_max"])
        s.update(x, p=p, steps=steps, n_req=n, ema=x["ema0"].clone() if c["alpha"] else None,
                 expected=list(_empty((steps, n), torch.float32)),
                 rem=list(_empty((steps, n), torch.int32)))
        if kind == "predict":
            s["ws"] = [star.Workspace(star.predict_workspace_size(p))]
        else:
            size = star.predict_overlap_workspace_size(p)
            s["ws"] = [star.Workspace(size), star.Workspace(size)]
        return s
    if kind == "mlp4":
        x = _mlp4_inputs(c, seed)
        p = star.mlp4_params(c["n_req"], c["d"], c["m1"], c["m2"], c["m3"], CODES[c["dtype"]],
                             c["alpha"], False, c["len_max"], x["b4"])
        s.update(x, p=p, ema=x["ema0"].clone() if c["alpha"] else None,
                 expected=_empty(c["n_req"], torch.float32), rem=_empty(c["n_req"], torch.int32),
                 ws=star.Workspace(star.predict_mlp4_workspace_size(p)))
        return s
    n, ni, b, K = c["n_req"], c["n_inst"], c["bucket"], c["n_buckets"]
    cur, rem, inst = _request_inputs(c, seed)
    s.update(cur=cur, rem=rem, inst=inst, load=_empty((ni, K), torch.int64),
             lp=star.load_params(n, ni, b, K))
    if kind == "schedule":
        k = c["top_k"]
        p = star.score_params(n, ni, b, K, k)
        s.update(p=p, scores=_empty((n, ni), torch.int64), bt=_empty(n, torch.int32),
                 bs=_empty(n, torch.int64), tr=_empty(k, torch.int32) if k else None,
                 tt=_empty(k, torch.int32) if k else None,
                 ts=_empty(k, torch.int64) if k else None,
                 ws=star.Workspace(star.project_and_score_workspace_size(p)))
        return s
    s.update(beta=_weights(K), ws_load=star.Workspace(star.project_load_workspace_size(s["lp"])))
    if kind == "variance":
        s.update(gain=_empty((n, ni, 2), torch.int64), bt=_empty(n, torch.int32),
                 bg=_empty((n, 2), torch.int64), move=_empty(star.MOVE_FIELDS, torch.int32),
                 ws=star.Workspace(star.score_variance_workspace_size(s["lp"])))
        return s
    p = star.plan_params(n, ni, b, K, c["moves"], theta=(1, 10), min_rem=64)
    s.update(p=p, inst0=inst.clone(), moves=_empty((c["moves"], star.MOVE_FIELDS), torch.int32),
             n_moves=_empty(1, torch.int32), ws=star.Workspace(star.plan_workspace_size(p)))
    return s


# ---------------------------------------------------------------------------
# one pass
# ---------------------------------------------------------------------------
# rem_len is a length rounded to a whole number.  Where it is returned, one
# row in a hundred may fall on the other side of a tie; batches too small for
# that share, and the regression head (whose bf16 first layer moves its
# outputs by tenths of a token), return the lengths before rounding alone.
TIES_FROM = 256


def _lengths(s, expected, rem, n):
    out = {"expected_len": expected}
    if s["ema"] is not None:
        out["ema"] = s["ema"]
    if s["kind"] != "mlp4" and n >= TIES_FROM:
        out["rem_len"] = rem
    return out


def run(s):
    kind = s["kind"]
    if kind == "predict":
        star.predict(s["p"], s["hidden"][0], s["w1"], s["b1"], s["w2"], s["b2"], s["bins"],
                     s["ema"], s["expected"][0], s["rem"][0], s["ws"][0])
        return _lengths(s, s["expected"][0], s["rem"][0], s["n_req"])
    if kind == "overlap":
        h, ws, T = s["hidden"], s["ws"], s["steps"]
        for i in range(T + 1):
            star.predict_overlap(s["p"], h[i] if i < T else None, ws[i & 1] if i < T else None,
                                 ws[(i - 1) & 1] if i else None, s["w1"], s["b1"], s["w2"],
                                 s["b2"], s["bins"], s["ema"] if i else None,
                                 s["expected"][i - 1] if i else None,
                                 s["rem"][i - 1] if i else None)
        return _lengths(s, s["expected"], s["rem"], s["n_req"])
    if kind == "mlp4":
        star.predict_mlp4(s["p"], s["hidden"], s["w1"], s["b1"], s["w2"], s["b2"], s["w3"],
                          s["b3"], s["w4"], s["ema"], s["expected"], s["rem"], s["ws"])
        return _lengths(s, s["expected"], s["rem"], 0)
    if kind == "schedule":
        star.project_and_score(s["p"], s["cur"], s["rem"], s["inst"], s["load"], s["scores"],
                               s["bt"], s["bs"], s["tr"], s["tt"], s["ts"], s["ws"])
        return {"load": s["load"], "scores": s["scores"], "best_target": s["bt"],
                "best_score": s["bs"], "topk_req": s["tr"], "topk_tgt": s["tt"],
                "topk_score": s["ts"]}
    if kind == "variance":
        star.project_load(s["lp"], s["cur"], s["rem"], s["inst"], s["load"], s["ws_load"])
        star.score_variance(s["lp"], s["cur"], s["rem"], s["inst"], s["load"], s["beta"],
                            s["gain"], s["bt"], s["bg"], s["move"], s["ws"])
        return {"load": s["load"], "gain": s["gain"], "best_target": s["bt"],
                "best_gain": s["bg"], "best_move": s["move"]}
    # a plan changes the placement in place: each pass starts from the crowded one
    s["inst"].copy_(s["inst0"])
    star.project_load(s["lp"], s["cur"], s["rem"], s["inst"], s["load"], s["ws_load"])
    star.plan_migrations(s["p"], s["cur"], s["rem"], s["inst"], s["load"], s["beta"], s["moves"],
                         s["n_moves"], s["ws"])
    return {"inst_of": s["inst"], "load": s["load"], "moves": s["moves"],
            "n_moves": s["n_moves"]}


# ---------------------------------------------------------------------------
# what a pass cannot do without, and how far its results may be off
# ---------------------------------------------------------------------------
def work(c):
    kind, n = c["kind"], c["n_req"]
    if kind in ("predict", "overlap"):
        e, T = (4 if c["dtype"] == "f32" else 2), c.get("steps", 1)
        byte = e * (T * n * c["d"] + c["m"] * c["d"] + c["nb"] * c["m"]) + T * 8 * n
        byte += 4 * c["nb"] + (4 * (c["m"] + c["nb"]) if c["bias"] else 0)
        byte += 8 * n if c["alpha"] else 0
        return {"bytes": byte, "flops": 2 * T * n * c["m"] * (c["d"] + c["nb"])}
    if kind == "mlp4":
        e = 4 if c["dtype"] == "f32" else 2
        w = c["d"] * c["m1"] + c["m1"] * c["m2"] + c["m2"] * c["m3"]
        byte = e * (n * c["d"] + w) + 4 * c["m3"] + 8 * n
        byte += 4 * (c["m1"] + c["m2"] + c["m3"]) if c["bias"] else 0
        byte += 8 * n if c["alpha"] else 0
        return {"bytes": byte, "flops": 2 * n * (w + c["m3"])}
    ni, K = c["n_inst"], c["n_buckets"]
    byte = 12 * n + 8 * ni * K
    if kind == "schedule":
        return {"bytes": byte + 8 * n * ni + 12 * n + 16 * c["top_k"], "flops": 0}
    if kind == "variance":
        return {"bytes": byte + 2 * K + 16 * n * ni + 20 * n + 32, "flops": 0}
    return {"bytes": byte + 2 * K + 8 * n + 32 * c["moves"] + 4, "flops": 0}


def tolerance(c):
    if c["kind"] in ("predict", "overlap"):
        return {"rel": 1e-5, "max": 1e-4, "differ": 0.01}
    if c["kind"] == "mlp4":     # the first layer's outputs are rounded to bf16
        return {"rel": 2.5e-3, "max": 1.5e-2}
    return "exact"


# ---------------------------------------------------------------------------
# the same in 64 bits (whole-number results are exact already)
# ---------------------------------------------------------------------------
def _smoothed(c, ema, y):
    return c["alpha"] * y + (1.0 - c["alpha"]) * ema


def _bias(z, b):
    return z if b is None else z + b.double()


def exact(case, seed):
    c = case
    if c["kind"] == "mlp4":
        x = _mlp4_inputs(c, seed)
        a = x["hidden"].double()
        for i in (1, 2, 3):
            a = torch.relu(_bias(a @ x["w%d" % i].double().t().contiguous(), x["b%d" % i]))
        y = a @ x["w4"].double() + x["b4"]
        out = {"expected_len": y}
        if c["alpha"]:
            out["ema"] = _smoothed(c, x["ema0"].double(), y)
        return out
    if c["kind"] not in ("predict", "overlap"):
        return None
    x = _head_inputs(c, seed)
    w1, w2 = (x[k].double().t().contiguous() for k in ("w1", "w2"))
    ema, E = x["ema0"].double(), []
    for h in x["hidden"]:
        z = _bias(h.double() @ w1, x["b1"])
        a = torch.relu(z) if c["act"] == "relu" else 0.5 * z * torch.special.erfc(-z / 2 ** 0.5)
        y = torch.softmax(_bias(a @ w2, x["b2"]), dim=1) @ x["bins"].double()
        ema = _smoothed(c, ema, y)
        E.append(y)
    out = {"expected_len": E[0] if c["kind"] == "predict" else E}
    if c["alpha"]:
        out["ema"] = ema
    if c["n_req"] >= TIES_FROM:
        out["rem_len"] = None if c["kind"] == "predict" else [None] * len(E)
    return out
