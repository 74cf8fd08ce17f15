"""The work whose speed counts here: the calls a training program makes on the library, at sizes from a toy decoder to a
1.2-billion-parameter state.

A state is a decoder's parameters laid out as such a program holds them: one flat array each for the weights, the shadow,
the fp32 master and the Adam moments, in layer order (embedding, blocks, final norm, head).  With ``world`` 1 every tensor is
one segment.  With ``world`` above 1 the program is one rank of a ZeRO-3 job and holds ceil(n / world) elements of each
tensor, one piece behind the other: for a world that is no power of two the pieces have odd lengths and start at any element.

Every fifth layer has a threshold of zero and is persisted at each step, about the 20% of the layers that the thresholds of
the paper are set for; the others stay below theirs.  So each pass persists the same layers, and what it moves is known.

The persistence store (files) is not among the cases: the disk decides its speed.
"""
import math
import random

import torch

from paper_2609_27193_amd import layercheck as LC

EPS_W = 1e-8
LR, BETA1, BETA2, ADAM_EPS, WEIGHT_DECAY = 1e-5, 0.9, 0.95, 1e-8, 0.1
ADAM_STEP0 = 100  # a run that is past its first steps
SGD_LR = 1e-2
DTYPES = {"bf16": (torch.bfloat16, LC.LC_DT_BF16, 2), "f32": (torch.float32, LC.LC_DT_F32, 4)}


def _case(name, op, **kw):
    c = {"name": name, "op": op, "dtype": "bf16", "master": True, "moments": True, "snapshot": False, "grad": "bf16",
         "log": False, "pinned": False, "hidden": 1024, "ffn": 2816, "blocks": 24, "vocab": 32000, "kv": 256, "bias": False,
         "gated": True, "tied": False, "world": 1}
    c.update(kw)
    return c


TOY = dict(dtype="f32", master=False, grad="f32", hidden=256, ffn=1024, blocks=4, vocab=1024, kv=256, gated=False)
ONE_B = dict(hidden=2048, ffn=8192, blocks=16, vocab=128256, kv=512, tied=True)  # the Llama-3.2-1B shape


def listed():
    return [
        # score, select and pack of a toy decoder (3.7 M parameters, fp32): launches and the host's round trip
        _case("decide_toy", "decide", **TOY),
        # the same on the largest state: the library's main path, beside an optimizer of the caller's own
        _case("decide_1b", "decide", **ONE_B),
        # drift against the last persisted version instead of the previous step
        _case("decide_1b_snapshot", "decide", snapshot=True, **ONE_B),
        # weights with biases and no master copy; the program logs u and Delta of every layer at each step
        _case("decide_bias_log", "decide", master=False, bias=True, log=True),
        # one rank's piece in a job of six: odd lengths, segments that start anywhere
        _case("decide_shard", "decide", world=6, **ONE_B),
        # the optimizer step that yields the drift itself, then select and pack
        _case("adamw_toy", "adamw", **TOY),
        _case("adamw_1b", "adamw", **ONE_B),
        # one rank's piece, with the fp32 gradients of an accumulating trainer
        _case("adamw_shard", "adamw", grad="f32", world=3),
        # plain SGD: records of weights and master alone
        _case("sgd", "sgd", moments=False),
        # recovery from a base and one later version, held on the device
        _case("restore_1b", "restore", **ONE_B),
        # and held in page-locked host memory
        _case("restore_pinned", "restore", pinned=True, hidden=512, ffn=1408, blocks=12, kv=128),
        # scores alone, for a program that cannot allocate
        _case("score_static", "static"),
    ]


def draw(rng):
    logint = lambda a, b: int(round(math.exp(rng.uniform(math.log(a), math.log(b)))))  # noqa: E731
    while True:
        op = rng.choice(["decide", "decide", "decide", "adamw", "adamw", "sgd", "restore", "static"])
        hidden = 64 * logint(2, 32) + rng.choice([0, 0, 0, 8, 10, 33])
        c = _case("", op, dtype=rng.choice(["bf16", "bf16", "bf16", "f32"]), master=rng.random() < 0.7,
                  snapshot=op == "decide" and rng.random() < 0.3, grad=rng.choice(["bf16", "f32"]), log=rng.random() < 0.25,
                  pinned=op == "restore" and rng.random() < 0.5, hidden=hidden, ffn=rng.choice([hidden * 4, hidden * 11 // 4]),
                  blocks=logint(2, 32), vocab=logint(500, 128256), kv=max(1, hidden // rng.choice([1, 4, 8])),
                  bias=rng.random() < 0.3, gated=rng.random() < 0.8, tied=rng.random() < 0.5,
                  world=rng.choice([1, 1, 1, 1, 3, 5, 6, 7, 12, 24]))
        c["master"] = c["master"] and c["dtype"] == "bf16"
        c["moments"] = op != "sgd" or rng.random() < 0.3
        c["log"] = c["log"] and op in ("decide", "adamw", "sgd")
        del c["name"]
        # within the largest listed case: its parameters, and its records where those cross the host link
        n = sum(k for _, k, _ in _tensors(c))
        if n * (2 if c["dtype"] == "f32" else 1) <= 1.2e9 and not (c["pinned"] and n > 7e7):
            return c


# ---- the layout ---------------------------------------------------------------------------------------------------------


def _tensors(c):
    """(layer, elements, decayed) of every segment in layout order."""
    h, f, kv = c["hidden"], c["ffn"], c["kv"]
    blk = [(h * h, 1)] + [(h, 0)] * c["bias"] + [(h * kv, 1)] + [(kv, 0)] * c["bias"] + [(h * kv, 1)] + [(kv, 0)] * c["bias"]
    blk += [(h * h, 1)] + [(h * f, 1)] * (3 if c["gated"] else 2) + [(h, 0), (h, 0)]
    layers = [[(c["vocab"] * h, 1)]] + [blk] * c["blocks"] + [[(h, 0)]] + ([] if c["tied"] else [[(c["vocab"] * h, 1)]])
    return [(i, -(-n // c["world"]), d) for i, l in enumerate(layers) for n, d in l]


def _ranges(c):
    """[first, last) element of every layer in the flat arrays."""
    out, at = [], 0
    for l, n, _ in _tensors(c):
        if l == len(out):
            out.append([at, at])
        at += n
        out[l][1] = at
    return out


def _persisted(n_layers):
    return [l for l in range(n_layers) if l % 5 == 2]


def _record_arrays(c):
    """Bytes an element of each array that a record holds."""
    return [DTYPES[c["dtype"]][2]] + [4] * c["master"] + [4, 4] * c["moments"]


def _record_bytes(c, layers):
    want = set(layers)
    return sum(-(-n * e // 256) * 256 for l, n, _ in _tensors(c) if l in want for e in _record_arrays(c))


# ---- the values ---------------------------------------------------------------------------------------------------------


def _values(c, seed):
    """The arrays before a step (0) and after an optimizer of the caller's own has made it (1)."""
    g = torch.Generator(device="cuda").manual_seed(seed)
    rng = random.Random(seed)
    segs, ranges = _tensors(c), _ranges(c)
    n = ranges[-1][1]
    wdt = DTYPES[c["dtype"]][0]
    randn = lambda scale: torch.randn(n, generator=g, device="cuda").mul_(scale)  # noqa: E731
    p = randn(0.02)
    at = 0
    for _, k, decayed in segs:
        if not decayed and k > 1:
            p[at:at + k] += 1.0  # norms and biases: no decay
        at += k
    v = {"w0": p.to(wdt)}
    if c["master"]:
        v["master0"] = p.clone()
    if c["op"] in ("adamw", "sgd"):
        v["grad"] = randn(1e-3).to(DTYPES[c["grad"]][0])
    else:
        d = randn(1e-3)  # the caller's step: layers move at rates that span two decades
        for a, b in ranges:
            d[a:b] *= 10.0 ** rng.uniform(-2.0, 0.0)
        p = v["w0"].float().add_(d) if not c["master"] else p.add_(d)
        v["w1"] = p.to(wdt)
        if c["master"]:
            v["master1"] = p
        del d
    if c["moments"] and c["op"] != "static":
        v["m"] = randn(1e-3)
        v["v"] = randn(1e-6).abs_()
    return v


class _State:
    """What the program keeps: its arrays, the library's context, the staging buffer."""

    def __init__(self):
        self.ctx, self.t = None, 0

    def __del__(self):
        if self.ctx is not None:
            LC.lc_destroy(self.ctx)


def prepare(c, seed):
    s = _State()
    s.case, v = c, _values(c, seed)
    op, segs, ranges = c["op"], _tensors(c), _ranges(c)
    wdt, lc_dt, esz = DTYPES[c["dtype"]]
    s.n = len(ranges)
    s.w, s.master, s.m, s.v = v["w0"], v.get("master0"), v.get("m"), v.get("v")
    s.shadow = torch.empty_like(s.w) if op not in ("adamw", "sgd") else None
    s.stream = torch.cuda.current_stream().cuda_stream
    s.segs, at = [], 0
    ptr = lambda a, e: None if a is None else a.data_ptr() + e * a.element_size()  # noqa: E731
    for l, k, _ in segs:
        s.segs.append(LC.Segment(l, k, ptr(s.w, at), ptr(s.shadow, at), ptr(s.master, at), ptr(s.m, at), ptr(s.v, at)))
        at += k
    if op == "static":
        s.shadow.copy_(s.w)
        s.w.copy_(v["w1"])
        s.u = torch.empty(s.n, dtype=torch.float64, device="cuda")
        s.lc_dt = lc_dt
        return s
    chosen = _persisted(s.n)
    k0 = [0.0 if l in chosen else 1e6 for l in range(s.n)]
    mode = LC.LC_MODE_SNAPSHOT if c["snapshot"] else LC.LC_MODE_ACCUM
    s.ctx = LC.lc_init_layout(LC.LayoutDesc(s.segs, s.n, lc_dt, c["master"], mode, k0, s_max=1 << 24, eps_w=EPS_W, stream=s.stream))
    s.staging = torch.zeros(_record_bytes(c, chosen) // 8, dtype=torch.int64, device="cuda")
    if op == "restore" or c["snapshot"]:  # the base version
        base = torch.empty(_record_bytes(c, range(s.n)) // 8, dtype=torch.int64, device="cuda")
        LC.lc_pack_selected(s.ctx, base.data_ptr(), base.numel() * 8, 0)
    if op in ("adamw", "sgd"):
        s.grad = v["grad"]
        s.lc_gdt, at = DTYPES[c["grad"]][1], 0
        s.grads, s.decay = [], [d for _, _, d in segs]
        for _, k, _ in segs:
            s.grads.append(ptr(s.grad, at))
            at += k
        return s
    s.w.copy_(v["w1"])
    if c["master"]:
        s.master.copy_(v["master1"])
    if op == "restore":
        _decide(s)
        records = [base, s.staging]
        if c["pinned"]:
            records = [torch.empty(r.shape, dtype=r.dtype, pin_memory=True).copy_(r) for r in records]
        masks = [torch.ones(s.n, dtype=torch.uint8).numpy(), s.mask]
        s.records = records
        s.versions = [{"step": i, "mask": k, "payload": r.data_ptr(), "payload_bytes": r.numel() * 8}
                      for i, (k, r) in enumerate(zip(masks, records))]
        for a in (s.w, s.shadow, s.master, s.m, s.v):  # the process that takes over starts with empty arrays
            if a is not None:
                a.zero_()
        torch.cuda.synchronize()
    return s


# ---- one pass -----------------------------------------------------------------------------------------------------------


def _decide(s):
    s.t += 1
    c = s.case
    if c["op"] == "adamw":
        LC.lc_adamw_step_score(s.ctx, s.t, s.grads, s.lc_gdt, LR, BETA1, BETA2, ADAM_EPS, WEIGHT_DECAY, ADAM_STEP0 + s.t, s.decay)
    elif c["op"] == "sgd":
        LC.lc_sgd_step_score(s.ctx, s.t, s.grads, s.lc_gdt, SGD_LR, WEIGHT_DECAY, s.decay)
    else:
        LC.lc_score_layers(s.ctx, s.t)
    out = {}
    if c["log"]:
        out["u"], out["delta"], _ = LC.lc_read_state(s.ctx, s.n)
    s.mask, stats = LC.lc_select(s.ctx, s.t, 1.0, s.n)
    rank, done = 0, 0
    while not done:
        r = LC.lc_pack_selected(s.ctx, s.staging.data_ptr(), s.staging.numel() * 8, rank)
        rank, done = r["next_rank"], r["done"]
    out.update(mask=s.mask, stats=stats, records=s.staging)
    return out


def run(s):
    op = s.case["op"]
    if op == "static":
        LC.lc_score_layers_static(s.segs, s.n, s.lc_dt, EPS_W, s.u.data_ptr(), s.stream)
        return {"u": s.u}
    if op == "restore":
        steps = LC.lc_restore_composite(s.ctx, s.versions, 1, s.n)
        return {"steps": steps, "w": s.w, "shadow": s.shadow, "master": s.master, "m": s.m, "v": s.v}
    out = _decide(s)
    if op == "decide":
        out["shadow"] = s.shadow
    else:
        out.update(w=s.w, master=s.master)
        if op == "adamw":
            out.update(m=s.m, v=s.v)
    return out


# ---- what a pass cannot do without, and what it has to give --------------------------------------------------------------


def work(c):
    segs, ranges = _tensors(c), _ranges(c)
    n, w = ranges[-1][1], DTYPES[c["dtype"]][2]
    chosen = _persisted(len(ranges))
    per = sum(_record_arrays(c))
    k = sum(b - a for l, (a, b) in enumerate(ranges) if l in chosen)
    records = _record_bytes(c, chosen)
    if c["op"] == "static":
        return {"bytes": 2 * w * n, "flops": 4 * n}
    if c["op"] == "restore":
        return {"bytes": n * (2 * per + w), "flops": 0}
    if c["op"] == "decide":  # W and S read, the rest of the chosen records read; S and the records written
        score = 2 * w * n + (k * w if c["snapshot"] else n * w)
        return {"bytes": score + k * (per - w) + records, "flops": 4 * n}
    g = DTYPES[c["grad"]][2]
    if c["op"] == "sgd":
        return {"bytes": n * (g + (8 + w if c["master"] else 2 * w)) + (8 * k if c["moments"] else 0) + records, "flops": 8 * n}
    return {"bytes": n * (g + 16 + (8 + w if c["master"] else 2 * w)) + records, "flops": 20 * n}


def tolerance(c):
    # copies are exact.  u and Delta are 64-bit sums over pairs of 32-bit terms: 7e-13 from 64 bits on large layers, nearer to
    # a rounding of one term on the smallest.  The optimizers work in fp32 (4e-8 from 64 bits on master, m and v), and a bf16
    # weight beside a tie may round the other way, by 2^-7 of its value.
    if c["op"] in ("adamw", "sgd"):
        return {"rel": 1e-5, "max": 8e-3}
    return {"rel": 1e-8, "max": 1e-7} if c["op"] != "restore" else "exact"


def _drift(ranges, before, after):
    u = []
    for a, b in ranges:
        x, y = before[a:b].double(), after[a:b].double()
        u.append(float((y - x).abs().mean() / (x.abs().mean() + EPS_W)))
    return torch.tensor(u, dtype=torch.float64)


def exact(c, seed):
    v, ranges = _values(c, seed), _ranges(c)
    if c["op"] == "static":
        return {"u": _drift(ranges, v["w0"], v["w1"])}
    chosen = _persisted(len(ranges))
    none = {"mask": None, "stats": {k: None for k in ("n_selected", "n_forced", "payload_bytes", "max_age", "weighted_age")},
            "records": None}
    if c["op"] == "restore":  # the chosen layers from the later version, the others from the base; the moments are alike
        for l in chosen:
            a, b = ranges[l]
            v["w0"][a:b] = v["w1"][a:b]
            if c["master"]:
                v["master0"][a:b] = v["master1"][a:b]
        return {"steps": None, "w": v["w0"].double(), "shadow": v["w0"].double(),
                "master": v["master0"].double() if c["master"] else None, "m": v["m"].double(), "v": v["v"].double()}
    if c["op"] == "decide":
        shadow = v["w1"].clone()
        if c["snapshot"]:
            shadow = v["w0"].clone()
            for l in chosen:
                a, b = ranges[l]
                shadow[a:b] = v["w1"][a:b]
        u = _drift(ranges, v["w0"], v["w1"]) if c["log"] else None
        return dict(none, shadow=shadow.double(), **({"u": u, "delta": u} if c["log"] else {}))
    p = (v["master0"] if c["master"] else v["w0"]).double()
    g, t = v["grad"].double(), ADAM_STEP0 + 1
    q, at, lr = p.clone(), 0, SGD_LR if c["op"] == "sgd" else LR
    for _, k, decayed in _tensors(c):
        if decayed:
            q[at:at + k] *= 1.0 - lr * WEIGHT_DECAY
        at += k
    out = dict(none)
    if c["op"] == "sgd":
        q -= lr * g
    else:
        m = v["m"].double().mul_(BETA1).add_(g, alpha=1.0 - BETA1)
        s = v["v"].double().mul_(BETA2).add_(g * g, alpha=1.0 - BETA2)
        q -= lr * (m / (1.0 - BETA1 ** t)) / ((s / (1.0 - BETA2 ** t)).sqrt_() + ADAM_EPS)
        out.update(m=m, v=s)
    if c["log"]:
        u = _drift(ranges, p, q)
        out.update(u=u, delta=u)
    return dict(out, w=q, master=q if c["master"] else None)
