"""Performance cases of the true-tail update: what a program using this package calls.

A case is one call (or the few calls that belong together) through the public entry
points, at sizes from the package's own workloads: 12K to 64K row character contexts,
tails of one token (speaking) to thousands (refilling), hybrid stacks of 2 and 48 layers
with three delta layers per attention layer, head shapes 16/2/256 and 16-32/128 and their
smaller relatives. `listed()` are the named cases, `draw(rng)` gives others of the same
ranges, `exact(case, seed)` the float64 result of the first pass.

An update case is a running program: a context holds untouched text and then records of
one length, and every pass revises the records that sit at fixed places of the row order
(their rows are removed, replacements of the same length are appended), so the context
keeps its length while its positions grow, pass after pass.
"""
import math
import random

import torch

import paper_2609_18935_amd as tu

DEV = "cuda"
THETA = 1.0e7

# (query heads, KV heads, head dim) and (key heads, value heads, d, chunk); the first of
# each is the shape of the package's own configurations
ATTN_SHAPES = [(16, 2, 256), (32, 8, 128), (16, 4, 64)]
DELTA_SHAPES = [(16, 32, 128, 64), (16, 16, 128, 32), (8, 16, 64, 64), (2, 2, 64, 16)]


def _attn(shape, **kw):
    hq, hkv, dim = shape
    return dict(hq=hq, hkv=hkv, dim=dim, rotary=dim, **kw)


def _delta(shape, **kw):
    hk, hv, d, chunk = shape
    return dict(hk=hk, hv=hv, d=d, chunk=chunk, **kw)


def listed():
    a, d = ATTN_SHAPES[0], DELTA_SHAPES[0]
    return [
        # a character speaks: one token of one attention layer over a 32K context whose
        # V^T copy is current
        _attn(a, name="attn-decode", kind="attention", rows=32768, T=1, vt=True),
        # a short line of dialogue enters a paper-sized (12K) context; no V^T copy kept
        _attn(a, name="attn-turn", kind="attention", rows=11907, T=24, vt=False),
        # one layer of a full refill: the comparator of every maintained update
        _attn(a, name="attn-refill", kind="attention", rows=0, T=8191, vt=False),
        # the recurrent layer's share of the same three: one token, a tail, a refill
        _delta(d, name="delta-decode", kind="delta", T=1),
        _delta(d, name="delta-tail", kind="delta", T=512),
        _delta(d, name="delta-refill", kind="delta", T=8191),
        # the short convolutions of one layer's q, k and v in front of the delta rule
        dict(name="conv-tail", kind="conv", T=300, cq=2048, ck=2048, cv=4096, width=4, silu=True),
        # one character refreshed: three 128-token records, one layer of each kind
        _attn(a, **_delta(d, name="update-refresh", kind="update", contexts=1, rows_lo=8576, rows_hi=8576, records=3,
                          rec_lo=128, rec_hi=128, n_attn=1, n_delta=1, at=0.5, placement="tail", delims=0)),
        # a paper-shaped revision: one record of a 12K context through the whole 48-layer stack
        _attn(a, **_delta(d, name="update-revision", kind="update", contexts=1, rows_lo=11300, rows_hi=11300,
                          records=1, rec_lo=291, rec_hi=291, n_attn=12, n_delta=36, at=0.5, placement="tail",
                          delims=0)),
        # a population of 32 characters maintained in one call
        _attn(a, **_delta(d, name="update-population", kind="update", contexts=32, rows_lo=4096, rows_hi=16384,
                          records=4, rec_lo=32, rec_hi=128, n_attn=1, n_delta=1, at=0.3, placement="tail",
                          delims=0)),
        # the long-lived character: eight 256-token records of a 64K context, 48 layers
        _attn(a, **_delta(d, name="update-64k", kind="update", contexts=1, rows_lo=65536, rows_hi=65536, records=8,
                          rec_lo=256, rec_hi=256, n_attn=12, n_delta=36, at=0.2, placement="tail", delims=0)),
        # the attention diagnostics of that context: 8 probe rows over its 12 attention
        # layers, the masses of its memory records, the distance to another distribution
        _attn(a, name="diagnostics-64k", kind="diagnostics", rows=65536, layers=12, probe=8, groups=174),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    a = ATTN_SHAPES[0] if rng.random() < 0.6 else rng.choice(ATTN_SHAPES[1:])
    d = DELTA_SHAPES[0] if rng.random() < 0.6 else rng.choice(DELTA_SHAPES[1:])
    kind = rng.choice(["attention", "attention", "attention", "delta", "delta", "conv", "update", "update", "update",
                       "diagnostics"])
    if kind == "attention":
        rows = 0 if rng.random() < 0.15 else _log_int(rng, 256, 65536)
        c = _attn(a, kind=kind, rows=rows, T=_log_int(rng, 1, 8192), vt=rng.random() < 0.5)
        if rng.random() < 0.2:
            c["rotary"] = c["dim"] // 2
        return c
    if kind == "delta":
        return _delta(d, kind=kind, T=_log_int(rng, 1, 8192))
    if kind == "conv":
        return dict(kind=kind, T=_log_int(rng, 1, 8192), cq=d[0] * d[2], ck=d[0] * d[2], cv=d[1] * d[2],
                    width=rng.choice([2, 3, 4, 4, 4]), silu=rng.random() < 0.8)
    if kind == "diagnostics":
        g = a[0] // a[1]
        return _attn(a, kind=kind, rows=_log_int(rng, 1024, 65536), layers=rng.choice([1, 4, 12]),
                     probe=rng.randint(1, max(1, min(8, 128 // g))), groups=rng.randint(8, 200))
    placement = rng.choice(["tail", "tail", "tail", "slot", "relocate"])
    records = rng.randint(1, 8)
    contexts = 1 if rng.random() < 0.7 else rng.randint(2, 32)
    stack = rng.choice([(1, 1), (2, 6), (12, 36)]) if contexts == 1 else (1, 1)
    hi = _log_int(rng, 4096, 65536 if contexts == 1 else 16384)
    lo = hi if contexts == 1 else rng.randint(2048, hi)
    rec_hi = rng.randint(max(16, lo // 512), max(256, lo // 512) if lo >= 8192 else min(256, lo // (4 * records)))
    return _attn(a, **_delta(d, kind=kind, contexts=contexts, rows_lo=lo, rows_hi=hi, records=records,
                             rec_lo=rng.randint(max(16, lo // 512, rec_hi // 2), rec_hi), rec_hi=rec_hi, n_attn=stack[0],
                             n_delta=stack[1], at=round(rng.uniform(0.0, 0.7), 2), placement=placement,
                             delims=rng.choice([0, 0, 2, 7]) if placement == "tail" else 0))


# ----------------------------------------------------------------------------- inputs

class _Inputs:
    """Seeded draws on the device, each tensor from a generator of its own."""

    def __init__(self, seed):
        self.seed, self.n = int(seed), 0

    def _gen(self):
        self.n += 1
        return torch.Generator(device=DEV).manual_seed((self.seed * 1000003 + self.n) & 0x7FFFFFFFFFFF)

    def bf16(self, *shape):
        return torch.randn(shape, generator=self._gen(), device=DEV, dtype=torch.float32).to(torch.bfloat16)

    def f32(self, *shape):
        return torch.randn(shape, generator=self._gen(), device=DEV, dtype=torch.float32)

    def keys(self, *shape):   # L2-normalised keys of the delta rule
        return torch.nn.functional.normalize(self.f32(*shape), dim=-1).to(torch.bfloat16)

    def beta(self, *shape):
        return torch.sigmoid(self.f32(*shape))

    def gate(self, *shape):
        return torch.exp(-torch.nn.functional.softplus(self.f32(*shape) - 4.0))


def _attn_params(c):
    return tu.attn_params(c["hq"], c["hkv"], c["dim"], c["rotary"], THETA)


def _delta_params(c):
    return tu.delta_params(c["hk"], c["hv"], c["d"], c["d"], c["chunk"])


def _sizes(c):
    """(rows, record length) of every context of an update case."""
    rng = random.Random(repr(sorted((k, v) for k, v in c.items() if k != "name")))
    return [(rng.randint(c["rows_lo"], c["rows_hi"]), rng.randint(c["rec_lo"], c["rec_hi"]))
            for _ in range(c["contexts"])]


def _revised(c, rows, n):
    """First row of each record a pass revises: spread evenly over the records, which fill
    the rows from the fraction `at` on (the text before takes what is left over)."""
    held = max(c["records"], int(rows * (1.0 - c["at"])) // n)
    return [rows - (held - i * held // c["records"]) * n for i in range(c["records"])]


def _attention_inputs(c, seed):
    x, rows, T = _Inputs(seed), c["rows"], c["T"]
    cap = rows + T
    kc = torch.zeros((cap, c["hkv"], c["dim"]), dtype=torch.bfloat16, device=DEV)
    vc = torch.zeros_like(kc)
    kc[:rows] = x.bf16(rows, c["hkv"], c["dim"])
    vc[:rows] = x.bf16(rows, c["hkv"], c["dim"])
    return kc, vc, x.bf16(T, c["hq"], c["dim"]), x.bf16(T, c["hkv"], c["dim"]), x.bf16(T, c["hkv"], c["dim"])


def _delta_inputs(c, x, n, T):
    """q, k, v, beta, g of n layers and their carried states."""
    return (x.bf16(n, T, c["hk"], c["d"]), x.keys(n, T, c["hk"], c["d"]), x.bf16(n, T, c["hv"], c["d"]),
            x.beta(n, T, c["hv"]), x.gate(n, T, c["hv"]))


def _conv_inputs(c, seed):
    x, w = _Inputs(seed), c["width"]
    return [(x.bf16(w - 1, ch), x.bf16(c["T"], ch), (x.f32(ch, w) * 0.5).to(torch.bfloat16))
            for ch in (c["cq"], c["ck"], c["cv"])]


def _update_inputs(c, seed):
    x, sizes = _Inputs(seed), _sizes(c)
    na, nd = c["n_attn"], c["n_delta"]
    T = [n * c["records"] + 2 * c["delims"] for _, n in sizes]
    total = sum(T)
    caches = []
    for rows, _ in sizes:
        cap = rows + 2 * c["delims"] + 64
        kv = [torch.zeros((na, cap, c["hkv"], c["dim"]), dtype=torch.bfloat16, device=DEV) for _ in range(2)]
        for t in kv:
            for l in range(na):
                t[l, :rows] = x.bf16(rows, c["hkv"], c["dim"])
        caches.append(kv)
    tail = (x.bf16(na, total, c["hq"], c["dim"]), x.bf16(na, total, c["hkv"], c["dim"]),
            x.bf16(na, total, c["hkv"], c["dim"]))
    dtail = _delta_inputs(c, x, nd, total)
    states = [x.f32(nd, c["hv"], c["d"], c["d"]) * 0.1 for _ in sizes]
    return sizes, T, caches, tail, dtail, states


def _diagnostics_inputs(c, seed):
    x, rows = _Inputs(seed), c["rows"]
    k = [x.bf16(rows, c["hkv"], c["dim"]) for _ in range(c["layers"])]
    q = [x.bf16(c["probe"], c["hq"], c["dim"]) for _ in range(c["layers"])]
    other = x.f32(rows).abs()
    other /= other.sum()
    n = c["groups"]
    size = max(1, rows * 3 // 4 // n)   # records fill the middle of the context
    groups = [(rows // 8 + i * size, rows // 8 + i * size + max(1, size - 1)) for i in range(n)]
    return k, q, other, groups


# ----------------------------------------------------------------------------- programs

class _Program:
    """One context set under revision: the loop an update case runs."""

    def __init__(self, c, seed):
        self.c = c
        self.sizes, self.T, self.caches, self.tail, self.dtail, self.states = _update_inputs(c, seed)
        na, nd, total = c["n_attn"], c["n_delta"], sum(self.T)
        self.out = torch.zeros((na, total, c["hq"], c["dim"]), dtype=torch.float32, device=DEV)
        self.dout = torch.zeros((nd, total, c["hv"], c["d"]), dtype=torch.float32, device=DEV)
        self.ctx, self.records = [], []
        vts = []
        for (rows, n), (kc, vc) in zip(self.sizes, self.caches):
            ctx = tu.Context(kc.shape[1], device=DEV)
            ctx.pos[:rows] = torch.arange(rows, dtype=torch.int32, device=DEV)
            ctx.set_metadata([(0, rows)], rows)
            vt = [tu.new_vt_cache(kc.shape[1], c["hkv"], c["dim"], device=DEV) for _ in range(na)]
            for t in vt:
                t.zero_()
            tu.refresh_vt_cache(ctx, [vc[l] for l in range(na)], vt)
            vts.append(vt)
            self.ctx.append(ctx)
            # the records in row order, by first position
            self.records.append([p for p in range(_revised(c, rows, n)[0], rows, n)])
        q, k, v = self.tail
        dq, dk, dv, beta, g = self.dtail
        self.layers, ai, di = [], 0, 0
        per = max(1, nd // max(1, na))
        while ai < na or di < nd:
            for _ in range(per):
                if di < nd:
                    self.layers.append(tu.LayerIO(tu.TU_LAYER_DELTA, dq[di], dk[di], dv[di], self.dout[di],
                                                  state=[s[di] for s in self.states], beta=beta[di], g=g[di]))
                    di += 1
            if ai < na:
                self.layers.append(tu.LayerIO(tu.TU_LAYER_ATTN, q[ai], k[ai], v[ai], self.out[ai],
                                              k_cache=[kv[0][ai] for kv in self.caches],
                                              v_cache=[kv[1][ai] for kv in self.caches],
                                              vt_cache=[vt[ai] for vt in vts]))
                ai += 1
        self.vts = vts
        self.attn, self.delta = _attn_params(c), _delta_params(c)
        plan = self.plan()
        up = tu.StackUpdate(self.ctx, plan[0], self.T, self.layers, self.attn, self.delta, **self.options(plan))
        self.workspace = torch.empty(up.workspace_size(), dtype=torch.uint8, device=DEV)

    def plan(self):
        """Position ranges of the records to revise, the tail's delimiters, its placement."""
        ranges, post, runs = [], [], []
        d = self.c["delims"]
        for ctx, (_, n), held, T in zip(self.ctx, self.sizes, self.records, self.T):
            gone = sorted(held[i] for i in self.turn(held))
            ranges.append([(p, p + n) for p in gone])
            p = ctx.next_pos
            post.append([(p, p + d), (p + T - d, p + T)] if d else None)
            runs.append(ranges[-1] if self.c["placement"] != "tail" else None)
        return ranges, post, runs

    def turn(self, held):
        """Which of the records held are revised (see _revised)."""
        r = self.c["records"]
        return [i * len(held) // r for i in range(r)]

    def options(self, plan):
        return dict(post_ranges=plan[1], placement=[self.c["placement"]] * len(self.ctx), place_runs=plan[2])

    def step(self):
        plan = self.plan()
        cursor = [ctx.next_pos for ctx in self.ctx]
        tu.update_layer_stack(self.ctx, plan[0], self.T, self.layers, self.attn, self.delta, workspace=self.workspace,
                              **self.options(plan))
        for s, (held, (_, n), p) in enumerate(zip(self.records, self.sizes, cursor)):
            gone = set(self.turn(held))
            if self.c["placement"] == "tail":
                new = [p + self.c["delims"] + i * n for i in range(len(gone))]
            else:
                new = [a for a, _ in plan[0][s]]
            self.records[s] = [x for i, x in enumerate(held) if i not in gone] + new

    def result(self):
        rows = [r for r, _ in self.sizes]
        return {"attention": self.out, "delta": self.dout, "states": self.states,
                "k_cache": [kv[0][:, :r] for kv, r in zip(self.caches, rows)][:4],
                "v_cache": [kv[1][:, :r] for kv, r in zip(self.caches, rows)][:4],
                "pos": [ctx.pos[:r] for ctx, r in zip(self.ctx, rows)][:4]}


def prepare(case, seed):
    c, kind = case, case["kind"]
    if kind == "update":
        return {"kind": kind, "program": _Program(c, seed)}
    if kind == "attention":
        kc, vc, q, k, v = _attention_inputs(c, seed)
        rows, T = c["rows"], c["T"]
        ctx = tu.Context(rows + T, device=DEV)
        ctx.pos[:rows] = torch.arange(rows, dtype=torch.int32, device=DEV)
        ctx.set_metadata([(0, rows)] if rows else [], rows)
        vt = None
        if c["vt"]:
            vt = tu.new_vt_cache(rows + T, c["hkv"], c["dim"], device=DEV)
            vt.zero_()
            if rows:
                tu.refresh_vt_cache(ctx, [vc], [vt])
        p = _attn_params(c)
        out = torch.zeros((T, c["hq"], c["dim"]), dtype=torch.float32, device=DEV)
        return dict(kind=kind, ctx=ctx, kc=kc, vc=vc, q=q, k=k, v=v, vt=vt, params=p, out=out)
    if kind == "delta":
        x = _Inputs(seed)
        q, k, v, beta, g = (t[0] for t in _delta_inputs(c, x, 1, c["T"]))
        state = x.f32(c["hv"], c["d"], c["d"]) * 0.1
        out = torch.zeros((c["T"], c["hv"], c["d"]), dtype=torch.float32, device=DEV)
        return dict(kind=kind, state=state, q=q, k=k, v=v, beta=beta, g=g, params=_delta_params(c), out=out)
    if kind == "conv":
        return dict(kind=kind, silu=c["silu"],
                    items=[(s, x, w, torch.empty_like(x)) for s, x, w in _conv_inputs(c, seed)])
    k, q, other, groups = _diagnostics_inputs(c, seed)
    ctx = tu.Context(c["rows"], device=DEV)
    ctx.pos[:] = torch.arange(c["rows"], dtype=torch.int32, device=DEV)
    ctx.set_metadata([(0, c["rows"])], c["rows"])
    probs = torch.zeros(c["rows"], dtype=torch.float32, device=DEV)
    return dict(kind=kind, ctx=ctx, k=k, q=q, other=other, groups=groups, params=_attn_params(c), probs=probs)


def run(state):
    s, kind = state, state["kind"]
    if kind == "update":
        s["program"].step()
        return s["program"].result()
    if kind == "attention":
        tu.tail_prefill_attention(s["ctx"], s["kc"], s["vc"], s["params"], s["q"], s["k"], s["v"], s["out"],
                                  vt_cache=s["vt"])
        return s["out"], s["kc"], s["vc"], s["ctx"].pos
    if kind == "delta":
        tu.delta_rule_continue(s["state"], s["q"], s["k"], s["v"], s["beta"], s["g"], s["params"], s["out"])
        return s["out"], s["state"]
    if kind == "conv":
        tu.short_conv_continue_batch(s["items"], "silu" if s["silu"] else "none")
        return [t for st, _, _, out in s["items"] for t in (out, st)]
    s["probs"].zero_()
    for k, q in zip(s["k"], s["q"]):
        tu.attention_probe(s["ctx"], k, s["params"], q, s["probs"], 1.0 / len(s["k"]))
    mass, window, summary = tu.attention_group_mass(s["ctx"], s["probs"], s["groups"])
    return s["probs"], mass, window, summary, tu.attention_tv_distance(s["probs"], s["other"])


# ----------------------------------------------------------------------------- cost

def _attn_work(c, rows, T):
    kv = c["hkv"] * c["dim"] * 2
    n_bytes = 2 * kv * (rows + T) + 2 * kv * T + T * c["hq"] * c["dim"] * (2 + 4)
    return n_bytes, 4.0 * c["dim"] * c["hq"] * (T * rows + T * (T + 1) / 2)


def _delta_work(c, T):
    d = c["d"]
    n_bytes = T * (2 * c["hk"] * d * 2 + c["hv"] * (2 * d + 8 + 4 * d)) + 2 * c["hv"] * d * d * 4
    return n_bytes, 6.0 * T * c["hv"] * d * d


def work(case):
    c, kind = case, case["kind"]
    if kind == "attention":
        b, f = _attn_work(c, c["rows"], c["T"])
    elif kind == "delta":
        b, f = _delta_work(c, c["T"])
    elif kind == "conv":
        ch = c["cq"] + c["ck"] + c["cv"]
        b = 2 * ch * (2 * c["T"] + 2 * (c["width"] - 1) + c["width"])
        f = 2.0 * ch * c["T"] * c["width"]
    elif kind == "diagnostics":
        row = c["hkv"] * c["dim"] * 2
        b = c["layers"] * (c["rows"] * row + c["probe"] * c["hq"] * c["dim"] * 2) + 4 * 4 * c["rows"]
        f = 2.0 * c["layers"] * c["rows"] * c["probe"] * c["hq"] * c["dim"]
    else:
        b = f = 0.0
        kv = c["hkv"] * c["dim"] * 2
        for rows, n in _sizes(c):
            gone, T = n * c["records"], n * c["records"] + 2 * c["delims"]
            moved = rows - gone - _revised(c, rows, n)[0]
            ab, af = _attn_work(c, rows - gone, T)
            db, df = _delta_work(c, T)
            b += c["n_attn"] * (ab + 2 * 2 * kv * moved) + c["n_delta"] * db + 8 * rows
            f += c["n_attn"] * af + c["n_delta"] * df
    return {"bytes": float(b), "flops": float(f)}


def tolerance(case):
    # Four times the error measured against exact(): attention 1.7e-4 to 2.9e-4 (f16
    # probabilities and partial results), delta rule 2.2e-4 to 3.8e-4 (f16 operands),
    # convolution 1.7e-3 (bf16 results); diagnostics are 32-bit sums (up to 4e-7). Caches
    # hold bf16, rounded once.
    kind = case["kind"]
    if kind == "conv":
        return {"rel": 7e-3}
    if kind == "diagnostics":
        return {"rel": 1e-5}
    return {"rel": 1.5e-3}


# ----------------------------------------------------------------------------- float64

def _rope64(x, pos, rotary, start=None):
    """Rotary embedding of x [T][H][D] (float64) at positions pos, rounded to bf16."""
    half = rotary // 2
    w = THETA ** (-2.0 * torch.arange(half, dtype=torch.float64, device=x.device) / rotary)
    ang = pos.to(torch.float64)[:, None] * w
    cos, sin = ang.cos()[:, None], ang.sin()[:, None]
    a, b = x[..., :half], x[..., half:rotary]
    return torch.cat([a * cos - b * sin, b * cos + a * sin, x[..., rotary:]], -1).to(torch.bfloat16).double()


def _attend64(q, k, v, rows, dim):
    """Causal grouped-query attention of rotated q [T][Hq][D] over k, v [rows + T][Hkv][D]."""
    T, hq, hkv = q.shape[0], q.shape[1], k.shape[1]
    g, n = hq // hkv, k.shape[0]
    out = torch.empty_like(q)
    step = max(1, (1 << 28) // max(1, n * g))
    key = torch.arange(n, device=q.device)
    for h in range(hkv):
        kt, vh = k[:, h].t().contiguous(), v[:, h].contiguous()
        for t0 in range(0, T, step):
            t1 = min(T, t0 + step)
            s = (q[t0:t1, h * g:(h + 1) * g].reshape(-1, dim) @ kt) * float(dim) ** -0.5
            s = s.view(t1 - t0, g, n)
            s.masked_fill_(key[None, None] > rows + torch.arange(t0, t1, device=q.device)[:, None, None], -math.inf)
            p = torch.softmax(s, -1)
            out[t0:t1, h * g:(h + 1) * g] = (p.view(-1, n) @ vh).view(t1 - t0, g, dim)
    return out


def _delta64(state, q, k, v, beta, g, scale):
    """Token by token: state [N][Hv][dv][dk], q, k [N][T][Hk][d], v [N][T][Hv][d]."""
    S = state.double().clone()
    r = v.shape[2] // q.shape[2]
    q, k = (t.double().repeat_interleave(r, 2) for t in (q, k))
    v, beta, g = v.double(), beta.double(), g.double()
    out = torch.empty(v.shape, dtype=torch.float64, device=v.device)
    for t in range(v.shape[1]):
        kt, bt = k[:, t], beta[:, t, :, None]
        S *= g[:, t, :, None, None]
        u = bt * (v[:, t] - (S @ kt[..., None])[..., 0])
        S += u[..., None] * kt[..., None, :]
        out[:, t] = scale * (S @ q[:, t][..., None])[..., 0]
    return out, S


def exact(case, seed):
    c, kind = case, case["kind"]
    if kind == "attention":
        rows, T = c["rows"], c["T"]
        kc, vc, q, k, v = (t.double() for t in _attention_inputs(c, seed))
        pos = rows + torch.arange(T, device=DEV)
        kc[rows:] = _rope64(k, pos, c["rotary"])
        vc[rows:] = v
        out = _attend64(_rope64(q, pos, c["rotary"]), kc, vc, rows, c["dim"])
        return out, kc, vc, None
    if kind == "delta":
        x = _Inputs(seed)
        q, k, v, beta, g = _delta_inputs(c, x, 1, c["T"])
        state = x.f32(c["hv"], c["d"], c["d"]) * 0.1
        out, S = _delta64(state[None], q, k, v, beta, g, c["d"] ** -0.5)
        return out[0], S[0]
    if kind == "conv":
        res, w1 = [], c["width"] - 1
        for st, x, w in _conv_inputs(c, seed):
            xt = torch.cat([st, x]).double()
            y = sum(xt[j:j + c["T"]] * w[:, j].double() for j in range(c["width"]))
            res += [y * torch.sigmoid(y) if c["silu"] else y, xt[xt.shape[0] - w1:]]
        return res
    if kind == "diagnostics":
        ks, qs, other, groups = _diagnostics_inputs(c, seed)
        rows, n = c["rows"], c["probe"]
        probs = torch.zeros(rows, dtype=torch.float64, device=DEV)
        at = rows - n + torch.arange(n, device=DEV)
        hidden = torch.arange(rows, device=DEV)[None] > at[:, None]
        g = c["hq"] // c["hkv"]
        for k, q in zip(ks, qs):
            qr = _rope64(q.double(), at, c["rotary"])
            for h in range(c["hq"]):
                s = (qr[:, h] @ k[:, h // g].double().t().contiguous()) * float(c["dim"]) ** -0.5
                probs += torch.softmax(s.masked_fill(hidden, -math.inf), -1).sum(0)
        probs /= len(ks) * n * c["hq"]
        mass = torch.stack([probs[a:b].sum() for a, b in groups])
        win = torch.stack([probs[a:min(b, a + 8)].sum() for a, b in groups])
        M = mass.sum()
        p = mass / M
        summary = torch.stack([M, torch.exp(-(p * p.log()).sum()), win.sum() / M])
        return probs, mass, win, summary, 0.5 * (probs - other.double()).abs().sum()[None]
    return _update64(c, seed)


def _update64(c, seed):
    sizes, Ts, caches, (q, k, v), dtail, states = _update_inputs(c, seed)
    na, d = c["n_attn"], c["delims"]
    outs, douts, s_after, kcs, vcs = [], [], [], [], []
    r0 = 0
    for (rows, n), T, (kc, vc), st in zip(sizes, Ts, caches, states):
        keep = torch.ones(rows, dtype=torch.bool, device=DEV)
        gone = []
        for a in _revised(c, rows, n):
            keep[a:a + n] = False
            gone.append(torch.arange(a, a + n, device=DEV))
        tail_pos = rows + torch.arange(T, device=DEV)
        slot_pos = torch.cat(gone)
        pos = slot_pos if c["placement"] == "slot" else tail_pos
        stays = slice(d, T - d) if d else slice(0, T)
        so, sk, sv = [], [], []
        for l in range(na):
            ql, kl, vl = (t[l, r0:r0 + T].double() for t in (q, k, v))
            kr = _rope64(kl, pos, c["rotary"])
            kk = torch.cat([kc[l, :rows][keep].double(), kr])
            vv = torch.cat([vc[l, :rows][keep].double(), vl])
            n_keep = kk.shape[0] - T
            so.append(_attend64(_rope64(ql, pos, c["rotary"]), kk, vv, n_keep, c["dim"]))
            if c["placement"] == "relocate":
                kr = _rope64(kr, slot_pos - tail_pos, c["rotary"])
            sk.append(torch.cat([kk[:n_keep], kr[stays]]).to(torch.bfloat16))
            sv.append(torch.cat([vv[:n_keep], vl[stays]]).to(torch.bfloat16))
        outs.append(torch.stack(so))
        o, S = _delta64(st, *(t[:, r0:r0 + T] for t in dtail), c["d"] ** -0.5)
        douts.append(o)
        s_after.append(S)
        if len(kcs) < 4:
            kcs.append(torch.stack(sk).double())
            vcs.append(torch.stack(sv).double())
        r0 += T
    return {"attention": torch.cat(outs, 1), "delta": torch.cat(douts, 1), "states": s_after, "k_cache": kcs,
            "v_cache": vcs, "pos": [None] * len(kcs)}
