"""Workloads of the decode path, as a program that serves a model runs them.

Every case calls the C ABI of ``include/m2r2.h`` through the symbols of
``paper_2502_02040_amd.binding``: a context over weights that stay in HBM, a
paged KV cache with a shuffled block table, and one call (or one short run of
calls) per pass.  Weights, cache content and tokens are random, drawn on the
GPU from the seed in the distributions of the package's synthetic models:
matrices N(0, 0.02), norm gains around 1, cached keys and values N(0, 1).  Rows
of the LM head differ in norm, as trained ones do, so that the greedy token is
seldom a near tie.

Kinds of cases:
  step     one dual-stream (or plain) decode step of one sequence
  batch    one dual-stream step of several sequences of different lengths
  spec     one self-speculative round: draft gamma tokens, verify them
  prefill  a prompt in chunks of up to 16 tokens
  moe      teacher-forced decode steps of a mixture-of-experts model
"""
from __future__ import annotations

import ctypes
import math
from concurrent.futures import ThreadPoolExecutor

import numpy as np
import torch

from paper_2502_02040_amd import binding as ab

EPS, THETA = 1e-5, 10000.0
NEVER = 2.0          # a threshold no signal (a cosine) reaches
PROJ = "qkvogud"     # order of a layer's adapters in the ABI

# layers, d_model, heads, head_dim, ffn, vocab, adapter rank, dtype (and the cache's, where it is
# another); for a mixture of experts its experts, top_k and expert width; for the FLOPs-optimised fast stream its heads, positions and head rank
MODELS = {
    "tiny": dict(N=2, d=256, H=4, hd=64, F=1024, V=1024, r=8, dt="f32"),
    "small": dict(N=3, d=192, H=2, hd=96, F=320, V=1000, r=4, dt="bf16", kv="f32"),
    "phi3": dict(N=32, d=3072, H=32, hd=96, F=8192, V=32064, r=16, dt="bf16"),
    "phi3_flops": dict(N=32, d=3072, H=32, hd=96, F=8192, V=32064, r=16, dt="bf16", fh=8, ftk=64, hr=64),
    # four layers of the OLMoE shape: its experts are 3.2 GB of pinned host memory
    "olmoe4": dict(N=4, d=2048, H=16, hd=128, F=0, V=50304, r=16, dt="bf16", E=64, K=8, Fe=1024),
}


def listed():
    return [
        # the smallest call: a float32 model of 10 MB, bound by the chain of its phases
        dict(name="tiny step", kind="step", model="tiny", ctx=16, cap=128, dual=True, exits="all"),
        # a small model of ragged widths with a float32 cache, three sequences of odd lengths
        dict(name="small batch 3", kind="batch", model="small", ctx=45, cap=64, batch=3, exits="every 2"),
        # the ordinary call: one sequence, both streams, gates observed at every layer
        dict(name="step 1024", kind="step", model="phi3", ctx=1024, cap=1360, dual=True, exits="all"),
        # plain decoding (the slow stream alone) late in a long context
        dict(name="plain step 7001", kind="step", model="phi3", ctx=7001, cap=8192, dual=False, exits="off"),
        # dynamic compute: the token leaves at the second gate
        dict(name="early exit 600", kind="step", model="phi3", ctx=600, cap=2048, dual=True, exits="exit 24"),
        # the FLOPs-optimised fast stream
        dict(name="flops step 1024", kind="step", model="phi3_flops", ctx=1024, cap=1360, dual=True, exits="all"),
        # serving batches: a full one of long contexts, and a small one of odd lengths
        dict(name="batch 8 x 4096", kind="batch", model="phi3", ctx=4096, cap=4352, batch=8, exits="every 1"),
        dict(name="batch 3 x 517", kind="batch", model="phi3", ctx=517, cap=1024, batch=3, exits="every 4"),
        # self-speculative decoding
        dict(name="speculative round", kind="spec", model="phi3", ctx=700, cap=1024, gamma=4, exit_layer=8),
        # a prompt of nine chunks, the last one short
        dict(name="prefill 133", kind="prefill", model="phi3", ctx=133, cap=1024),
        # mixture of experts: every expert in HBM
        dict(name="experts resident", kind="moe", model="olmoe4", ctx=190, cap=512, slots=64, tokens=4,
             policy="on_demand"),
        # half of the experts in HBM, copies ahead of time from the host
        dict(name="experts ahead of time", kind="moe", model="olmoe4", ctx=190, cap=512, slots=32, tokens=4,
             policy="ahead_of_time"),
    ]


def draw(rng):
    def log(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    def cap(ctx, most=8192):
        return min(most, max(ctx + 16, rng.choice([256, 1024, 2048, 4096, 8192])))

    kind = rng.choice(["tiny", "small", "step", "step", "exit", "flops", "batch", "batch", "spec", "prefill", "moe"])
    if kind == "tiny":
        ctx = log(1, 1000)
        return dict(kind="step", model="tiny", ctx=ctx, cap=ctx + 64, dual=rng.random() < 0.7, exits="all")
    if kind == "small":
        ctx = log(8, 2000)
        return dict(kind="batch", model="small", ctx=ctx, cap=ctx + 40, batch=rng.randint(1, 8), exits="every 2")
    if kind == "step":
        ctx = log(16, 8000)
        dual = rng.random() < 0.6
        return dict(kind="step", model="phi3", ctx=ctx, cap=cap(ctx), dual=dual,
                    exits=rng.choice(["all", "every 4"]) if dual else "off")
    if kind == "exit":
        ctx = log(16, 4000)
        return dict(kind="step", model="phi3", ctx=ctx, cap=cap(ctx, 4096), dual=True,
                    exits="exit %d" % rng.randint(16, 31))
    if kind == "flops":
        ctx = log(16, 4000)
        return dict(kind="step", model="phi3_flops", ctx=ctx, cap=cap(ctx, 4096), dual=True, exits="all")
    if kind == "batch":
        ctx = log(32, 4096)
        return dict(kind="batch", model="phi3", ctx=ctx, cap=cap(ctx, 4352), batch=rng.randint(2, 8),
                    exits=rng.choice(["every 1", "every 4"]))
    if kind == "spec":
        ctx = log(16, 4000)
        return dict(kind="spec", model="phi3", ctx=ctx, cap=cap(ctx, 4096), gamma=rng.randint(2, 10),
                    exit_layer=rng.randint(4, 12))
    if kind == "prefill":
        ctx = log(2, 144)
        return dict(kind="prefill", model="phi3", ctx=ctx, cap=cap(ctx, 4096))
    ctx = log(16, 2000)
    policy = rng.choice(["on_demand", "ahead_of_time"])
    return dict(kind="moe", model="olmoe4", ctx=ctx, cap=ctx + 64, slots=64 if policy == "on_demand" else 32, tokens=4,
                policy=policy)


# ---- what both the calls and the 64-bit results start from -------------------------------

def _shape(case):
    return MODELS[case["model"]]


def _gates(case, N):
    """(mode, gates, tau).  "every k": gates that no signal fires.  "exit b": gates at 4 and b; the threshold lies between the two signals,
    so the token leaves at b (a layer's relative update shrinks with depth)."""
    e = case.get("exits", "off")
    if e == "off":
        return "off", [], NEVER
    if e == "all":
        return "observe", list(range(1, N)), 0.9
    if e.startswith("every "):
        k = int(e.split()[1])
        return "observe", list(range(k, N, k)), NEVER
    return "exit", [4, int(e.split()[1])], 0.93


def _context(case, b):
    """Cached positions of sequence b of a batch: the case's, and shorter ones."""
    return max(1, case["ctx"] - b * case["ctx"] // (3 * case.get("batch", 1)))


def _generator(seed, stream):
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed) * 1000003 + stream)
    return g


def _weights(case, seed):
    """Every weight on the GPU, in its storage dtype (experts apart: _expert)."""
    m = _shape(case)
    dt = torch.bfloat16 if m["dt"] == "bf16" else torch.float32
    g = _generator(seed, 1)

    def mat(rows, cols):
        return torch.randn(rows, cols, generator=g, device="cuda", dtype=dt).mul_(0.02)

    def gain():
        return 1.0 + 0.1 * torch.randn(m["d"], generator=g, device="cuda")

    d, q, F, r = m["d"], m["H"] * m["hd"], m["F"], m["r"]
    moe, flops = "E" in m, "fh" in m
    w = dict(embed=mat(m["V"], d), final_norm=gain(), lm_head=mat(m["V"], d), layers=[])
    w["lm_head"] *= torch.exp(0.3 * torch.randn(m["V"], 1, generator=g, device="cuda")).to(dt)
    if flops:
        w["head_a"], w["head_b"] = mat(m["hr"], d), mat(m["V"], m["hr"])
    for _ in range(m["N"]):
        L = dict(attn_norm=gain(), mlp_norm=gain(), wq=mat(q, d), wk=mat(q, d), wv=mat(q, d), wo=mat(d, q))
        if moe:
            L["router"] = mat(m["E"], d)
        else:
            L["wg"], L["wu"], L["wd"] = mat(F, d), mat(F, d), mat(d, F)
        sides = [("q", d, q), ("k", d, q), ("v", d, q), ("o", q, d)]
        sides += [("m", d, d)] if moe or flops else [("g", d, F), ("u", d, F), ("d", F, d)]
        for p, din, dout in sides:
            L["A_" + p], L["B_" + p] = mat(r, din), mat(dout, r)
        w["layers"].append(L)
    return w


def _experts(case, seed, layer):
    """Gate, up ([E][Fe][d]) and down ([E][d][Fe]) of every expert of a layer."""
    m = _shape(case)
    g = _generator(seed, 100 + layer)
    return [torch.randn(m["E"], rows, cols, generator=g, device="cuda", dtype=torch.bfloat16).mul_(0.02)
            for rows, cols in ((m["Fe"], m["d"]), (m["Fe"], m["d"]), (m["d"], m["Fe"]))]


def _kv_bf16(m):
    return m.get("kv", m["dt"]) == "bf16"


def _written(case):
    """(sequence, position) of every cache entry that a pass writes."""
    if case["kind"] == "prefill":
        return [(0, i) for i in range(case["ctx"])]
    n = case["gamma"] + 1 if case["kind"] == "spec" else case.get("tokens", 1)
    return [(b, _context(case, b) + i) for b in range(case.get("batch", 1)) for i in range(n)]


def _pages(case, seed):
    """Keys and values ([N][blocks][H][16][hd]), the block table ([sequences][blocks]) and the number of blocks that a
    pass writes to.  Those are the first ones of the pages, the others are shuffled."""
    m = _shape(case)
    n_seqs, bps = case.get("batch", 1), (case["cap"] + 15) // 16
    dt = torch.bfloat16 if _kv_bf16(m) else torch.float32
    g = _generator(seed, 2)
    shape = (m["N"], n_seqs * bps, m["H"], 16, m["hd"])
    if case["kind"] == "prefill":
        k, v = (torch.zeros(shape, device="cuda", dtype=dt) for _ in range(2))
    else:
        k, v = (torch.randn(shape, generator=g, device="cuda", dtype=dt) for _ in range(2))
    first = sorted({b * bps + pos // 16 for b, pos in _written(case)})
    rest = np.setdiff1d(np.arange(n_seqs * bps), first)
    table = np.empty(n_seqs * bps, np.int32)
    table[first] = np.arange(len(first))
    table[rest] = len(first) + np.random.RandomState(int(seed) % (1 << 31)).permutation(len(rest))
    return k, v, table.reshape(n_seqs, bps), len(first)


def _tokens(case, seed, n):
    return torch.randint(0, _shape(case)["V"], (n,), generator=_generator(seed, 3), device="cuda", dtype=torch.int32)


# ---- the calls -----------------------------------------------------------------------------

def _call(name, *args):
    status = getattr(ab.lib(), name)(*args)
    if status:
        raise ab.M2R2Error(status, name)


class _Program:
    """What a serving program keeps: weights, context, cache and the buffers of its calls."""

    def __init__(self, case, seed):
        m = self.m = _shape(case)
        self.case = case
        dt, kv_dt = ab.BF16 if m["dt"] == "bf16" else ab.F32, ab.BF16 if _kv_bf16(m) else ab.F32
        flops = "fh" in m
        self.cfg = ab.Config(m["N"], m["d"], m["H"], m["hd"], m["F"], m["V"], m["r"], dt, kv_dt, EPS, THETA,
                             m.get("E", 0), m.get("K", 0), m.get("Fe", 0), case.get("slots", 0), m.get("fh", 0),
                             m.get("ftk", 0), int(flops), m.get("hr", 0))
        self.w = _weights(case, seed)
        layers = (ab.LayerWeights * m["N"])()
        for L, t in zip(layers, self.w["layers"]):
            for f in ("attn_norm", "mlp_norm", "wq", "wk", "wv", "wo", "wg", "wu", "wd", "router"):
                if f in t:
                    setattr(L, f, t[f].data_ptr())
            for i, p in enumerate(PROJ):
                if "A_" + p in t:
                    L.A[i], L.B[i] = t["A_" + p].data_ptr(), t["B_" + p].data_ptr()
            if "A_m" in t:
                L.A_m, L.B_m = t["A_m"].data_ptr(), t["B_m"].data_ptr()
        self.store = self._expert_store(seed) if "E" in m else None
        weights = ab.Weights(self.w["embed"].data_ptr(), self.w["final_norm"].data_ptr(), self.w["lm_head"].data_ptr(),
                             layers, self.store.data_ptr() if self.store is not None else None,
                             self.w["head_a"].data_ptr() if flops else None,
                             self.w["head_b"].data_ptr() if flops else None)
        sizes = (case.get("batch", 1), 16, case["cap"])
        need = ctypes.c_size_t(0)
        _call("m2r2_workspace_size", ctypes.byref(self.cfg), *sizes, ctypes.byref(need))
        self.workspace = torch.empty(need.value + 256, dtype=torch.uint8, device="cuda")
        self.ctx = ctypes.c_void_p()
        torch.cuda.synchronize()   # the context packs the weights on the null stream
        _call("m2r2_create", ctypes.byref(self.cfg), ctypes.byref(weights), *sizes,
              (self.workspace.data_ptr() + 255) & ~255, need.value, ctypes.byref(self.ctx))
        if self.store is not None:
            _call("m2r2_moe_set_policy", self.ctx, ab.POLICIES[case["policy"]])

        self.k, self.v, table, n = _pages(case, seed)
        self.table = torch.from_numpy(table).cuda()
        n_seqs, bps = table.shape
        self.seq_lens = torch.zeros(n_seqs, dtype=torch.int32, device="cuda")
        self.kv = ab.KV(self.k.data_ptr(), self.v.data_ptr(), self.table.data_ptr(), self.seq_lens.data_ptr(),
                        n_seqs * bps, 16, bps)
        self.out = dict(seq_lens=self.seq_lens, k=self.k[:, :n], v=self.v[:, :n])
        self._buffers(seed)
        self.stream = torch.cuda.current_stream().cuda_stream

    def _expert_store(self, seed):
        m = self.m
        size = ctypes.c_size_t(0)
        _call("m2r2_expert_bytes", ctypes.byref(self.cfg), ctypes.byref(size))
        size = size.value
        store = torch.empty(m["N"] * m["E"] * size, dtype=torch.uint8, pin_memory=True)
        with ThreadPoolExecutor(8) as pool:
            for layer in range(m["N"]):
                host = [torch.empty(t.shape, dtype=t.dtype, pin_memory=True).copy_(t)
                        for t in _experts(self.case, seed, layer)]

                def pack(e):
                    _call("m2r2_pack_expert", ctypes.byref(self.cfg), *(t[e].data_ptr() for t in host),
                          store.data_ptr() + (layer * m["E"] + e) * size)

                list(pool.map(pack, range(m["E"])))
        return store

    def _buffers(self, seed):
        case, m, kind = self.case, self.m, self.case["kind"]
        new = lambda *shape, dt=torch.int32: torch.zeros(shape, dtype=dt, device="cuda")  # noqa: E731
        f32 = torch.float32
        if kind in ("spec", "prefill"):
            n = case["gamma"] + 1 if kind == "spec" else case["ctx"]
            start = case["ctx"] if kind == "spec" else 0
            self.chunk = _tokens(case, seed, n)
            self.start, self.pos = torch.full((1,), start, dtype=torch.int32, device="cuda"), new(1)
            self.targets, self.accepted, self.bonus = new(16), new(1), new(1)
            if kind == "spec":
                self.out.update(chunk=self.chunk, targets=self.targets[:n], accepted=self.accepted, bonus=self.bonus)
            else:   # the targets of the last chunk
                self.out.update(targets=self.targets[: (n - 1) % 16 + 1])
            return
        mode, gates, tau = _gates(case, m["N"])
        self.dual = case.get("dual", True)
        self.gates_h = (ctypes.c_int32 * max(1, len(gates)))(*gates)
        self.exit = ab.Exit(ctypes.cast(self.gates_h, ctypes.POINTER(ctypes.c_int32)), len(gates), tau, ab.MODES[mode])
        B, T = case.get("batch", 1), case.get("tokens", 1)
        self.tokens = _tokens(case, seed, B * T)
        self.pos = torch.tensor([_context(case, b) + t for t in range(T) for b in range(B)], dtype=torch.int32).cuda()
        o = dict(token=new(T * B), logits=new(T * B, m["V"], dt=f32), h=new(T * B, m["d"], dt=f32))
        if self.dual:
            o["p"] = new(T * B, m["d"], dt=f32)
        if gates:
            o["boundary"], o["signal"] = new(T * B), new(T * B, m["N"], dt=f32)
        at = lambda name, t: o[name][t * B:].data_ptr() if name in o else None  # noqa: E731
        self.steps = [ab.StepOut(at("token", t), at("boundary", t), at("signal", t), at("logits", t), at("h", t),
                                 at("p", t), 0, None, None) for t in range(T)]
        self.out.update(o)

    def __del__(self):
        if getattr(self, "ctx", None) is not None and self.ctx.value:
            torch.cuda.synchronize()
            ab.lib().m2r2_destroy(self.ctx)
            self.ctx = ctypes.c_void_p()


def prepare(case, seed):
    return _Program(case, seed)


def run(p):
    kind, ref = p.case["kind"], ctypes.byref
    if kind == "spec":
        p.pos.copy_(p.start)   # (a pass is the same round again)
        _call("m2r2_draft", p.ctx, p.chunk.data_ptr(), p.pos.data_ptr(), p.case["exit_layer"], p.case["gamma"], ref(p.kv),
              p.chunk.data_ptr() + 4, p.stream)
        _call("m2r2_verify", p.ctx, p.chunk.data_ptr(), p.case["gamma"] + 1, p.pos.data_ptr(), ref(p.kv),
              p.targets.data_ptr(), p.accepted.data_ptr(), p.bonus.data_ptr(), p.stream)
    elif kind == "prefill":
        p.pos.copy_(p.start)
        for c in range(0, p.case["ctx"], 16):
            _call("m2r2_verify", p.ctx, p.chunk.data_ptr() + 4 * c, min(16, p.case["ctx"] - c), p.pos.data_ptr(),
                  ref(p.kv), p.targets.data_ptr(), None, None, p.stream)
    else:
        B = p.case.get("batch", 1)
        for t, out in enumerate(p.steps):
            _call("m2r2_decode_step", p.ctx, B, 1 if p.dual else 0, p.tokens.data_ptr() + 4 * B * t,
                  p.pos.data_ptr() + 4 * B * t, ref(p.kv), ref(p.exit), ref(out), p.stream)
    return p.out


# ---- what a pass cannot do without -----------------------------------------------------------

def work(case):
    """Every weight a call needs read once per call, every cached key and value once, results written once."""
    m = _shape(case)
    N, d, q, F, V, r = m["N"], m["d"], m["H"] * m["hd"], m["F"], m["V"], m["r"]
    ws, kvs = 2 if m["dt"] == "bf16" else 4, 2 if _kv_bf16(m) else 4
    kind, dual, flops = case["kind"], case.get("dual", True), "fh" in m
    attn = 4 * q * d
    mlp = 3 * d * F if "E" not in m else m["K"] * 3 * d * m["Fe"] + m["E"] * d
    adapters = r * (3 * (d + q) + q + d + (2 * d if "E" in m or flops else 3 * (d + F)))
    head = V * d
    b = f = 0

    def one(rows, seqs, layers, cached, new, heads, fast):
        """A call of `rows` rows over `seqs` sequences; it writes `new` cache entries and `heads` rows of logits."""
        nonlocal b, f
        b += ws * (layers * (attn + mlp + (adapters if fast else 0)) + head) + 4 * V * heads
        b += kvs * layers * 2 * q * (cached + new)
        f += 2 * rows * layers * (attn + mlp) + 2 * heads * head + 4 * rows * layers * q * cached / seqs

    if kind == "spec":
        for j in range(case["gamma"]):
            one(1, 1, case["exit_layer"], case["ctx"] + j, 1, 1, True)
        n = case["gamma"] + 1
        one(n, 1, N, case["ctx"], n, n, False)
    elif kind == "prefill":
        for c in range(0, case["ctx"], 16):
            n = min(16, case["ctx"] - c)
            one(n, 1, N, c, n, n, False)
    else:
        B = case.get("batch", 1)
        mode, gates, _ = _gates(case, N)
        run_layers = gates[-1] if mode == "exit" else N
        for t in range(case.get("tokens", 1)):
            cached = sum(_context(case, i) + t for i in range(B))
            one(2 * B if dual else B, B, run_layers, cached, B, B, dual)
        if run_layers < N:   # the other layers' cache entries only
            b += (N - run_layers) * (ws * 2 * q * d + kvs * 2 * q)
            f += 2 * (N - run_layers) * 2 * q * d
    return {"bytes": float(b), "flops": float(f)}


def tolerance(case):
    """float32 models: sums in another order.  bf16 models: keys and values rounded to the cache now and then fall
    on the other side of a rounding; in the FLOPs-optimised form a position at the edge of a head's selection
    falls on the other side of it."""
    if case["model"] == "tiny":
        return {"rel": 1e-5, "max": 1e-4}
    if case["model"] == "phi3_flops":
        return {"rel": 2e-2, "max": 0.3}
    if case["kind"] == "prefill":   # short contexts: such a rounding weighs more
        return {"rel": 1e-2, "max": 0.3}
    if case.get("batch", 1) == 8:   # at rank 16 the eighth fast row has been seen 2e-2 off the 64-bit result
        return {"rel": 2e-2, "max": 0.3}
    return {"rel": 4e-3, "max": 0.1}


# ---- the same in 64 bits, in plain torch ----------------------------------------------------------

def _norm(x, gain):
    return x * torch.rsqrt((x * x).mean(-1, keepdim=True) + EPS) * gain.double()


def _rope(x, pos):
    """Rotate-half embedding of x [..., H, hd] at the positions pos [...]."""
    half = x.shape[-1] // 2
    inv = THETA ** (-torch.arange(half, dtype=torch.float64, device=x.device) / half)
    a = pos.double()[..., None, None] * inv
    lo, hi = x[..., :half], x[..., half:]
    return torch.cat([lo * a.cos() - hi * a.sin(), hi * a.cos() + lo * a.sin()], -1)


def _attend(q, K, V):
    """q [H][hd] over K, V [T][H][hd]."""
    s = (K * q).sum(-1) / math.sqrt(q.shape[-1])
    return (torch.softmax(s, 0)[..., None] * V).sum(0)


class _Exact:
    def __init__(self, case, seed):
        self.case, self.m, self.seed = case, _shape(case), seed
        self.w = _weights(case, seed)
        self.k, self.v, self.table, self.n = _pages(case, seed)
        self.kv_dt = self.k.dtype
        self.experts = {}

    def mul(self, L, p, x, fast, name=None):
        """x times a projection's transpose, plus its adapter on a fast row."""
        y = x @ L[name or "w" + p].double().T
        return y + (x @ L["A_" + p].double().T) @ L["B_" + p].double().T if fast and "A_" + p in L else y

    def cache(self, l, seq, n):
        """Cached keys and values [n][H][hd] of a sequence's first n positions."""
        at = torch.from_numpy(self.table[seq][: (n + 15) // 16].astype(np.int64)).cuda()
        return [t[l, at].double().transpose(1, 2).reshape(-1, self.m["H"], self.m["hd"])[:n] for t in (self.k, self.v)]

    def write(self, l, seq, pos, k, v):
        at = int(self.table[seq, pos // 16])
        self.k[l, at, :, pos % 16] = k.to(self.kv_dt)
        self.v[l, at, :, pos % 16] = v.to(self.kv_dt)

    def qkv(self, L, x, pos, fast):
        u = _norm(x, L["attn_norm"])
        q, k, v = (self.mul(L, p, u, fast).reshape(*x.shape[:-1], self.m["H"], self.m["hd"]) for p in "qkv")
        return _rope(q, pos), _rope(k, pos), v

    def mlp(self, l, x, fast):
        L, m = self.w["layers"][l], self.m
        u = _norm(x, L["mlp_norm"])
        if fast and "A_m" in L:
            return (u @ L["A_m"].double().T) @ L["B_m"].double().T
        if "E" not in m:
            a = torch.nn.functional.silu(self.mul(L, "g", u, fast)) * self.mul(L, "u", u, fast)
            return self.mul(L, "d", a, fast)
        if l not in self.experts:
            self.experts[l] = _experts(self.case, self.seed, l)
        wg, wu, wd = self.experts[l]
        prob = torch.softmax(L["router"].double() @ u, 0)
        y = torch.zeros_like(x)
        for e in torch.topk(prob, m["K"]).indices.tolist():
            y += prob[e] * (wd[e].double() @ (torch.nn.functional.silu(wg[e].double() @ u) * (wu[e].double() @ u)))
        return y

    def out(self, L, o, fast):
        return self.mul(L, "o", o.reshape(*o.shape[:-2], -1), fast)

    def head(self, x):
        return _norm(x, self.w["final_norm"]) @ self.w["lm_head"].double().T

    def slow_chunk(self, l, x, seq, pos0):
        """One layer of the slow stream on rows x [n][d] at pos0.. (causal)."""
        L, n = self.w["layers"][l], x.shape[0]
        q, k, v = self.qkv(L, x, pos0 + torch.arange(n, device="cuda"), False)
        for i in range(n):
            self.write(l, seq, pos0 + i, k[i], v[i])
        K, V = self.cache(l, seq, pos0 + n)
        o = torch.stack([_attend(q[i], K[: pos0 + i + 1], V[: pos0 + i + 1]) for i in range(n)])
        x = x + self.out(L, o, False)
        return x + torch.stack([self.mlp(l, r, False) for r in x]) if "E" in self.m else x + self.mlp(l, x, False)

    def fast(self, l, p, h, seq, pos, extra=()):
        """One layer of the fast stream; `extra`: keys and values of earlier fast positions."""
        L, m = self.w["layers"][l], self.m
        q, k, v = self.qkv(L, p, torch.tensor(pos, device="cuda"), True)
        K, V = self.cache(l, seq, pos - len(extra))
        K = torch.cat([K] + [e[0][None] for e in extra] + [k[None]])
        V = torch.cat([V] + [e[1][None] for e in extra] + [v[None]])
        if "fh" in m:
            qs, _, _ = self.qkv(L, h, torch.tensor(pos, device="cuda"), False)
            o = torch.zeros_like(q)
            score = (K[:-1] * qs).sum(-1)
            for j in range(m["fh"]):
                keep = torch.arange(pos, device="cuda")
                if pos > m["ftk"]:
                    keep = torch.topk(score[:, j], m["ftk"]).indices
                keep = torch.cat([keep, torch.tensor([pos], device="cuda")])
                o[j] = _attend(q[j][None], K[keep, j][:, None], V[keep, j][:, None])[0]
        else:
            o = _attend(q, K, V)
        p = p + self.out(L, o, True)
        return p + self.mlp(l, p, True), (k, v)

    def step(self, token, seq, pos, dual):
        N = self.m["N"]
        mode, gates, tau = _gates(self.case, N)
        h = self.w["embed"][token].double()
        p, signal = h.clone(), torch.zeros(N, dtype=torch.float64, device="cuda")
        for l in range(N):
            if dual:
                before = p
                p, _ = self.fast(l, p, h, seq, pos)
                signal[l] = torch.nn.functional.cosine_similarity(before, p, 0, 0.0)
            h = self.slow_chunk(l, h[None], seq, pos)[0]
            if l + 1 in gates:
                if mode == "exit" and float(signal[l]) >= tau:
                    for rest in range(l + 1, N):
                        _, k, v = self.qkv(self.w["layers"][rest], h, torch.tensor(pos, device="cuda"), False)
                        self.write(rest, seq, pos, k, v)
                    return self.head(p), h, p, signal
                p = h
        return self.head(h), h, p, signal


def exact(case, seed):
    x, m = _Exact(case, seed), _shape(case)
    if case["kind"] == "spec":
        chunk, t = _tokens(case, seed, case["gamma"] + 1).tolist(), case["ctx"]
        extra = [[] for _ in range(case["exit_layer"])]
        for j in range(case["gamma"]):
            p = x.w["embed"][chunk[j]].double()
            for l, e in enumerate(extra):
                p, (k, v) = x.fast(l, p, None, 0, t + j, e)
                e.append((k.to(x.kv_dt).double(), v.to(x.kv_dt).double()))
            chunk[j + 1] = int(x.head(p).argmax())
        rows = x.w["embed"][torch.tensor(chunk, device="cuda")].double()
        for l in range(m["N"]):
            rows = x.slow_chunk(l, rows, 0, t)
        return dict(chunk=None, targets=None, accepted=None, bonus=None, seq_lens=None, k=x.k[:, :x.n], v=x.v[:, :x.n])
    if case["kind"] == "prefill":
        rows = x.w["embed"][_tokens(case, seed, case["ctx"]).long()].double()
        for l in range(m["N"]):
            rows = x.slow_chunk(l, rows, 0, 0)
        return dict(targets=None, seq_lens=None, k=x.k[:, :x.n], v=x.v[:, :x.n])
    B, T, dual = case.get("batch", 1), case.get("tokens", 1), case.get("dual", True)
    tokens, rows = _tokens(case, seed, B * T).tolist(), []
    for t in range(T):
        for b in range(B):
            rows.append(x.step(tokens[t * B + b], b, _context(case, b) + t, dual))
    got = {n: torch.stack([r[i] for r in rows]) for i, n in enumerate(("logits", "h", "p", "signal"))}
    res = dict(token=None, logits=got["logits"], h=got["h"], seq_lens=None, k=x.k[:, :x.n], v=x.v[:, :x.n])
    if dual:
        res["p"] = got["p"]
    if _gates(case, m["N"])[1]:
        res["boundary"], res["signal"] = None, got["signal"]
    return res
