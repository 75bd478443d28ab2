"""Batched decoding and chunks at the sizes where their kernels can go wrong
(rows, ranks and context lengths at the edges of tiles and splits), against
the oracle under the rule of ``gpu_harness``."""
import copy

import numpy as np
import pytest
import torch

import synth
from tests.gpu_harness import Pair, Tally

pytestmark = pytest.mark.gpu


def batch_step(pair: Pair, lens, t: Tally, *, tol=None, seed=3, mode="observe", gates=None, pick=None):
    """One dual step of sequences with random cache content of the given
    lengths: logits, h, p, signal, token and the new cache entries.  EXIT mode:
    pick(sorted signals at the first gate) is the threshold.  Returns how many
    sequences exited."""
    cfg, B, dev, tol = pair.cfg, len(lens), pair.dev, tol or pair.tol
    N = cfg.n_layers
    for s, n in enumerate(lens):
        for l, (K, V) in synth.synthetic_kv(cfg, n, seq=s).items():
            if n:
                pair.kv.load(s, l, K, V)
                pair.caches[s].load(l, K, V)
    toks = synth.prompt_ids(cfg, B, seed=seed)
    out = {k: torch.zeros(B * n, dtype=torch.float32, device=dev)
           for k, n in (("signal", N), ("logits", cfg.vocab), ("h_out", cfg.d_model), ("p_out", cfg.d_model))}
    nxt = torch.zeros(B, dtype=torch.int32, device=dev)
    gates, tau = gates or list(range(1, N)), 0.9
    if pick:
        obs = [pair.orc.decode_step(int(toks[s]), n, copy.deepcopy(pair.caches[s]), gates=gates, tau=2.0,
                                    mode="observe") for s, n in enumerate(lens)]
        tau = pick(sorted(r.signal[gates[0] - 1] for r in obs))
        assert all(abs(r.signal[b - 1] - tau) > tol for r in obs for b in gates), "no clear threshold"
    exits = 0
    pair.model.decode_step(torch.tensor(toks, dtype=torch.int32, device=dev),
                           torch.tensor(lens, dtype=torch.int32, device=dev), pair.kv.desc(), gates=gates, tau=tau,
                           mode=mode, next_token=nxt, **out)
    torch.cuda.synchronize()
    got = {k: v.cpu().numpy().reshape(B, -1) for k, v in out.items()}
    for s, n in enumerate(lens):
        r = pair.orc.decode_step(int(toks[s]), n, pair.caches[s], gates=gates, tau=tau, mode=mode)
        last = r.exit_boundary if mode == "exit" else N
        exits += last < N
        t.rel(got["logits"][s], r.logits, tol, f"seq {s} logits")
        t.rel(got["h_out"][s], r.h, tol, f"seq {s} h")
        t.rel(got["p_out"][s], r.p, tol, f"seq {s} p")
        t.close(got["signal"][s][:last], r.signal[:last], tol, f"seq {s} signal")
        t.token(int(nxt[s].item()), r.logits, tol, f"seq {s} token")
        pair.check_cache(s, n, n + 1, t, f"seq {s}")
        t.steps += 1
    return exits


@pytest.mark.parametrize("rank,B", [(16, 8), (32, 4), (32, 8)])
def test_more_adapter_sums_than_threads(rank, B):
    """Ranks at which the gate/up kernel's rows x (1 + 2 rank) adapter sums
    outnumber its 512 threads (float32 weights: 1e-4)."""
    cfg = synth.CONFIGS["tiny"].replace(name=f"tiny_r{rank}", rank=rank)
    pair = Pair(cfg, synth.make_weights(cfg), max_ctx=64, max_batch=B, n_seqs=B, table_seed=7)
    t = Tally()
    batch_step(pair, [5, 19, 37, 2, 11, 30, 8, 23][:B], t)
    assert t.steps == B and t.arrays >= 6 * B


# head_dim 64, 96 and 128 with a bfloat16 cache; float32 weights too
MF_CONFIGS = {
    "hd64": synth.CONFIGS["tiny"].replace(name="hd64", kvdtype="bf16"),
    "hd96": synth.CONFIGS["small_bf16"],
    "hd128": synth.CONFIGS["small_rw"],
}


@pytest.mark.parametrize("name", MF_CONFIGS)
@pytest.mark.parametrize("block_size", [1, 16, 24])
@pytest.mark.parametrize("lens", [(0, 1, 31, 32, 33), (127, 128, 129), (255, 257, 300, 511, 640, 2, 16, 1000)])
def test_batch_attention_context_edges(name, block_size, lens):
    """Contexts at the edges of the matrix-core attention's tiles (32 tokens),
    waves and splits (128 tokens), pages of one, 16 and 24 tokens."""
    cfg = MF_CONFIGS[name]
    pair = Pair(cfg, synth.make_weights(cfg), max_ctx=max(lens) + 20, block_size=block_size, max_batch=len(lens),
                n_seqs=len(lens), table_seed=11)
    t = Tally()
    # a cached value on the other side of a bfloat16 rounding is 2^-8 of itself
    batch_step(pair, lens, t, tol=2e-2)
    assert t.steps == len(lens)


@pytest.mark.parametrize("name", MF_CONFIGS)
@pytest.mark.parametrize("ctx,n", [(0, 3), (0, 16), (1, 15), (31, 7), (128, 9), (129, 16), (700, 5), (1000, 16)])
def test_chunk_attention_context_edges(name, ctx, n):
    """A chunk of n slow rows after ctx cached positions: targets and the
    chunk's cache entries in every layer."""
    chunk(MF_CONFIGS[name], ctx, n, ctx + 40)


def chunk(cfg, ctx, n, cap):
    pair = Pair(cfg, synth.make_weights(cfg), max_ctx=cap, block_size=16, table_seed=13)
    # float32 weights with a bfloat16 cache: a value whose rounding falls on
    # the other side is one unit in the last place off, at most 2^-7 of itself
    pair.tol = max(pair.tol, 2.0 ** -7)
    t = Tally()
    if ctx:
        for l, (K, V) in synth.synthetic_kv(cfg, ctx).items():
            pair.kv.load(0, l, K, V)
            pair.caches[0].load(l, K, V)
    toks = [int(x) for x in synth.prompt_ids(cfg, n, seed=9)]
    dev = pair.dev
    pos, targets = torch.tensor([ctx], dtype=torch.int32, device=dev), torch.zeros(16, dtype=torch.int32, device=dev)
    pair.model.verify(torch.tensor(toks, dtype=torch.int32, device=dev), n, pos, pair.kv.desc(), targets)
    torch.cuda.synchronize()
    ref = pair.orc.slow_chunk(toks, ctx, pair.caches[0])
    for i in range(n):
        t.token(int(targets[i].item()), ref[i], pair.tol, f"row {i}")
    pair.check_cache(0, ctx, ctx + n, t)
    assert int(pos.item()) == ctx + n == int(pair.kv.seq_lens[0].item())


@pytest.mark.parametrize("name,ctx,cap", [
    # one split up to 64 positions, then one per head's share of the workgroups; 256 positions per pass
    *[("tiny", n, 300) for n in (0, 1, 63, 64, 65, 257)],
    # float32 on one workgroup per compute unit: capacities of one split, and above 4096
    *[("tiny", n, 64) for n in (0, 63)], *[("tiny", n, 4200) for n in (10, 65, 4100)],
    *[("small_rw", n, 300) for n in (0, 31, 64, 65, 257)],
    ("small_rw", 1025, 2048),
    # more than 63 splits of 128 positions; more than 1024 positions per split
    ("small_rw", 8100, 8200),
    ("small_rw", 16600, 16700),
    # matrices of fewer blocks than the stream-K kernels take: short-chain attention with per-tile projections
    ("hd96_f32cache", 130, 200),
])
def test_one_sequence_context_edges(name, ctx, cap):
    """One sequence's dual step at the edges of the attention's splits."""
    cfg = (synth.CONFIGS["small_bf16"].replace(name=name, kvdtype="f32") if name == "hd96_f32cache"
           else synth.CONFIGS[name])
    pair = Pair(cfg, synth.make_weights(cfg), max_ctx=cap, table_seed=17)
    t = Tally()
    batch_step(pair, [ctx], t)
    assert t.steps == 1


@pytest.mark.parametrize("name", ["small_bf16", "small_rw"])
@pytest.mark.parametrize("lens", [(5, 40, 17), (130, 1, 64, 33, 90, 12, 7, 257)])
def test_batch_exits(name, lens):
    """EXIT mode with every sequence, and with a part of them, gone at a gate:
    their skipped layers' keys and values come from the slow row, their rows
    stay as they are, and the others go on."""
    cfg = synth.CONFIGS[name]
    n = len(lens)
    widest = lambda v: max(range(n - 1), key=lambda i: v[i + 1] - v[i])   # noqa: E731
    for pick, gates, want in ((lambda v: -2.0, [1], lambda e: e == n),
                              (lambda v: (v[widest(v)] + v[widest(v) + 1]) / 2, [2], lambda e: 0 < e < n)):
        pair = Pair(cfg, synth.make_weights(cfg), max_ctx=max(lens) + 20, max_batch=n, n_seqs=n, table_seed=19)
        t = Tally()
        # the least tolerance that decides every signal here: 2^-8 is one bfloat16 rounding
        assert want(batch_step(pair, lens, t, tol=2.0 ** -8, mode="exit", gates=gates, pick=pick))
        assert t.steps == n


@pytest.mark.parametrize("ffn", [3072, 4096, 5120, 8192])
@pytest.mark.parametrize("d,B", [(192, 5), (224, 8), (512, 7)])
def test_long_down_reductions(ffn, d, B):
    """Down projections of 9 and more rows whose reduction is split over
    workgroups (and one that is not): tiles in whole groups of four, a group of
    two, an odd number of groups."""
    cfg = synth.CONFIGS["small_bf16"].replace(name=f"ffn{ffn}_{d}", d_model=d, ffn=ffn, n_layers=2)
    pair = Pair(cfg, synth.make_weights(cfg), max_ctx=80, max_batch=B, n_seqs=B, table_seed=23)
    t = Tally()
    batch_step(pair, [3, 40, 17, 0, 65, 33, 9, 21][:B], t)
    batch_step(pair, [4, 41, 18, 1, 66, 34, 10, 22][:B], t)   # counters back at zero
    assert t.steps == 2 * B


@pytest.mark.parametrize("name,ctx,block_size", [
    *[("tiny", n, 16) for n in (0, 1, 63, 64, 65)],
    *[("small_rw", n, 16) for n in (0, 1, 63, 64, 65, 200)],
    ("small_rw", 600, 1),      # block tables of more entries than the selection kernel has threads
])
def test_flops_whole_selection(name, ctx, block_size):
    """The FLOPs-optimised form with a selection that keeps every position (no
    ties to decide), at the edges of the selected positions' passes of 64."""
    cfg = synth.CONFIGS[name].replace(name=f"{name}_all", fast_heads=2, fast_topk=4096, fast_mlp_adapter=True,
                                      head_rank=16)
    pair = Pair(cfg, synth.make_weights(cfg), max_ctx=ctx + 20, block_size=block_size, table_seed=29)
    t = Tally()
    batch_step(pair, [ctx], t)
    assert t.steps == 1


@pytest.mark.parametrize("name", ["hd64", "hd96", "hd128", "tiny"])
@pytest.mark.parametrize("lens", [(5,), (200,), (5, 200, 33)])
def test_overflowing_fast_row_leaves_the_slow_row(name, lens):
    """A fast row whose own value overflows: no slow row sees it."""
    cfg = {**MF_CONFIGS, "tiny": synth.CONFIGS["tiny"]}[name]
    plain = synth.make_weights(cfg)
    big = {k: (100 * v if k.endswith(".A_v") else np.full_like(v, 2.0 ** 127) if k.endswith(".B_v") else v)
           for k, v in plain.items()}
    pair, t, n = Pair(cfg, big, max_ctx=256, max_batch=len(lens), n_seqs=len(lens), table_seed=31), Tally(), len(lens)
    orc = Pair(cfg, plain, max_ctx=256).orc
    for s, m in enumerate(lens):
        for l, (K, V) in synth.synthetic_kv(cfg, m, seq=s).items():
            pair.kv.load(s, l, K, V)
            pair.caches[s].load(l, K, V)
    toks = synth.prompt_ids(cfg, n, seed=3)
    h, z = (torch.zeros(n * w, dtype=torch.float32, device=pair.dev) for w in (cfg.d_model, cfg.vocab))
    nxt = torch.zeros(n, dtype=torch.int32, device=pair.dev)
    pair.model.decode_step(torch.tensor(toks, dtype=torch.int32, device=pair.dev),
                           torch.tensor(lens, dtype=torch.int32, device=pair.dev), pair.kv.desc(), gates=[1], tau=2.0,
                           mode="observe", next_token=nxt, h_out=h, logits=z)
    torch.cuda.synchronize()
    for s, m in enumerate(lens):
        r = orc.decode_step(int(toks[s]), m, pair.caches[s], gates=[1], tau=2.0, mode="observe")
        # a cached value on the other side of a bfloat16 rounding is 2^-8 of itself
        t.rel(h.cpu().numpy().reshape(n, -1)[s], r.h, 2e-2, f"seq {s} h")
        t.rel(z.cpu().numpy().reshape(n, -1)[s], r.logits, 2e-2, f"seq {s} logits")
        t.steps += 1
    assert t.steps == n


@pytest.mark.parametrize("name", MF_CONFIGS)
@pytest.mark.parametrize("n,bad", [(2, 1), (9, 6), (16, 15)])
def test_overflowing_chunk_row_leaves_the_rows_before_it(name, n, bad):
    """A chunk row of infinite values reaches no row before it."""
    cfg = MF_CONFIGS[name]
    w, ctx = synth.make_weights(cfg), 40
    toks = [i + 1 for i in range(n)]
    w["embed"] = w["embed"].copy()
    w["embed"][toks[bad]] = np.inf
    pair, t = Pair(cfg, w, max_ctx=80, table_seed=37), Tally()
    pair.tol = max(pair.tol, 2.0 ** -7)   # (one unit in the last place of a cached value)
    for l, (K, V) in synth.synthetic_kv(cfg, ctx).items():
        pair.kv.load(0, l, K, V)
        pair.caches[0].load(l, K, V)
    pos = torch.tensor([ctx], dtype=torch.int32, device=pair.dev)
    targets = torch.zeros(16, dtype=torch.int32, device=pair.dev)
    pair.model.verify(torch.tensor(toks, dtype=torch.int32, device=pair.dev), n, pos, pair.kv.desc(), targets)
    torch.cuda.synchronize()
    ref = pair.orc.slow_chunk(toks[:bad], ctx, pair.caches[0])
    for i in range(bad):
        t.token(int(targets[i].item()), ref[i], pair.tol, f"row {i}")
    pair.check_cache(0, ctx, ctx + bad, t)
    assert t.arrays == 2 * cfg.n_layers
    for l in range(cfg.n_layers):
        assert not np.isfinite(pair.kv.read(0, l, ctx + bad, ctx + bad + 1)[1]).any()


def test_attention_chunks_switch_beyond_its_capacity(monkeypatch):
    """Two chunks per split asked for at a capacity of more splits than the
    short-chain attention holds (64): the general attention serves it."""
    monkeypatch.setenv("M2R2_ATTN_CHUNKS", "2")
    monkeypatch.setenv("M2R2_ONE_LAUNCH", "0")
    cfg = synth.CONFIGS["small_rw"]
    pair = Pair(cfg, synth.make_weights(cfg), max_ctx=16700, table_seed=41)
    t = Tally()
    batch_step(pair, [16600], t)
    assert t.steps == 1


# few heads and capacities of more than 63 splits of 128 positions
@pytest.mark.parametrize("name", ["hd64", "hd96"])
@pytest.mark.parametrize("cap,lens", [(8200, (8100, 60)), (16700, (16600, 8191, 1))])
def test_batch_attention_large_capacities(name, cap, lens):
    cfg = MF_CONFIGS[name].replace(name=f"{name}_1", n_layers=1)
    pair = Pair(cfg, synth.make_weights(cfg), max_ctx=cap, max_batch=len(lens), n_seqs=len(lens), table_seed=43)
    t = Tally()
    batch_step(pair, lens, t, tol=2e-2)
    assert t.steps == len(lens)


@pytest.mark.parametrize("name", MF_CONFIGS)
@pytest.mark.parametrize("ctx,cap", [(8100, 8200), (16600, 16700)])
def test_chunk_attention_large_capacities(name, ctx, cap):
    """16 rows behind more positions than 63 splits of the general attention
    hold scores of (256 positions each)."""
    chunk(MF_CONFIGS[name].replace(name=f"{name}_1", n_layers=1), ctx, 16, cap)


def wide(hd, heads):
    """One layer of many heads: few splits, so a wave takes several tiles."""
    return synth.ModelConfig(f"wide{hd}_{heads}", n_layers=1, d_model=512, n_heads=heads, head_dim=hd, ffn=512, vocab=300,
                             rank=8, wdtype="bf16", kvdtype="bf16", seed=47)


# (capacities at which the kernel's LDS, with the row table of a split, is above 64 KB)
@pytest.mark.parametrize("hd,heads,cap", [(64, 32, 2048), (96, 32, 2048), (128, 32, 32768)])
def test_batch_attention_long_splits(hd, heads, cap):
    """Eight sequences on four splits: two to four tiles per wave, an odd
    number of them, a masked last one after full ones."""
    cfg, lens = wide(hd, heads), (129, 160, 257, 289, 700, 1000, 1025, 1537)
    pair = Pair(cfg, synth.make_weights(cfg), max_ctx=cap, max_batch=8, n_seqs=8, table_seed=53)
    t = Tally()
    batch_step(pair, lens, t)
    assert t.steps == 8


@pytest.mark.parametrize("hd,heads,cap,ctx,n", [(64, 64, 3000, 2600, 5), (96, 64, 5000, 4200, 9),
                                                (128, 64, 40000, 4200, 16)])
def test_chunk_attention_long_splits(hd, heads, cap, ctx, n):
    """Chunks on 16 splits: up to three tiles per wave."""
    chunk(wide(hd, heads), ctx, n, cap)


@pytest.mark.filterwarnings("ignore::RuntimeWarning")   # (the oracle's infinite scores)
@pytest.mark.parametrize("name", [*MF_CONFIGS, "tiny"])
@pytest.mark.parametrize("lens", [(5,), (200,), (700,), (5, 200, 700)])
def test_infinite_cached_key(name, lens):
    """One infinite element of a cached key: the position has weight zero where
    the score is minus infinity; the other rows are not finite."""
    cfg = {**MF_CONFIGS, "tiny": synth.CONFIGS["tiny"]}[name].replace(n_layers=1)
    w, n = synth.make_weights(cfg), len(lens)
    toks, seen = synth.prompt_ids(cfg, n, seed=3), 0
    for inf in (np.inf, -np.inf):
        pair, t = Pair(cfg, w, max_ctx=max(lens) + 20, max_batch=n, n_seqs=n, table_seed=59), Tally()
        for s, m in enumerate(lens):
            for l, (K, V) in synth.synthetic_kv(cfg, m, seq=s).items():
                K = K.copy()
                K[m // 2, 1, 7] = inf
                pair.kv.load(s, l, K, V)
                pair.caches[s].load(l, K, V)
        h, p, z = (torch.zeros(n * k, dtype=torch.float32, device=pair.dev)
                   for k in (cfg.d_model, cfg.d_model, cfg.vocab))
        nxt = torch.zeros(n, dtype=torch.int32, device=pair.dev)
        pair.model.decode_step(torch.tensor(toks, dtype=torch.int32, device=pair.dev),
                               torch.tensor(lens, dtype=torch.int32, device=pair.dev), pair.kv.desc(), gates=[], tau=2.0,
                               mode="observe", next_token=nxt, h_out=h, p_out=p, logits=z)
        torch.cuda.synchronize()
        for s, m in enumerate(lens):
            r = pair.orc.decode_step(int(toks[s]), m, pair.caches[s], gates=[], tau=2.0, mode="observe")
            for got, ref, what in ((h, r.h, "h"), (p, r.p, "p"), (z, r.logits, "logits")):
                got = got.cpu().numpy().reshape(n, -1)[s]
                if np.isfinite(ref).all():
                    t.rel(got, ref, 2e-2, f"seq {s} {what}")   # (a rounding of a cached value)
                    seen += 1
                else:
                    assert not np.isfinite(got).any(), f"seq {s} {what}"
    assert seen >= 2 * n   # (a slow row's h and logits with one of the signs)


@pytest.mark.filterwarnings("ignore::RuntimeWarning")
@pytest.mark.parametrize("name", MF_CONFIGS)
@pytest.mark.parametrize("ctx", [5, 700])
def test_infinite_cached_key_chunk(name, ctx):
    """The same for the rows of a chunk (one layer: a row that is not finite reaches no other)."""
    cfg = MF_CONFIGS[name].replace(n_layers=1)
    pair, t, n = Pair(cfg, synth.make_weights(cfg), max_ctx=ctx + 20, table_seed=61), Tally(), 16
    for l, (K, V) in synth.synthetic_kv(cfg, ctx).items():
        K = K.copy()
        K[ctx // 2, 1, 7] = np.inf
        pair.kv.load(0, l, K, V)
        pair.caches[0].load(l, K, V)
    toks = [int(x) for x in synth.prompt_ids(cfg, n, seed=9)]
    pos = torch.tensor([ctx], dtype=torch.int32, device=pair.dev)
    targets = torch.zeros(16, dtype=torch.int32, device=pair.dev)
    pair.model.verify(torch.tensor(toks, dtype=torch.int32, device=pair.dev), n, pos, pair.kv.desc(), targets)
    torch.cuda.synchronize()
    ref = pair.orc.slow_chunk(toks, ctx, pair.caches[0])
    finite = [i for i in range(n) if np.isfinite(ref[i]).all()]
    for i in finite:
        t.token(int(targets[i].item()), ref[i], pair.tol, f"row {i}")
    assert 0 < len(finite) < n and t.compared > 0


@pytest.mark.parametrize("n", [3, 8, 9, 16])
def test_head_of_infinitely_low_logits(n):
    """Every logit overflows to minus infinity: the arg-max is the lowest id."""
    cfg = synth.CONFIGS["small_bf16"].replace(n_layers=1)
    w = {k: v.copy() for k, v in synth.make_weights(cfg).items()}
    for k in w:
        if k.endswith(".wo") or k.endswith(".wd"):
            w[k][:] = 0   # the head's input is the embedding
    w["embed"][:, 0], w["lm_head"][:, 0] = 1, -(2.0 ** 127)
    w["final_norm"][:] = 0
    w["final_norm"][0] = 16
    pair = Pair(cfg, w, max_ctx=32)
    pos = torch.zeros(1, dtype=torch.int32, device=pair.dev)
    targets = torch.full((16,), -1, dtype=torch.int32, device=pair.dev)
    toks = [int(x) for x in synth.prompt_ids(cfg, n, seed=9)]
    pair.model.verify(torch.tensor(toks, dtype=torch.int32, device=pair.dev), n, pos, pair.kv.desc(), targets)
    torch.cuda.synchronize()
    assert targets[:n].tolist() == [0] * n


@pytest.mark.parametrize("d", [512, 544, 768, 1024, 1056, 1536])
@pytest.mark.parametrize("B", [3, 8])
def test_reduction_lengths(d, B):
    """Projections whose waves have 2, 3, 4, 5 and 6 steps of the reduction,
    whole and ragged: the edges of the resident instantiations."""
    cfg = synth.CONFIGS["small_bf16"].replace(name=f"d{d}", d_model=d, ffn=d, n_layers=2)
    pair = Pair(cfg, synth.make_weights(cfg), max_ctx=80, max_batch=B, n_seqs=B, table_seed=67)
    t = Tally()
    batch_step(pair, [3, 40, 17, 0, 65, 33, 9, 21][:B], t)
    assert t.steps == B


# q/k/v of 3072 rows per matrix, o and down of 3072 rows, on 256 compute units: tiles of 12 rows
TILE12 = {"qkv": wide(96, 32).replace(name="qkv12"), "o_down": wide(128, 4).replace(name="o_down12", d_model=3072)}


@pytest.mark.parametrize("name", TILE12)
@pytest.mark.parametrize("B", [2, 3, 8])
def test_batch_on_tiles_of_12_rows(name, B):
    cfg = TILE12[name]
    pair = Pair(cfg, synth.make_weights(cfg), max_ctx=80, max_batch=B, n_seqs=B, table_seed=71)
    t = Tally()
    batch_step(pair, [3, 40, 17, 0, 65, 33, 9, 21][:B], t)
    assert t.steps == B


@pytest.mark.parametrize("name", TILE12)
@pytest.mark.parametrize("n", [3, 16])
def test_chunk_on_tiles_of_12_rows(name, n):
    chunk(TILE12[name], 40, n, 80)


@pytest.mark.parametrize("rank,ctx", [(8, 0), (8, 33), (8, 200), (4, 33), (12, 33)])
@pytest.mark.parametrize("wdtype,kvdtype", [("bf16", "bf16"), ("bf16", "f32"), ("f32", "f32")])
def test_one_sequence_on_the_stream_k_projections(rank, ctx, wdtype, kvdtype):
    """Rows that are no whole 1 KB pieces, at least eight blocks each; ranks
    whose adapter rows are no whole 16 bytes."""
    cfg = synth.CONFIGS["small_bf16"].replace(name=f"streamk{rank}", d_model=544, n_heads=3, ffn=608, rank=rank,
                                              wdtype=wdtype, kvdtype=kvdtype)
    pair = Pair(cfg, synth.make_weights(cfg), max_ctx=256, table_seed=73)
    t = Tally()
    batch_step(pair, [ctx], t, tol=2e-2 if kvdtype == "bf16" else 1e-3)
    assert t.steps == 1
