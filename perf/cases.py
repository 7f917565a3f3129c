"""The work this library is used for, as cases that can be timed and compared.

Every case goes through the package's public entry points (paper_2511_22880_amd.binding), with inputs a
serving process would have in hand: adapters loaded into the pools, the segment objects planned, x and
y in device memory.  Sizes are those of the repository's benchmark configurations (workloads.py) or
generic ones of the same ranges.

A case is a dict.  `kind` says what one pass does:
  apply   lora_apply of one projection on `layers` pools in turn; with `rebuild` the batch is planned
          and its table uploaded first (lora_segments_rebuild), as once per step of a serving loop
  layers  the same for whole layers: q|k|v and gate|up through lora_apply_multi, o and down through
          lora_apply (`in` = hidden size, `kv` = k and v size, `out` = inner size of the MLP)
  shard   lora_shrink, then lora_expand: the two halves apart, as a row-parallel shard calls them
          (v leaves as fp32 for the exchange between the ranks, and comes back)
  linear  lora_linear: the frozen layer with the delta in its epilogue
  load    lora_pool_load of `adapters` adapters, from device memory, or (`host`) lora_pool_load_staged
          from pinned host memory: adapters arriving at a server
The batch: `prompts` prefill requests (lengths lognormal, median `median`, `sigma`; sigma 0: all of
that length) and `decode` tokens of one request each, a share `idle` of the requests without an
adapter.  `own`: request i uses adapter i; else adapters are drawn with P(k) ~ (k + 1)^-alpha.
`ranks`: "mixed" = {8, 16, 32, 64, 128} in equal shares, "skew" = half 8, half 256, "odd" = anything
from 1 to 256, or one number.  `routing` seeds group sizes and ranks; the seed given to prepare()
decides the order of the requests and every value.
"""
import math

import numpy as np
import torch

from paper_2511_22880_amd import binding as L
from paper_2511_22880_amd import workloads as wl


def _case(kind, in_features, out_features, *, prompts=0, median=512, sigma=1.0, decode=0, adapters=1, ranks="mixed",
          own=False, alpha=1.1, idle=0.0, layers=1, rebuild=False, kv=0, host=False, routing=0, **name):
    return dict(name, kind=kind, **{"in": in_features, "out": out_features}, prompts=prompts, median=median, sigma=sigma,
                decode=decode, adapters=adapters, ranks=str(ranks), own=own, alpha=alpha, idle=idle, layers=layers,
                rebuild=rebuild, kv=kv, host=host, routing=routing)


def listed():
    return [
        # one user, one token: the latency of a single decode step of one projection
        _case("apply", 4096, 4096, decode=1, ranks=16, own=True, name="decode_one"),
        # a few requests with ranks nobody rounded, some without an adapter, on a projection of odd size
        _case("apply", 3008, 1920, decode=57, adapters=24, ranks="odd", alpha=0.6, idle=0.15, name="decode_ragged"),
        # bench.py's default step: 256 decode tokens, planned once, through one projection of 32 layers
        _case("apply", 4096, 4096, decode=256, adapters=128, layers=32, rebuild=True, name="decode_step"),
        # rank skew: rank-8 and rank-256 adapters share a decode batch of a large model
        _case("apply", 8192, 8192, decode=512, adapters=64, ranks="skew", alpha=0.0, name="decode_skew"),
        # the decode batch through all seven projections of a layer, the layers of a short stack in turn
        _case("layers", 4096, 14336, kv=1024, decode=256, adapters=128, layers=8, rebuild=True, name="decode_layers"),
        # one prompt of 2000 tokens with a rank-128 adapter (the isolated prefill of the paper)
        _case("apply", 4096, 4096, prompts=1, median=2000, sigma=0.0, ranks=128, own=True, name="prompt_one"),
        # 32 prompts of mixed lengths, an adapter each
        _case("apply", 4096, 4096, prompts=32, adapters=32, own=True, name="prefill"),
        # 8 prompts beside 384 decode tokens, 256 resident adapters, whole layers
        _case("layers", 4096, 14336, kv=1024, prompts=8, median=1150, sigma=0.6, decode=384, adapters=256, layers=4,
              rebuild=True, name="mixed_layers"),
        # one rank's share of a row-parallel down projection: shrink and expand apart
        _case("shard", 1792, 4096, prompts=32, adapters=32, own=True, name="shard_prefill"),
        # the adapted layer (base weight and delta) for a decode batch ...
        _case("linear", 4096, 4096, decode=256, adapters=128, name="linear_decode"),
        # ... and for the 32 prompts
        _case("linear", 4096, 4096, prompts=32, adapters=32, own=True, name="linear_prefill"),
        # adapters arriving from another GPU: packed into the pool from device memory
        _case("load", 4096, 4096, adapters=16, name="load_adapters"),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _multiple(rng, lo, hi, m):
    return max(m, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi))) / m)) * m)


def _ranks(rng):
    return rng.choice(["mixed", "mixed", "odd", "skew", str(rng.choice([8, 16, 64, 128, _log(rng, 1, 256)]))])


def draw(rng):
    kind = rng.choice(["decode", "decode", "prefill", "mixed", "layers", "shard", "linear", "linear", "load"])
    routing = rng.randrange(1, 1 << 20)
    in_f, out_f = _multiple(rng, 512, 16384, 64), _multiple(rng, 512, 16384, 128)
    if kind == "load":
        return _case("load", in_f, out_f, adapters=_log(rng, 1, 32), ranks=_ranks(rng), host=rng.random() < 0.4,
                     routing=routing)
    few = dict(decode=_log(rng, 1, 512), adapters=_log(rng, 1, 128), alpha=rng.choice([0.0, 0.6, 1.1]))
    prompts = _log(rng, 1, 32)
    many = dict(prompts=prompts, median=_log(rng, 40, min(2048, 18000 // prompts)), sigma=rng.choice([0.0, 0.5, 0.7]),
                adapters=prompts, own=True)
    both = dict(many, decode=_log(rng, 16, 400), adapters=_log(rng, 16, 256), own=False, alpha=rng.choice([0.6, 1.1]))
    idle = rng.choice([0.0, 0.0, round(rng.uniform(0.02, 0.4), 2)])
    more = dict(ranks=_ranks(rng), idle=idle, routing=routing)
    if kind == "decode":
        return _case("apply", in_f, out_f, layers=rng.choice([1, 1, 4, 8]), rebuild=rng.random() < 0.5, **few, **more)
    if kind == "prefill":
        return _case("apply", in_f, out_f, **many, **more)
    if kind == "mixed":
        return _case("apply", in_f, out_f, rebuild=rng.random() < 0.3, **both, **more)
    if kind == "layers":
        hidden = _multiple(rng, 1024, 5120, 128)
        batch = rng.choice([few, few, dict(both, prompts=min(prompts, 6), median=min(both["median"], 1000))])
        return _case("layers", hidden, _multiple(rng, 2 * hidden, 3.5 * hidden, 128), kv=rng.choice([hidden, 512, 1024]),
                     layers=rng.choice([1, 2]), rebuild=rng.random() < 0.5, **batch, **dict(more, ranks="mixed"))
    if kind == "shard":
        return _case("shard", in_f, out_f, **rng.choice([few, many]), **more)
    in_f, out_f = min(in_f, 8192), min(out_f, 8192)
    return _case("linear", in_f, out_f, **rng.choice([few, many, dict(both, prompts=min(prompts, 8))]), **more)


# ---- the batch of a case: group sizes and ranks from `routing`, the same for every seed -------------------
def _adapter_ranks(case):
    n, key = case["adapters"], [case["routing"], 1]
    if case["ranks"] == "mixed":
        return wl.balanced_ranks(n, wl.RANK_SET, key)
    if case["ranks"] == "skew":
        return wl.balanced_ranks(n, (8, 256), key)
    if case["ranks"] == "odd":
        return np.random.default_rng(key).integers(1, 257, size=n).astype(np.int32)
    return np.full(n, int(case["ranks"]), dtype=np.int32)


def _requests(case):
    """(length, adapter or -1) of every request."""
    r = case["routing"]
    lens = np.ones(case["prompts"] + case["decode"], dtype=np.int64)
    if case["prompts"]:
        lens[:case["prompts"]] = wl.lognormal_lengths(case["prompts"], float(case["median"]), case["sigma"], 16, 4096,
                                                      [r, 2])
    n = lens.shape[0]
    adapter = (np.arange(n) % case["adapters"] if case["own"]
               else wl.zipf_route(n, case["adapters"], case["alpha"], [r, 3])).astype(np.int32)
    if case["idle"]:
        adapter[np.random.default_rng([r, 4]).random(n) < case["idle"]] = -1
        if (adapter < 0).all():
            adapter[0] = 0
    return lens, adapter


def _projections(case):
    """[(in_features, (out_features of the projections that share x, ...)), ...] of one layer."""
    if case["kind"] != "layers":
        return [(case["in"], (case["out"],))]
    h, kv, inner = case["in"], case["kv"], case["out"]
    return [(h, (h, kv, kv)), (h, (h,)), (h, (inner, inner)), (inner, (h,))]


def _randn(gen, *shape, scale=1.0):
    return torch.empty(*shape, dtype=torch.bfloat16, device="cuda").normal_(0.0, scale, generator=gen)


class _State:
    """Pools, segment objects and tensors of one prepared case; the library's objects go with it."""

    def __init__(self, case):
        self.case = case
        self.pools, self.segs = [], []

    def __del__(self):
        try:
            for s in self.segs:
                L.lora_segments_destroy(s)
            for p in self.pools:
                L.lora_pool_destroy(p)
        except Exception:
            pass


def _pool(st, gen, in_f, out_f, ranks, arena, load=True):
    """A pool over `arena` with every adapter loaded: A and B are pieces of one buffer of N(0, 0.02) values."""
    scales = (2.0 / ranks).astype(np.float32)
    pool = L.lora_pool_create(in_f, out_f, ranks, scales, arena)
    st.pools.append(pool)
    if not load:
        return pool
    need = int(ranks.max()) * (in_f + out_f)
    total = int(ranks.astype(np.int64).sum()) * (in_f + out_f)
    src = _randn(gen, max(need, min(total, 1 << 24)), scale=0.02)
    at = 0
    for a in range(len(ranks)):
        r = int(ranks[a])
        n = r * (in_f + out_f)
        if at + n > src.numel():
            at = (at + 4096) % (src.numel() - n + 1) // 8 * 8
        L.lora_pool_load(pool, a, src[at:at + r * in_f].view(in_f, r), src[at + r * in_f:at + n].view(r, out_f))
        at += n
    return pool


def prepare(case, seed):
    st = _State(case)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    ranks = _adapter_ranks(case)
    scales = (2.0 / ranks).astype(np.float32)
    if case["kind"] == "load":
        in_f, out_f = case["in"], case["out"]
        arena = torch.zeros(L.lora_pool_bytes(in_f, out_f, ranks, scales), dtype=torch.uint8, device="cuda")
        st.arena, st.pool = arena, _pool(st, gen, in_f, out_f, ranks, arena, load=False)
        st.weights = [(_randn(gen, in_f, int(r), scale=0.02), _randn(gen, int(r), out_f, scale=0.02)) for r in ranks]
        if case["host"]:
            st.staging = [torch.empty(L.lora_pool_load_staging_bytes(st.pool, a), dtype=torch.uint8, device="cuda")
                          for a in range(len(ranks))]
            pinned = [torch.empty(t.numel(), dtype=torch.bfloat16, pin_memory=True) for w in st.weights for t in w]
            for p, t in zip(pinned, (t for w in st.weights for t in w)):
                p.copy_(t.view(-1))
            st.weights = list(zip(pinned[0::2], pinned[1::2]))
        return st

    lens, adapter = _requests(case)
    order = np.random.default_rng([seed, 5]).permutation(lens.shape[0])
    st.token_adapter = np.repeat(adapter[order], lens[order]).astype(np.int32)
    T = int(st.token_adapter.shape[0])
    st.layers = []
    for _ in range(case["layers"]):
        applies = []
        for in_f, outs in _projections(case):
            sizes = [(L.lora_pool_bytes(in_f, o, ranks, scales) + 4095) // 4096 * 4096 for o in outs]
            arena = torch.zeros(sum(sizes), dtype=torch.uint8, device="cuda")
            starts = np.concatenate([[0], np.cumsum(sizes)])
            pools = [_pool(st, gen, in_f, o, ranks, arena[int(starts[q]):int(starts[q + 1])])
                     for q, o in enumerate(outs)]
            applies.append((pools, _randn(gen, T, in_f), _randn(gen, T, sum(outs))))
        st.layers.append(applies)
    # the layers' pools lie alike, so one segment object per projection serves all of them
    st.ws = []
    for pools, _x, _y in st.layers[0]:
        build = L.lora_segments_build_multi if len(pools) > 1 else L.lora_segments_build
        seg = build(pools if len(pools) > 1 else pools[0], st.token_adapter)
        st.segs.append(seg)
        st.ws.append(torch.empty(max(L.lora_apply_workspace_bytes(pools[0], seg), 256), dtype=torch.uint8, device="cuda"))
    if case["kind"] == "shard":
        st.v = torch.empty(L.lora_segments_info(st.segs[0])["v_floats"], dtype=torch.float32, device="cuda")
        st.ws[0] = torch.empty(max(L.lora_workspace_bytes(st.layers[0][0][0][0], st.segs[0]), 256), dtype=torch.uint8,
                               device="cuda")
    if case["kind"] == "linear":
        st.w = torch.empty(case["in"] * case["out"], dtype=torch.bfloat16, device="cuda")
        L.lora_linear_pack_weight(_randn(gen, case["out"], case["in"], scale=0.02), case["in"], case["out"], st.w)
    return st


def run(st):
    kind = st.case["kind"]
    if kind == "load":
        for a, (A, B) in enumerate(st.weights):
            if st.case["host"]:
                L.lora_pool_load_staged(st.pool, a, A, B, st.staging[a])
            else:
                L.lora_pool_load(st.pool, a, A, B)
        return st.arena
    if kind == "shard":
        pools, x, y = st.layers[0][0]
        L.lora_shrink(pools[0], st.segs[0], x, st.v, st.ws[0])
        L.lora_expand(pools[0], st.segs[0], st.v, y)
        return st.v, y
    if kind == "linear":
        pools, x, y = st.layers[0][0]
        L.lora_linear(pools[0], st.segs[0], x, st.w, y, st.ws[0])
        return y
    if st.case["rebuild"]:
        for seg in st.segs:
            L.lora_segments_rebuild(seg, st.token_adapter)
    for applies in st.layers:
        for (pools, x, y), seg, ws in zip(applies, st.segs, st.ws):
            if len(pools) > 1:
                L.lora_apply_multi(pools, seg, x, y, ws)
            else:
                L.lora_apply(pools[0], seg, x, y, ws)
    return [y for applies in st.layers for _pools, _x, y in applies]


def work(case):
    """Each adapter the batch uses, x, and y (read and written; written only by `linear`) once per pass; v only
    where it leaves the library.  Products: both halves of the delta, and the base layer of `linear`."""
    ranks = _adapter_ranks(case).astype(np.int64)
    if case["kind"] == "load":
        size = 2 * (case["in"] + case["out"])
        return {"bytes": int(size * (ranks.sum() + ((ranks + 7) // 8 * 8).sum())), "flops": 0}
    lens, adapter = _requests(case)
    T, act = int(lens.sum()), adapter >= 0
    n_act = int(lens[act].sum())
    used = int(ranks[np.unique(adapter[act])].sum())
    v = int((lens[act] * ranks[adapter[act]]).sum())
    nbytes = flops = 0
    for in_f, outs in _projections(case):
        nbytes += 2 * n_act * in_f
        for o in outs:
            nbytes += 2 * used * (in_f + o) + 4 * n_act * o
            flops += 2 * v * (in_f + o)
    if case["kind"] == "linear":
        in_f, o = case["in"], case["out"]
        nbytes += 2 * in_f * o + 2 * (T - n_act) * in_f + 2 * T * o - 4 * n_act * o
        flops += 2 * T * in_f * o
    if case["kind"] == "shard":
        nbytes += 8 * v
    return {"bytes": int(nbytes * case["layers"]), "flops": int(flops * case["layers"])}


def tolerance(case):
    """Packed adapters are bytes.  y is rounded to bf16 once from fp32 sums (half a unit in the last place, 2^-9
    of the value at most): against the same path in 64 bits it is seen 1.4e-3 to 1.7e-3 off in the 2-norm and
    3.9e-3 at most; four times that."""
    return "exact" if case["kind"] == "load" else {"rel": 6e-3, "max": 1.6e-2}
