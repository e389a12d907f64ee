"""The work a serving engine has this library do, as cases that can be timed and compared.

Five kinds of pass, each through the calls of `PrismKV` as an engine's step makes them:

  decode    one decode step of the models that share a pool: where `append` is set, every layer first
            appends its new token's K and V, then the layer attends (one model: `decode_attention`, several:
            one grouped launch of `decode_attention_multi`)
  prefill   one chunk of chunked prefill: the chunk's K and V are appended, then its queries attend to
            what was cached and, causally, to the chunk
  append    the write path of a prompt chunk by itself; the pool's bytes are the result
  restore   a sequence whose K and V come from elsewhere (migration, swap-in) is written in bulk with
            `kv_write`; the pool's bytes are the result
  turnover  a model falls idle and another batch of requests takes its place: release, deflate, inflate,
            reserve, all enqueue-only; the block table is the result

Models are written "q_heads/kv_heads/head_dim dtype xbatch", several separated by commas.  Context lengths
are lognormal around `ctx` (sigma `spread`, capped at `cap`; `spread` 0: all equal to `ctx`, `lo` > 0: uniform
from `lo` to `cap`); they belong to the case and the seed only deals them to the sequences, so that passes over
different inputs do the same work.  Values are N(0, 1) in bf16, e4m3 caches hold them quantised per (block, kv head).
"""
import math
import random
import weakref

import numpy as np
import torch

from paper_2505_04021_amd import PKV_BF16, PKV_E4M3, PrismKV

T = 16                      # tokens per block
FRAME = 2 << 20
DEV = "cuda:0"
E4M3_MAX = 448.0

LISTED = [
    # the smallest call: four short chats of a small model, where launches and latency are all there is
    dict(name="decode_tiny", kind="decode", models="8/2/64 bf16 x4", ctx=128, spread=0.0, lo=16, cap=256, layers=1,
         append=True, pool_gib=1),
    # a lightly loaded model: a small batch of ordinary contexts, several layers back to back
    dict(name="decode_light", kind="decode", models="32/8/128 bf16 x8", ctx=2048, spread=0.8, lo=0, cap=8192, layers=4,
         append=True, pool_gib=8),
    # two co-located models at full batch, the grouped launch of the headline benchmark
    dict(name="decode_two_models", kind="decode", models="32/8/128 bf16 x64, 32/8/64 bf16 x64", ctx=1024, spread=0.8, lo=0,
         cap=8192, layers=1, append=False, pool_gib=32),
    # four models on e4m3 caches, batches of unlike size
    dict(name="decode_fp8_models", kind="decode",
         models="32/8/128 e4m3 x128, 32/8/128 e4m3 x64, 32/8/128 e4m3 x32, 32/8/128 e4m3 x32", ctx=2048, spread=0.0, lo=512,
         cap=4096, layers=1, append=False, pool_gib=8),
    # long contexts, the largest decode launch
    dict(name="decode_long", kind="decode", models="64/8/128 bf16 x16", ctx=32768, spread=0.0, lo=0, cap=32768, layers=1,
         append=False, pool_gib=16),
    # chunked prefill at the size the benchmark times, both cache types
    dict(name="prefill_chunk", kind="prefill", models="32/8/128 bf16 x8", cached=2048, cached_spread=0.0, new=512, new_spread=0.0,
         cap=8192, pool_gib=8),
    dict(name="prefill_chunk_fp8", kind="prefill", models="32/8/128 e4m3 x8", cached=2048, cached_spread=0.0, new=512,
         new_spread=0.0, cap=8192, pool_gib=8),
    # one long document, its last chunk: few queries in front of a long context
    dict(name="prefill_long", kind="prefill", models="64/8/128 bf16 x1", cached=15872, cached_spread=0.0, new=512, new_spread=0.0,
         cap=32768, pool_gib=8),
    # a step's worth of fresh prompts of ragged length on a model with 64-wide heads, some with a cached prefix
    dict(name="prefill_prompts", kind="prefill", models="32/8/64 bf16 x24", cached=64, cached_spread=1.0, new=220, new_spread=0.7,
         cap=900, pool_gib=8),
    # prompts going into an e4m3 cache: scales and codes
    dict(name="append_fp8", kind="append", models="32/8/128 e4m3 x8", cached=0, cached_spread=0.0, new=512, new_spread=0.0,
         cap=8192),
    # a migrated sequence written back in bulk
    dict(name="restore_seq", kind="restore", models="32/8/128 bf16 x1", ctx=8192, cap=8192),
    # one model of a bursty group goes, the next batch comes
    dict(name="turnover", kind="turnover", models="32/8/128 bf16 x32", ctx=2048, spread=0.8, lo=0, cap=8192, pool_gib=8),
]


def listed():
    return [dict(c) for c in LISTED]


def _logint(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    most = [max(work(c)[w] for c in LISTED) for w in ("bytes", "flops")]
    while True:
        case = _draw(rng)
        w = work(case)
        if w["bytes"] <= most[0] and w["flops"] <= most[1]:
            return case


def _draw(rng):
    kind = rng.choice(["decode", "decode", "prefill", "prefill", "prefill", "append", "restore", "turnover"])
    dtypes = ["bf16", "bf16", "e4m3"]

    def shape(dtype, batch):
        hkv = rng.choice([1, 2, 4, 8, 8])
        return "%d/%d/%d %s x%d" % (hkv * rng.choice([1, 2, 3, 4, 4, 5, 7, 8]), hkv, rng.choice([64, 128, 128]), dtype, batch)

    if kind == "decode":
        n = rng.choice([1, 1, 2, 3])
        ctx = _logint(rng, 60, 12000)
        most = max(1, min(128, int(1.5e5 / ctx)))
        models = ", ".join(shape(rng.choice(dtypes), _logint(rng, 1, most)) for _ in range(n))
        layers = rng.choice([1, 1, 2]) if n == 1 else 1
        append = n == 1 and rng.random() < 0.6
        return dict(kind=kind, models=models, ctx=ctx, spread=rng.choice([0.0, 0.5, 0.8]), lo=0, cap=min(32768, 4 * ctx),
                    layers=layers, append=append, pool_gib=8)
    if kind == "prefill":
        new = _logint(rng, 17, 1500)
        cached = rng.choice([0, _logint(rng, 16, 4000), _logint(rng, 16, 12000)])
        batch = _logint(rng, 1, max(1, min(32, int(2e6 / (new * (new + cached))), int(3e4 / (new + cached)))))
        return dict(kind=kind, models=shape(rng.choice(dtypes), batch), cached=cached, cached_spread=rng.choice([0.0, 0.8]), new=new,
                    new_spread=rng.choice([0.0, 0.7]), cap=8192, pool_gib=8)
    if kind == "append":
        new = _logint(rng, 5, 2000)
        return dict(kind=kind, models=shape(rng.choice(dtypes), _logint(rng, 1, max(1, min(32, int(8192 / new))))),
                    cached=rng.choice([0, _logint(rng, 8, 500)]), cached_spread=0.7, new=new, new_spread=rng.choice([0.0, 0.7]), cap=8192)
    if kind == "restore":
        n = _logint(rng, 30, 12000)
        return dict(kind=kind, models=shape(rng.choice(dtypes), 1), ctx=n, cap=n)
    ctx = _logint(rng, 60, 4000)
    return dict(kind=kind, models=shape(rng.choice(dtypes), _logint(rng, 1, max(1, min(64, int(1e5 / ctx))))), ctx=ctx,
                spread=rng.choice([0.0, 0.5, 0.8]), lo=0, cap=8192, pool_gib=4)


# ---------------------------------------------------------------- what a case says

class Spec:
    def __init__(self, text):
        heads, dtype, batch = text.split()
        self.hq, self.hkv, self.d = (int(x) for x in heads.split("/"))
        self.dtype = PKV_BF16 if dtype == "bf16" else PKV_E4M3
        self.batch = int(batch[1:])
        self.e = 2 if self.dtype == PKV_BF16 else 1

    def layer_bytes(self):
        return 2 * T * self.hkv * self.d * self.e + (0 if self.dtype == PKV_BF16 else 128)

    def kv_bytes(self, tokens, blocks):
        """K and V of so many tokens, and the scales of so many blocks."""
        return tokens * self.hkv * self.d * 2 * self.e + (0 if self.dtype == PKV_BF16 else blocks * self.hkv * 8)


def _specs(case):
    return [Spec(s) for s in case["models"].split(",")]


def _rng(case, what, i=0):
    return random.Random("%s %d %s" % (what, i, sorted((k, v) for k, v in case.items() if k != "name")))


def _lengths(rng, n, median, spread, lo, cap, least=1):
    if lo > 0:
        return [rng.randint(lo, cap) for _ in range(n)]
    if spread == 0.0:
        return [min(median, cap)] * n
    return [min(cap, max(least, int(round(median * math.exp(spread * rng.gauss(0.0, 1.0)))))) for _ in range(n)]


def _ctx(case, i=0):
    """Context lengths of model i's sequences (decode, restore, turnover)."""
    return _lengths(_rng(case, "ctx", i), _specs(case)[i].batch, case["ctx"], case.get("spread", 0.0), case.get("lo", 0), case["cap"])


def _chunks(case):
    """[(cached tokens, new tokens)] of a prefill or an append.  A chunk on an e4m3 cache starts on a block, as
    schedulers cut chunks: appending it again then gives the same codes (a block's scale starts afresh)."""
    s = _specs(case)[0]
    rng = _rng(case, "chunk")
    new = _lengths(rng, s.batch, case["new"], case["new_spread"], 0, case["cap"])
    old = _lengths(rng, s.batch, case["cached"], case["cached_spread"], 0, case["cap"], 0) if case["cached"] else [0] * s.batch
    if s.dtype == PKV_E4M3:
        old = [c // T * T for c in old]
    return list(zip(old, new))


def _blocks(tokens):
    return (tokens + T - 1) // T


def work(case):
    kind, specs = case["kind"], _specs(case)
    if kind == "decode":
        nbytes = flops = 0
        for i, s in enumerate(specs):
            ctx = _ctx(case, i)
            nbytes += s.kv_bytes(sum(ctx), sum(_blocks(c) for c in ctx)) + s.batch * (s.hq * s.d * 6 + 4)
            if case["append"]:
                nbytes += s.batch * s.hkv * s.d * 4 + s.kv_bytes(s.batch, s.batch)
            flops += 4 * s.d * s.hq * sum(ctx)
        return {"bytes": nbytes * case["layers"], "flops": flops * case["layers"]}
    s = specs[0]
    if kind in ("prefill", "append"):
        chunks = _chunks(case)
        new = sum(n for _, n in chunks)
        nbytes = new * s.hkv * s.d * 4 + s.kv_bytes(new, sum(_blocks(n) for _, n in chunks))
        if kind == "append":
            return {"bytes": nbytes, "flops": 0}
        nbytes += s.kv_bytes(sum(o + n for o, n in chunks), sum(_blocks(o + n) for o, n in chunks)) + new * s.hq * s.d * 6
        return {"bytes": nbytes, "flops": 4 * s.d * s.hq * sum(n * o + n * (n + 1) // 2 for o, n in chunks)}
    if kind == "restore":
        return {"bytes": 2 * s.kv_bytes(case["ctx"], _blocks(case["ctx"])), "flops": 0}
    ctx = _ctx(case)
    # a block: its id written, its slot bit set and cleared; a list entry: two words
    return {"bytes": 8 * sum(_blocks(c) for c in ctx) + 8 * len(_grow(ctx, 64)[0]), "flops": 0}


def tolerance(case):
    if case["kind"] in ("append", "restore", "turnover"):
        return "exact"
    # fp32 sums of products with probabilities of 16 significant bits (2^-17 each): sums in another order and
    # split elsewhere differ by 1e-6 to 4e-6.  A prefill on an e4m3 cache multiplies with probabilities of 8 bits.
    if case["kind"] == "prefill" and "e4m3" in case["models"]:
        return {"rel": 1e-2, "max": 0.3}
    return {"rel": 1e-5, "max": 4e-4}


# ---------------------------------------------------------------- inputs

def _gen(seed, *key):
    g = torch.Generator(device=DEV)
    g.manual_seed((seed * 1000003 + sum((k + 1) * 7919 ** (i + 1) for i, k in enumerate(key))) % (1 << 62))
    return g


def _randn(shape, g):
    return torch.randn(shape, generator=g, device=DEV, dtype=torch.float32).to(torch.bfloat16)


def _deal(seed, values, i=0):
    values = list(values)
    random.Random("deal %d %d" % (seed, i)).shuffle(values)
    return values


def _quantise(x):
    """[blocks][T][Hkv][D] fp32 -> e4m3 codes and one scale per (block, kv head)."""
    amax = x.abs().amax(dim=(1, 3))
    scale = torch.where(amax > 0, amax / E4M3_MAX, torch.ones_like(amax))
    return (x / scale[:, None, :, None]).clamp(-E4M3_MAX, E4M3_MAX).to(torch.float8_e4m3fn), scale


def _cache(s, lens, g):
    """K and V of the sequences' first `lens` tokens, every sequence padded to whole blocks: bf16 tensors, or e4m3 codes
    with their scales."""
    rows = sum(_blocks(n) for n in lens) * T
    kv = []
    for _ in range(2):
        x = _randn((rows, s.hkv, s.d), g)
        if s.dtype == PKV_E4M3:
            x, scale = _quantise(x.float().view(-1, T, s.hkv, s.d))
            kv.append((x.view(torch.uint8).view(rows, s.hkv, s.d), scale))
        else:
            kv.append((x, None))
    return kv


def _grow(lens, step):
    """A reserve list in which sequences grow side by side, `step` tokens a round, as under concurrent decoding."""
    seqs, ctx = [], []
    for r in range((max(lens) + step - 1) // step):
        for i, n in enumerate(lens):
            if n > r * step:
                seqs.append(i)
                ctx.append(min(n, (r + 1) * step))
    return np.array(seqs, dtype=np.int32), np.array(ctx, dtype=np.int32)


class _Table:
    """The library's block table as an array that torch can look at without a copy."""

    def __init__(self, ptr, rows, stride):
        self.__cuda_array_interface__ = {"shape": (rows, stride), "typestr": "<i4", "data": (ptr, False), "version": 3}


def _close(be, pool, models):
    torch.cuda.synchronize()
    for m, n in models:
        be.seq_release_batch(m, np.arange(n, dtype=np.int32))
        be.balloon_resize(m, 0)
        be.model_unregister(m)
    be.pool_destroy(pool)
    torch.cuda.synchronize()


class State:
    """A pool with its models, their sequences admitted, and the tensors a step hands in."""

    def __init__(self, case, seed, lens, layers=1, frames=None, spare=0):
        specs = self.specs = _specs(case)
        self.case, self.lens = case, lens
        be = self.be = PrismKV(DEV)
        need = []
        for s, ls in zip(specs, lens):
            slots = FRAME // (layers * s.layer_bytes())
            need.append((sum(_blocks(n) for n in ls) + slots - 1) // slots)
        self.need = need
        # where the pool's bytes are the result, the pool is a tensor of the caller's; else the library allocates
        n_frames = sum(need) if frames is None else max(frames, sum(need) + spare)
        self.storage = torch.zeros(n_frames * FRAME, dtype=torch.uint8, device=DEV) if frames is None else None
        self.pool = be.pool_create(n_frames * FRAME, T, FRAME, storage=self.storage)
        assert self.pool >= 0, be.last_error()
        order = np.random.RandomState(seed % (1 << 31)).permutation(n_frames).astype(np.uint32)
        assert be.pool_seed_free_order(self.pool, order) >= 0
        self.models, owned = [], []
        weakref.finalize(self, _close, be, self.pool, owned)
        for s, ls in zip(specs, lens):
            m = be.model_register(self.pool, s.hq, s.hkv, s.d, s.dtype, s.batch, max(_blocks(n) for n in ls) + 1, layers)
            assert m >= 0, be.last_error()
            self.models.append(m)
            owned.append((m, s.batch))
        # balloons grow in turns of 8 frames, so that the models' frames interleave
        have = [0] * len(specs)
        while have != need:
            for i, m in enumerate(self.models):
                if have[i] < need[i]:
                    have[i] = min(need[i], have[i] + 8)
                    assert be.balloon_resize(m, have[i]) == have[i]
        for m, ls in zip(self.models, lens):
            seqs, ctx = _grow(ls, 64)
            for a in range(0, len(seqs), 4096):
                assert be.seq_reserve_batch(m, seqs[a:a + 4096], ctx[a:a + 4096]) >= 0

    def fill(self, i, lens, g):
        """K and V of the first `lens` tokens of model i's sequences into the pool; returns them."""
        s, m, be = self.specs[i], self.models[i], self.be
        (k, ks), (v, vs) = kv = _cache(s, lens, g)
        if s.dtype == PKV_BF16 and sum(lens):
            starts = np.cumsum([0] + [_blocks(n) * T for n in lens])
            pick = torch.cat([torch.arange(a, a + n) for a, n in zip(starts, lens)]).to(DEV)
            ctx = torch.tensor(lens, dtype=torch.int32, device=DEV)
            assert be.kv_append_chunk_dev(m, k[pick], v[pick], np.array(lens, dtype=np.int32), ctx) == sum(lens)
            torch.cuda.synchronize()
        elif s.dtype == PKV_E4M3:
            at = 0
            for q, n in enumerate(lens):
                b = _blocks(n)
                if n:
                    assert be.kv_write(m, q, 0, k[at:at + n], v[at:at + n], ks[at // T:at // T + b], vs[at // T:at // T + b]) == n
                at += b * T
        return kv


def _parts(case, seed, given=None):
    """The tensors of a pass, from the seed: per layer and model (or for the chunk) queries and new K and V.
    With a State given, its pool is filled as well; the K and V cached before the pass are part of the answer."""
    kind, specs = case["kind"], _specs(case)
    got = []
    if kind == "decode":
        for layer in range(case["layers"]):
            for i, s in enumerate(specs):
                lens = _deal(seed, _ctx(case, i), i)
                g = _gen(seed, layer, i)
                if given:
                    given.be.set_layer(given.models[i], layer)
                    cache = given.fill(i, lens, g)
                else:
                    cache = _cache(s, lens, g)
                got.append(dict(spec=s, lens=lens, cache=cache, q=_randn((s.batch, s.hq, s.d), g),
                                k=_randn((s.batch, s.hkv, s.d), g), v=_randn((s.batch, s.hkv, s.d), g)))
        return got
    s, g = specs[0], _gen(seed)
    chunks = _deal(seed, _chunks(case))
    old, new = [o for o, _ in chunks], [n for _, n in chunks]
    cache = given.fill(0, old, g) if given else _cache(s, old, g)
    rows = sum(new)
    return [dict(spec=s, old=old, new=new, cache=cache, q=_randn((rows, s.hq, s.d), g) if kind == "prefill" else None,
                 k=_randn((rows, s.hkv, s.d), g), v=_randn((rows, s.hkv, s.d), g))]


def prepare(case, seed):
    kind, specs = case["kind"], _specs(case)
    i32 = lambda x: torch.tensor(x, dtype=torch.int32, device=DEV)  # noqa: E731
    if kind == "decode":
        lens = [_deal(seed, _ctx(case, i), i) for i in range(len(specs))]
        st = State(case, seed, lens, case["layers"], frames=(case["pool_gib"] << 30) // FRAME)
        st.steps = []
        ctx = [i32(n) for n in lens]
        parts = _parts(case, seed, st)
        for layer in range(case["layers"]):
            p = parts[layer * len(specs):(layer + 1) * len(specs)]
            st.steps.append(dict(ctx=ctx, q=[x["q"] for x in p], k=[x["k"] for x in p], v=[x["v"] for x in p],
                                 out=[torch.empty((s.batch, s.hq, s.d), dtype=torch.float32, device=DEV) for s in specs]))
        return st
    if kind in ("prefill", "append"):
        chunks = _deal(seed, _chunks(case))
        st = State(case, seed, [[o + n for o, n in chunks]], frames=(case["pool_gib"] << 30) // FRAME if kind == "prefill" else None)
        p = _parts(case, seed, st)[0]
        st.k, st.v, st.q = p["k"], p["v"], p["q"]
        st.q_lens = np.array(p["new"], dtype=np.int32)
        st.ctx = i32([o + n for o, n in chunks])
        if kind == "prefill":
            st.out = torch.empty(st.q.shape, dtype=torch.float32, device=DEV)
        return st
    if kind == "restore":
        st = State(case, seed, [[case["ctx"]]])
        (k, ks), (v, vs) = _cache(specs[0], [case["ctx"]], _gen(seed))
        st.k, st.v, st.ks, st.vs = k[:case["ctx"]], v[:case["ctx"]], ks, vs
        return st
    lens = _deal(seed, _ctx(case))
    st = State(case, seed, [lens], frames=(case["pool_gib"] << 30) // FRAME)
    st.gone = np.arange(specs[0].batch, dtype=np.int32)
    st.seqs, st.ctx = _grow(_deal(seed, lens, 1), 64)
    ptr, stride = st.be.model_block_table(st.models[0])
    st.table = torch.as_tensor(_Table(ptr, specs[0].batch, stride), device=DEV)
    return st


# ---------------------------------------------------------------- one pass

def run(st):
    be, kind, m = st.be, st.case["kind"], st.models[0]
    if kind == "decode":
        layers = st.case["layers"]
        for layer, x in enumerate(st.steps):
            if layers > 1:
                be.set_layer(m, layer)
            if st.case["append"]:
                be.kv_append_dev(m, x["k"][0], x["v"][0], x["ctx"][0])
            if len(st.models) == 1:
                be.decode_attention_dev(m, x["q"][0], x["ctx"][0], x["out"][0])
            else:
                be.decode_attention_multi_dev(st.models, x["q"], x["ctx"], x["out"])
        return [o for x in st.steps for o in x["out"]]
    if kind in ("prefill", "append"):
        be.kv_append_chunk_dev(m, st.k, st.v, st.q_lens, st.ctx)
        if kind == "append":
            return st.storage
        be.prefill_attention_dev(m, st.q, st.q_lens, st.ctx, st.out)
        return st.out
    if kind == "restore":
        be.kv_write(m, 0, 0, st.k, st.v, st.ks, st.vs)
        return st.storage
    be.seq_release_batch_enqueue(m, st.gone)
    be.balloon_resize_enqueue(m, 0)
    be.balloon_resize_enqueue(m, st.need[0])
    for a in range(0, len(st.seqs), 4096):
        be.seq_reserve_batch_enqueue(m, st.seqs[a:a + 4096], st.ctx[a:a + 4096])
    return st.table


# ---------------------------------------------------------------- the same in 64 bits

def _append_e4m3(codes, scale, x, lo, hi):
    """The append rule of an e4m3 cache for one block per row: tokens lo[b] .. hi[b] - 1 of x [n][T][Hkv][D] (bf16 values) go in
    order into codes [n][T][Hkv][D] (e4m3) under scale [n][Hkv]; a larger token raises the scale and re-encodes what is there."""
    enc = lambda y: y.clamp(-E4M3_MAX, E4M3_MAX).to(torch.float8_e4m3fn).float()  # noqa: E731
    c, s = codes.float(), scale.clone()
    for t in range(T):
        on = ((lo <= t) & (t < hi))[:, None]
        amax = x[:, t].float().abs().amax(dim=-1)
        cand = amax / E4M3_MAX
        if t == 0:
            s = torch.where(on, torch.where(amax > 0, cand, torch.ones_like(cand)), s)
        else:
            grow = on & (cand > s)
            again = enc((c * s[:, None, :, None]) / torch.where(grow, cand, torch.ones_like(cand))[:, None, :, None])
            c = torch.where(grow[:, None, :, None], again, c)
            s = torch.where(grow, cand, s)
        c[:, t] = torch.where(on[:, :, None], enc(x[:, t].float() / s[:, :, None]), c[:, t])
    return c, s


def _values(s, cache, olds, news, x, which):
    """Cached values after the append, per sequence, fp64 [tokens][Hkv][D]; olds[i] tokens were there, news[i] more come from x."""
    data, scale = cache[which]
    seqs, at, row = [], 0, 0
    for o, n in zip(olds, news):
        b = _blocks(o) * T
        if s.dtype == PKV_BF16:
            seqs.append(torch.cat([data[at:at + o], x[row:row + n]]).double())
        else:
            full = _blocks(o + n)
            c = torch.zeros((full * T, s.hkv, s.d), device=DEV)
            y = torch.zeros((full * T, s.hkv, s.d), device=DEV)
            sc = torch.ones((full, s.hkv), device=DEV)
            c[:o] = data[at:at + o].view(torch.float8_e4m3fn).float()
            sc[:b // T] = scale[at // T:(at + b) // T]
            y[o:o + n] = x[row:row + n].float()
            if n:
                tok0 = torch.arange(full, device=DEV) * T
                c, sc = _append_e4m3(c.view(full, T, s.hkv, s.d), sc, y.view(full, T, s.hkv, s.d), o - tok0, o + n - tok0)
            seqs.append((c.view(full, T, s.hkv, s.d).double() * sc.double()[:, None, :, None]).view(full * T, s.hkv, s.d)[:o + n])
        at += b
        row += n
    return seqs


def _attend(q, k, v, back):
    """softmax(q K^T / sqrt(D)) V in fp64: q [n][Hq][D], k and v [L][Hkv][D]; query i sees back + i + 1 tokens."""
    n, hq, d = q.shape
    length, hkv, _ = k.shape
    g = hq // hkv
    out = torch.empty((n, hq, d), dtype=torch.float64, device=DEV)
    seen = torch.arange(length, device=DEV)[None, :] <= back + torch.arange(n, device=DEV)[:, None]
    for h in range(hkv):
        qh = q[:, h * g:(h + 1) * g].double().reshape(n * g, d)
        p = (qh @ k[:, h].t().contiguous()) / math.sqrt(d)
        p = torch.softmax(p.view(n, g, length).masked_fill(~seen[:, None, :], -math.inf), dim=-1)
        out[:, h * g:(h + 1) * g] = (p.view(n * g, length) @ v[:, h].contiguous()).view(n, g, d)
    return out


def exact(case, seed):
    kind = case["kind"]
    if kind not in ("decode", "prefill"):
        return None
    answers = []
    for p in _parts(case, seed):
        s = p["spec"]
        if kind == "decode":
            if case["append"] and s.dtype == PKV_E4M3:
                ks, vs = (_last_again(s, p["cache"][w], p["lens"], x) for w, x in ((0, p["k"]), (1, p["v"])))
            else:
                ks, vs = (_values(s, p["cache"], p["lens"], [0] * s.batch, x, w) for w, x in ((0, p["k"]), (1, p["v"])))
                if case["append"]:
                    for i in range(s.batch):
                        ks[i][-1], vs[i][-1] = p["k"][i].double(), p["v"][i].double()
            answers.append(torch.cat([_attend(p["q"][i:i + 1], ks[i], vs[i], ks[i].shape[0] - 1) for i in range(s.batch)]))
        else:
            ks, vs = (_values(s, p["cache"], p["old"], p["new"], x, w) for w, x in ((0, p["k"]), (1, p["v"])))
            rows = np.cumsum([0] + p["new"])
            answers.append(torch.cat([_attend(p["q"][rows[i]:rows[i + 1]], ks[i], vs[i], p["old"][i]) for i in range(s.batch)]))
    return answers if kind == "decode" else answers[0]


def _last_again(s, cache, lens, x):
    """A decode step's append into an e4m3 cache that already holds the token's place: the last block's scale stays unless the
    token is larger than all it has seen (its first slot starts afresh)."""
    data, scale = cache
    seqs, at = [], 0
    for i, n in enumerate(lens):
        b = _blocks(n)
        c = data[at:at + b * T].view(torch.float8_e4m3fn).float().view(b, T, s.hkv, s.d).clone()
        c.view(b * T, s.hkv, s.d)[n:] = 0
        sc = scale[at // T:at // T + b].clone()
        y = torch.zeros((1, T, s.hkv, s.d), device=DEV)
        slot = torch.tensor([(n - 1) % T], device=DEV)
        y[0, (n - 1) % T] = x[i].float()
        c[-1:], sc[-1:] = _append_e4m3(c[-1:], sc[-1:], y, slot, slot + 1)
        seqs.append((c.double() * sc.double()[:, None, :, None]).view(b * T, s.hkv, s.d)[:n])
        at += b * T
    return seqs
