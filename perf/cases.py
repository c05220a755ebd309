"""Performance cases of the mixed-batch paged-attention library: what a serving instance has it do, step by step.

A case is a batch of requests over one paged KV pool and the call or calls that a step makes on it:

  entry "plan"    ooco_plan + ooco_attn_mixed: one attention layer of a step, planned from the scheduler's lengths
  entry "static"  ooco_attn_mixed_static: the same step for callers that hold no context
  entry "graph"   a captured decode step of several layers (ooco_kv_append + ooco_attn_mixed each), replayed
  entry "append"  ooco_kv_append: this step's K/V vectors into their paged slots
  entry "copy"    ooco_kv_block_copy: eviction of whole KV blocks to a staging pool

Lengths belong to the case (its "lengths" number seeds them), values, block tables and block ids to the seed of
`prepare`.  Head layouts are those of the repository's configurations and tests: 32/8 and 64/8 heads of 128, 28/4 heads
of 128, 32/4 heads of 64, 4/1 heads of 64.
"""
import math
from types import SimpleNamespace

import numpy as np
import torch

BS = 16          # tokens per KV block

HEADS = [(32, 8, 128), (64, 8, 128), (28, 4, 128), (32, 4, 64)]


# ------------------------------------------------------------------------------------------------- the cases
def _case(name, entry, heads, lengths, decodes=0, dist="uniform", lo=512, hi=4096, chunks=0, rows_lo=0, rows_hi=0, ctx_lo=0,
          ctx_hi=0, layers=1, victims=0):
    Hq, Hkv, hd = heads
    c = {"entry": entry, "Hq": Hq, "Hkv": Hkv, "hd": hd, "lengths": lengths, "decodes": decodes, "dist": dist, "lo": lo, "hi": hi,
         "chunks": chunks, "rows_lo": rows_lo, "rows_hi": rows_hi, "ctx_lo": ctx_lo, "ctx_hi": ctx_hi, "layers": layers,
         "victims": victims}
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # the smallest step: a handful of short decodes and one short prompt (4/1 heads of 64); launches and latency
        _case("static-tiny", "static", (4, 1, 64), 0, decodes=4, lo=37, hi=129, chunks=1, rows_lo=32, rows_hi=32),
        # a small offline decode batch, four layers captured once and replayed, each appending its K/V first
        _case("graph-decode-16", "graph", (32, 8, 128), 1, decodes=16, layers=4),
        # an online prompt in two ragged chunks beside a few short decodes: a lightly loaded instance
        _case("mixed-small", "plan", (28, 4, 128), 2, decodes=24, dist="lognormal", lo=128, hi=4096, chunks=2, rows_lo=90,
              rows_hi=230, ctx_lo=0, ctx_hi=1024),
        # offline decode of 64 sequences of 512..4096 tokens
        _case("decode-64", "plan", (32, 8, 128), 2, decodes=64),
        # a large decode batch of a small-head model: 256 sequences, heads of 64
        _case("decode-256-hd64", "plan", (32, 4, 64), 3, decodes=256),
        # online prefill only: eight 512-token chunks on up to 2048 cached tokens
        _case("prefill-8x512", "plan", (32, 8, 128), 3, chunks=8, rows_lo=512, rows_hi=512, ctx_hi=2048),
        # long prefill chunks of the large model: two of 2048 tokens on 4096 cached ones
        _case("prefill-2x2048", "plan", (64, 8, 128), 5, chunks=2, rows_lo=2048, rows_hi=2048, ctx_lo=4096, ctx_hi=4096),
        # one online turn on a long cached conversation: few rows, many keys
        _case("chunk-on-prefix", "plan", (32, 8, 128), 7, chunks=1, rows_lo=300, rows_hi=300, ctx_lo=12000, ctx_hi=16000),
        # the co-located step: eight online chunks beside 128 offline decodes
        _case("mixed-8x512-128", "plan", (32, 8, 128), 3, decodes=128, dist="lognormal", lo=128, hi=8192, chunks=8, rows_lo=512,
              rows_hi=512, ctx_hi=2048),
        # the long-context co-located step of the large model: 2 x 2048 rows beside 32 decodes of 32K..131K tokens
        _case("mixed-long", "plan", (64, 8, 128), 5, decodes=32, lo=32768, hi=131072, chunks=2, rows_lo=2048, rows_hi=2048,
              ctx_lo=4096, ctx_hi=4096),
        # the co-located step's K/V append: 128 single tokens and eight chunks of 512
        _case("append-8x512-128", "append", (32, 8, 128), 3, decodes=128, dist="lognormal", lo=128, hi=8192, chunks=8, rows_lo=512,
              rows_hi=512, ctx_hi=2048),
        # a preemption: the blocks of 64 of 512 offline sequences leave for free slots of a staging pool
        _case("evict-64", "copy", (32, 8, 128), 4, decodes=512, dist="lognormal", lo=64, hi=32768, victims=64),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


MAX_KV_TOKENS = 600_000      # of 8 kv heads of 128: 2.4 GB, under the largest listed case
MAX_PAIRS = 12_000_000       # visible (row, key) pairs of all chunks


def draw(rng):
    """A case of the listed ranges: 1..512 decodes, 0..8 chunks of 2..2048 rows on 0..32K cached tokens."""
    while True:
        heads = rng.choice(HEADS)
        kind = rng.choice(["decode", "decode", "prefill", "prefill", "mixed", "mixed", "static", "graph", "append", "copy"])
        lengths = rng.randrange(1 << 20)
        top = _log(rng, 256, 32768)
        dec = dict(decodes=_log(rng, 1, 512), dist=rng.choice(["uniform", "lognormal"]), lo=max(16, top // rng.choice([4, 8, 64])), hi=top)
        r_hi = _log(rng, 2, 2048)
        c_hi = _log(rng, 16, 32768)
        pf = dict(chunks=rng.randint(1, 8), rows_lo=max(2, r_hi // rng.choice([1, 2, 4])), rows_hi=r_hi,
                  ctx_lo=rng.choice([0, c_hi // 2, c_hi]), ctx_hi=c_hi)
        if kind == "decode":
            c = _case("", "plan", heads, lengths, **dec)
        elif kind == "prefill":
            c = _case("", "plan", heads, lengths, **pf)
        elif kind == "mixed":
            c = _case("", "plan", heads, lengths, **dec, **pf)
        elif kind == "static":
            c = _case("", "static", heads, lengths, **dict(dec, decodes=min(dec["decodes"], 64)), **dict(pf, chunks=min(pf["chunks"], 2)))
        elif kind == "graph":
            c = _case("", "graph", heads, lengths, **dict(dec, decodes=min(dec["decodes"], 64), lo=min(dec["lo"], 512), hi=min(dec["hi"], 4096)),
                      layers=rng.randint(2, 6))
        elif kind == "append":
            c = _case("", "append", heads, lengths, **dec, **pf)
        else:
            c = _case("", "copy", heads, lengths, **dict(dec, decodes=max(dec["decodes"], 2)))
            c["victims"] = max(1, c["decodes"] // rng.choice([2, 4, 8]))
        L = _lengths(c)
        if int(L.seq.sum()) <= MAX_KV_TOKENS and _pairs(L) <= MAX_PAIRS:
            return c


# ------------------------------------------------------------------------------------------------- lengths and sizes
def _lengths(c):
    """Chunks first, then decodes: query rows, cached tokens before the step, tokens after it, victims."""
    r = np.random.default_rng(c["lengths"])
    n, m = c["chunks"], c["decodes"]
    ctx = r.integers(c["ctx_lo"], c["ctx_hi"] + 1, size=n) if n else np.zeros(0, np.int64)
    rows = r.integers(c["rows_lo"], c["rows_hi"] + 1, size=n) if n else np.zeros(0, np.int64)
    if c["dist"] == "uniform":
        dec = r.integers(c["lo"], c["hi"] + 1, size=m)
    else:                       # lognormal around a quarter of the cap on short ranges, 2048 tokens on long ones
        median = min(2048, max(c["lo"], c["hi"] // 4))
        dec = np.clip(np.rint(np.exp(np.log(median) + 0.8 * r.standard_normal(m))), c["lo"], c["hi"]).astype(np.int64)
    q = np.concatenate([rows, np.ones(m, np.int64)]).astype(np.int32)
    ctx = np.concatenate([ctx, dec - 1]).astype(np.int32)
    qsl = np.zeros(n + m + 1, np.int32)
    qsl[1:] = np.cumsum(q)
    victims = np.sort(r.choice(n + m, size=min(c["victims"], n + m), replace=False)) if c["victims"] else np.zeros(0, np.int64)
    return SimpleNamespace(q=q, ctx=ctx, seq=(ctx + q).astype(np.int32), qsl=qsl, victims=victims, total_q=int(qsl[-1]))


def _pairs(L):
    """Visible (query row, key) pairs of the chunks."""
    q, ctx = L.q.astype(np.int64), L.ctx.astype(np.int64)
    return int(np.where(q > 1, q * ctx + q * (q + 1) // 2, 0).sum())


def work(case):
    L = _lengths(case)
    Hq, Hkv, hd = case["Hq"], case["Hkv"], case["hd"]
    token = 2 * Hkv * hd * 2                                    # bytes of one token's K and V
    nb = (L.seq.astype(np.int64) + BS - 1) // BS
    if case["entry"] == "copy":
        n = int(nb[L.victims].sum())
        return {"bytes": 2 * n * BS * token, "flops": 0}
    append = 2 * L.total_q * token                              # new vectors read, slots written
    if case["entry"] == "append":
        return {"bytes": append, "flops": 0}
    attn = int(L.seq.astype(np.int64).sum()) * token + int(nb.sum()) * 4 + 2 * L.total_q * Hq * hd * 2
    q, ctx = L.q.astype(np.int64), L.ctx.astype(np.int64)
    flops = 4 * Hq * hd * int((q * ctx + q * (q + 1) // 2).sum())
    n = case["layers"] if case["entry"] == "graph" else 1
    return {"bytes": n * (attn + (append if case["entry"] == "graph" else 0)), "flops": n * flops}


def tolerance(case):
    """bf16 inputs and outputs, weights rounded to bf16 before the second product, sums in fp32: measured 1.7e-3 to 2.3e-3
    away from 64 bits, of which the output's rounding alone is 1.7e-3.  Block copy and KV append move bytes."""
    if case["entry"] in ("append", "copy"):
        return "exact"
    return {"rel": 1e-2}


# ------------------------------------------------------------------------------------------------- inputs
def _inputs(case, seed):
    """Everything a step works on, on the GPU, from the seed alone (no code of this repository)."""
    L = _lengths(case)
    Hq, Hkv, hd = case["Hq"], case["Hkv"], case["hd"]
    g = torch.Generator(device="cuda").manual_seed(int(seed))
    normal = lambda *shape: torch.empty(shape, dtype=torch.bfloat16, device="cuda").normal_(0.0, 1.0, generator=g)
    nb = (L.seq.astype(np.int64) + BS - 1) // BS
    s = SimpleNamespace(case=case, L=L, nb=nb, num_blocks=int(nb.sum()) * 9 // 8 + 64)
    free = torch.randperm(s.num_blocks, generator=g, device="cuda").to(torch.int32).cpu().numpy()
    s.tables = np.full((len(nb), max(int(nb.max()), 1)), -1, np.int32)
    at = 0
    for i, n in enumerate(nb):
        s.tables[i, :n] = free[at:at + n]
        at += n
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()
    s.block_tables, s.seq_lens, s.query_start_loc, s.ctx_lens = dev(s.tables), dev(L.seq), dev(L.qsl), dev(L.ctx)
    layers = case["layers"] if case["entry"] == "graph" else 1
    s.k_cache = [normal(s.num_blocks, Hkv, hd // 8, BS, 8) for _ in range(layers)]
    s.v_cache = [normal(s.num_blocks, Hkv, hd, BS) for _ in range(layers)]
    if case["entry"] == "copy":
        ids = np.concatenate([s.tables[i, : nb[i]] for i in L.victims]).astype(np.int64)
        s.src_ids = dev(ids)
        n = len(ids) * 9 // 8 + 16
        s.dst_ids = torch.randperm(n, generator=g, device="cuda")[: len(ids)].contiguous()
        s.k_dst = torch.zeros((n, Hkv, hd // 8, BS, 8), dtype=torch.bfloat16, device="cuda")
        s.v_dst = torch.zeros((n, Hkv, hd, BS), dtype=torch.bfloat16, device="cuda")
        return s
    if case["entry"] in ("append", "graph"):
        s.k_new = [normal(L.total_q, Hkv, hd) for _ in range(layers)]
        s.v_new = [normal(L.total_q, Hkv, hd) for _ in range(layers)]
    if case["entry"] != "append":
        s.q = [normal(L.total_q, Hq, hd) for _ in range(layers)]
        s.out = [torch.zeros((L.total_q, Hq, hd), dtype=torch.bfloat16, device="cuda") for _ in range(layers)]
    return s


def prepare(case, seed):
    from paper_2511_21862_amd import binding as B

    s = _inputs(case, seed)
    s.B = B
    if case["entry"] == "static":
        return s
    s.ctx = B.Context(case["Hq"], case["Hkv"], case["hd"], BS, s.num_blocks, s.tables.shape[1])
    if case["entry"] == "graph":
        s.ctx.set_option("plan_persistent", 1)     # one plan serves all layers of the step
        s.ctx.plan(s.L.seq, s.L.qsl, s.L.ctx)
        side = torch.cuda.Stream()
        side.wait_stream(torch.cuda.current_stream())
        with torch.cuda.stream(side):
            _layers(s)                             # once eagerly, then into the graph
            side.synchronize()
            s.graph = torch.cuda.CUDAGraph()
            with torch.cuda.graph(s.graph, stream=side):
                _layers(s)
        torch.cuda.current_stream().wait_stream(side)
    return s


def _layers(s):
    for k, v, kn, vn, q, out in zip(s.k_cache, s.v_cache, s.k_new, s.v_new, s.q, s.out):
        s.ctx.kv_append(kn, vn, k, v, s.block_tables, s.query_start_loc, s.ctx_lens)
        s.ctx.attn_mixed(q, k, v, s.block_tables, s.seq_lens, s.query_start_loc, s.ctx_lens, out)


def run(state):
    s, c = state, state.case
    if c["entry"] == "plan":
        s.ctx.plan(s.L.seq, s.L.qsl, s.L.ctx)
        s.ctx.attn_mixed(s.q[0], s.k_cache[0], s.v_cache[0], s.block_tables, s.seq_lens, s.query_start_loc, s.ctx_lens, s.out[0])
        return s.out[0]
    if c["entry"] == "static":
        s.B.ooco_attn_mixed_static(c["Hq"], c["Hkv"], c["hd"], BS, s.tables.shape[1], 0.0, s.L.seq, s.L.qsl, s.L.ctx, s.q[0],
                                   s.k_cache[0], s.v_cache[0], s.block_tables, s.seq_lens, s.query_start_loc, s.ctx_lens, s.out[0],
                                   len(s.L.seq), s.L.total_q)
        return s.out[0]
    if c["entry"] == "graph":
        s.graph.replay()
        return {"out": s.out, "k": s.k_cache, "v": s.v_cache}
    if c["entry"] == "append":
        s.ctx.kv_append(s.k_new[0], s.v_new[0], s.k_cache[0], s.v_cache[0], s.block_tables, s.query_start_loc, s.ctx_lens)
        return {"k": s.k_cache[0], "v": s.v_cache[0]}
    s.ctx.kv_block_copy(s.k_cache[0], s.v_cache[0], s.k_dst, s.v_dst, s.src_ids, s.dst_ids)
    return {"k": s.k_dst, "v": s.v_dst}


# ------------------------------------------------------------------------------------------------- the same in 64 bits
def _append_exact(s, layer):
    """This step's vectors in their slots (a move of bytes: in the pools' own type)."""
    k, v = s.k_cache[layer].clone(), s.v_cache[layer].clone()
    blk, slot = [], []
    for i in range(len(s.nb)):
        t = int(s.L.ctx[i]) + np.arange(int(s.L.q[i]))
        blk.append(s.tables[i, t // BS])
        slot.append(t % BS)
    blk = torch.from_numpy(np.concatenate(blk).astype(np.int64)).cuda()
    slot = torch.from_numpy(np.concatenate(slot).astype(np.int64)).cuda()
    T, Hkv, hd = s.k_new[layer].shape
    k[blk, :, :, slot, :] = s.k_new[layer].reshape(T, Hkv, hd // 8, 8)
    v[blk, :, :, slot] = s.v_new[layer]
    return k, v


def _attn_exact(s, q, k_cache, v_cache):
    Hq, Hkv, hd = s.case["Hq"], s.case["Hkv"], s.case["hd"]
    g = Hq // Hkv
    out = torch.empty(q.shape, dtype=torch.float64, device="cuda")
    for i in range(len(s.nb)):
        ids = torch.from_numpy(s.tables[i, : s.nb[i]].astype(np.int64)).cuda()
        S, q0, n, ctx = int(s.L.seq[i]), int(s.L.qsl[i]), int(s.L.q[i]), int(s.L.ctx[i])
        kb, vb = k_cache.index_select(0, ids), v_cache.index_select(0, ids)
        for h in range(Hkv):
            k = kb[:, h].permute(1, 3, 0, 2).reshape(hd, -1)[:, :S].double().contiguous()        # [hd][tokens]
            v = vb[:, h].permute(0, 2, 1).reshape(-1, hd)[:S].double().contiguous()              # [tokens][hd]
            qh = q[q0:q0 + n, h * g:(h + 1) * g].double().reshape(n * g, hd)                     # [row][head of the group]
            sc = (qh @ k) / math.sqrt(hd)
            if n > 1:
                pos = ctx + torch.arange(n, device="cuda").repeat_interleave(g)
                sc.masked_fill_(torch.arange(S, device="cuda")[None, :] > pos[:, None], -math.inf)
            out[q0:q0 + n, h * g:(h + 1) * g] = (torch.softmax(sc, dim=1) @ v).reshape(n, g, hd)
    return out


def exact(case, seed):
    s = _inputs(case, seed)
    if case["entry"] == "copy":
        s.k_dst[s.dst_ids], s.v_dst[s.dst_ids] = s.k_cache[0][s.src_ids], s.v_cache[0][s.src_ids]
        return {"k": s.k_dst.double(), "v": s.v_dst.double()}
    if case["entry"] == "append":
        k, v = _append_exact(s, 0)
        return {"k": k.double(), "v": v.double()}
    if case["entry"] == "graph":
        r = {"out": [], "k": [], "v": []}
        for j in range(case["layers"]):
            k, v = _append_exact(s, j)
            r["out"].append(_attn_exact(s, s.q[j], k, v))
            r["k"].append(k.double())
            r["v"].append(v.double())
        return r
    return _attn_exact(s, s.q[0], s.k_cache[0], s.v_cache[0])
