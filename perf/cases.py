"""The work this library does for a serving engine, as cases that can be timed.

One case is one attention call of one layer: a decode step of a batch (plain,
with this step's token appended, over nested prefixes, without a workspace, or
reading each request's prefix by itself) or the prefill of a batch's new prompt
tokens.  Lengths and group structure come from the case alone, so the work of a
case is known without its seed; values, the physical order of the KV blocks and
the order of the requests come from the seed.

Fields of a case
  entry       decode | append | noalloc | per_request | nested | prefill
  dtype       cache type: float32 | float16 | bfloat16
  heads, head_dim
  groups      shared prefixes; prefix_lo .. prefix_hi tokens each
  grouped     requests that read one (Zipf shares with exponent skew)
  ungrouped   requests with no shared prefix, contexts of free_lo .. free_hi
  own_lo/hi   own tokens of a grouped request
  levels      > 1: group 0 is the root of a tree of that depth; the other
              groups add sub_lo .. sub_hi tokens each and hold the requests
  rows_lo/hi  prefill: new tokens per request, at most its own tokens (0: all)
  lengths     seed of the lengths
"""
import math
import random

import numpy as np
import torch

from paper_2405_19888_amd import binding

BLOCK = 16
DTYPES = {"float32": torch.float32, "float16": torch.float16, "bfloat16": torch.bfloat16}


def case(name, entry, dtype, heads, head_dim, **kw):
    c = {"entry": entry, "dtype": dtype, "heads": heads, "head_dim": head_dim,
         "groups": 0, "grouped": 0, "skew": 0.0, "prefix_lo": 1, "prefix_hi": 1,
         "ungrouped": 0, "free_lo": 1, "free_hi": 1, "own_lo": 1, "own_hi": 1,
         "levels": 1, "sub_lo": 1, "sub_hi": 1, "rows_lo": 0, "rows_hi": 0, "lengths": 0}
    if name:
        c["name"] = name
    c.update(kw)
    return c


def listed():
    return [
        # the smallest call: 4 requests on a 128-token prompt, 4 heads, fp32;
        # launches and memory round trips count, not bytes
        case("decode_tiny_f32", "decode", "float32", 4, 64, groups=1, grouped=4,
             prefix_lo=128, prefix_hi=128, own_lo=16, own_hi=32),
        # a handful of interactive chats, each step appending its token: four
        # on one short system prompt, three with prompts of their own
        case("decode_chat_append", "append", "float16", 32, 128, groups=1, grouped=4,
             prefix_lo=317, prefix_hi=317, own_lo=20, own_hi=200, ungrouped=3,
             free_lo=40, free_hi=700),
        # an ordinary batch: 32 requests on a 2048-token prompt
        case("decode_g32_p2048", "decode", "float16", 32, 128, groups=1, grouped=32,
             prefix_lo=2048, prefix_hi=2048, own_lo=64, own_hi=512),
        # the first steps after 64 contexts forked from a long system prompt:
        # the prefix is nearly all there is to read
        case("decode_fork_g64_p6000", "decode", "float16", 32, 128, groups=1, grouped=64,
             prefix_lo=6000, prefix_hi=6000, own_lo=1, own_hi=64),
        # a smaller model (64-wide heads) serving several applications
        case("decode_apps_d64", "decode", "bfloat16", 20, 64, groups=5, grouped=110, skew=0.7,
             prefix_lo=300, prefix_hi=3000, own_lo=16, own_hi=900, ungrouped=9,
             free_lo=100, free_hi=2500),
        # one layer of the full mixed serving step, the largest decode call
        case("decode_mixed_288", "decode", "bfloat16", 32, 128, groups=8, grouped=256, skew=1.1,
             prefix_lo=512, prefix_hi=4096, own_lo=32, own_hi=1024, ungrouped=32,
             free_lo=544, free_hi=5120),
        # two levels of sharing: a system prompt, then few-shot blocks
        case("decode_nested_8x8", "nested", "float16", 32, 128, groups=9, grouped=64, levels=2,
             prefix_lo=6000, prefix_hi=6000, sub_lo=256, sub_hi=256, own_lo=64, own_hi=512),
        # a batch above 1024 requests on one tensor-parallel share of the heads
        case("decode_batch_1500", "decode", "bfloat16", 8, 128, groups=24, grouped=1300, skew=0.8,
             prefix_lo=150, prefix_hi=1800, own_lo=1, own_hi=400, ungrouped=200,
             free_lo=50, free_hi=1500),
        # the smallest prefill: the tiny batch's whole prompts, fp32
        case("prefill_tiny_f32", "prefill", "float32", 4, 64, groups=1, grouped=4,
             prefix_lo=128, prefix_hi=128, own_lo=16, own_hi=32),
        # the Fill of one long prompt that nothing shares yet
        case("prefill_prompt_6000", "prefill", "bfloat16", 32, 128, ungrouped=1,
             free_lo=5987, free_hi=5987),
        # 64 contexts forked from a 6000-token prompt, each continuing its own
        # prompt by 16 tokens (chunked prefill)
        case("prefill_fork_q16", "prefill", "float16", 32, 128, groups=1, grouped=64,
             prefix_lo=6000, prefix_hi=6000, own_lo=100, own_hi=1000, rows_lo=16, rows_hi=16),
        # the same contexts filling their whole prompts, the largest call
        case("prefill_fork_whole", "prefill", "float16", 32, 128, groups=1, grouped=64,
             prefix_lo=6000, prefix_hi=6000, own_lo=100, own_hi=1000),
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    """One more case of the ranges the listed ones stand for."""
    while True:
        entry = rng.choice(["decode"] * 4 + ["append", "append", "noalloc", "per_request", "nested"]
                           + ["prefill"] * 5)
        dtype = rng.choice(["float16"] * 4 + ["bfloat16"] * 4 + ["float32"])
        c = case(None, entry, dtype, rng.choice([4, 5, 8, 12, 16, 20, 25, 32, 32, 40]),
                 rng.choice([128, 128, 128, 64]), lengths=rng.randrange(1 << 20))
        prefill = entry == "prefill"
        requests = _log_int(rng, 1, 96 if prefill else 1600)
        c["ungrouped"] = requests if rng.random() < 0.15 else rng.randint(0, requests // 4)
        c["grouped"] = requests - c["ungrouped"]
        if entry == "nested" or (prefill and rng.random() < 0.2 and c["grouped"] > 1):
            c["levels"] = rng.choice([2, 2, 3])
            c["grouped"] = max(2, c["grouped"])
        if c["grouped"]:
            c["groups"] = _log_int(rng, 1, max(1, min(24, c["grouped"])))
            c["skew"] = round(rng.uniform(0.0, 1.2), 2)
        if c["levels"] > 1:
            c["groups"] = max(2, c["groups"])
            c["sub_lo"] = _log_int(rng, 1, 300)
            c["sub_hi"] = c["sub_lo"] + _log_int(rng, 1, 400)
        c["prefix_lo"] = _log_int(rng, 16, 3000)
        c["prefix_hi"] = c["prefix_lo"] + (0 if rng.random() < 0.4 else _log_int(rng, 1, 4000))
        c["own_lo"] = _log_int(rng, 1, 200)
        c["own_hi"] = c["own_lo"] + _log_int(rng, 1, 1000)
        c["free_lo"] = _log_int(rng, 10, 1500)
        c["free_hi"] = c["free_lo"] + _log_int(rng, 1, 3000)
        if prefill and rng.random() < 0.5:
            c["rows_lo"] = _log_int(rng, 1, 128)
            c["rows_hi"] = c["rows_lo"] + (0 if rng.random() < 0.5 else _log_int(rng, 1, 128))
        if entry == "noalloc":       # its partial results have to fit the library's fixed array
            c["prefix_hi"] = min(c["prefix_hi"], 2000)
            c["prefix_lo"] = min(c["prefix_lo"], c["prefix_hi"])
            c["free_lo"], c["free_hi"] = min(c["free_lo"], 1000), min(c["free_hi"], 1900)
            if requests * c["heads"] > 500:
                continue
        w = work(c)
        most = 2.0e12 if dtype != "float32" else 5.0e10
        if w["bytes"] < 3.0e9 and w["flops"] < most:
            return c


# ------------------------------------------------------------------- layout
def _zipf(total, n, s):
    w = [k ** -s for k in range(1, n + 1)]
    raw = [total * x / sum(w) for x in w]
    base = [int(x) for x in raw]
    for i in sorted(range(n), key=lambda i: base[i] - raw[i])[: total - sum(base)]:
        base[i] += 1
    return base


def layout(c):
    """Lengths and groups of a case: (group of request, prefix lengths, own
    lengths, parents, new rows), in an order the seed then shuffles."""
    rng = random.Random("%s %d %d" % (c["entry"], c["lengths"], c["grouped"] + c["ungrouped"]))
    ng = c["groups"]
    parents, depth = [-1] * ng, [1] * ng
    if c["levels"] > 1:
        for g in range(1, ng):
            # the deepest chain first, then anywhere that leaves room below
            p = g - 1 if g < c["levels"] else rng.choice([x for x in range(g) if depth[x] < c["levels"]])
            parents[g], depth[g] = p, depth[p] + 1
        plen = [rng.randint(c["prefix_lo"], c["prefix_hi"])]
        plen += [rng.randint(c["sub_lo"], c["sub_hi"]) for _ in range(ng - 1)]
        gid = [1 + i % (ng - 1) for i in range(c["grouped"])]
        if c["levels"] == 2:
            parents = [-1] + [0] * (ng - 1)
    else:
        plen = [rng.randint(c["prefix_lo"], c["prefix_hi"]) for _ in range(ng)]
        sizes = _zipf(c["grouped"], ng, c["skew"]) if ng else []
        gid = [g for g, n in enumerate(sizes) for _ in range(n)]
    own = [rng.randint(c["own_lo"], c["own_hi"]) for _ in gid]
    own += [rng.randint(c["free_lo"], c["free_hi"]) for _ in range(c["ungrouped"])]
    gid += [-1] * c["ungrouped"]
    rows = [s if not c["rows_hi"] else min(s, rng.randint(c["rows_lo"], c["rows_hi"])) for s in own]
    return gid, plen, own, parents, rows


def _chain(g, parents):
    out = []
    while g >= 0:
        out.append(g)
        g = parents[g]
    return out[::-1]


def work(c):
    """K and V of every prefix and of every request's own tokens once, the
    queries and the results; two products over the keys each query sees."""
    gid, plen, own, parents, rows = layout(c)
    elt = 4 if c["dtype"] == "float32" else 2
    hd = c["heads"] * c["head_dim"]
    read = {a for g in gid for a in _chain(g, parents)}
    tokens = sum(plen[g] for g in read) + sum(own)
    keys, nq = 0, 0
    for g, s, n in zip(gid, own, rows):
        p = sum(plen[a] for a in _chain(g, parents))
        if c["entry"] == "prefill":
            keys += n * (p + s - n) + n * (n + 1) // 2
            nq += n
        else:
            keys += p + s
            nq += 1
    extra = 4 * len(gid) * hd * elt if c["entry"] == "append" else 0   # new K/V in and out
    return {"bytes": 2 * tokens * hd * elt + 2 * nq * hd * elt + 4 * nq * c["heads"] + extra,
            "flops": 4 * keys * hd}


# -------------------------------------------------------------------- inputs
def _inputs(c, seed):
    """Tables and values of one call, on the GPU, from the seed."""
    gid, plen, own, parents, rows = layout(c)
    host = np.random.default_rng([int(seed), 77])
    order = host.permutation(len(gid))
    gid, own, rows = ([x[i] for i in order] for x in (gid, own, rows))
    h, d, dt = c["heads"], c["head_dim"], DTYPES[c["dtype"]]
    dev = torch.device("cuda")

    def tables(lens):
        n = [-(-x // BLOCK) for x in lens]
        total = sum(n)
        ids = host.permutation(total).astype(np.int32)
        t = np.zeros((len(lens), max(n + [1])), dtype=np.int32)
        at = 0
        for i, k in enumerate(n):
            t[i, :k] = ids[at:at + k]
            at += k
        return t, max(total, 1)

    ptab, npre = tables(plen)
    stab, nown = tables(own)
    gen = torch.Generator(device=dev).manual_seed(int(seed) * 7919 + 13)

    def normal(*shape):
        return torch.randn(*shape, generator=gen, device=dev, dtype=dt)

    def ints(x):
        return torch.tensor(np.asarray(x, dtype=np.int32), device=dev)

    off = np.concatenate([[0], np.cumsum(rows)]).astype(np.int32)
    prefill = c["entry"] == "prefill"
    t = {"prefix_k": normal(npre, h, BLOCK, d), "prefix_v": normal(npre, h, BLOCK, d),
         "suffix_k": normal(nown, h, BLOCK, d), "suffix_v": normal(nown, h, BLOCK, d),
         "prefix_tables": ints(ptab), "prefix_lens": ints(plen), "suffix_tables": ints(stab),
         "suffix_lens": ints(own), "group_ids": ints(gid), "prefix_parents": ints(parents)}
    if prefill:
        t["q_rows"], t["query_offsets"] = normal(int(off[-1]), h, d), ints(off)
    else:
        t["q"] = normal(len(gid), h, d)
    if c["entry"] == "append":
        t["k_new"], t["v_new"] = normal(len(gid), h, d), normal(len(gid), h, d)
    nested = c["levels"] > 1
    prob = binding.problem_from_host(
        num_heads=h, head_dim=d, block_size=BLOCK, dtype=dt, sm_scale=d ** -0.5, group_ids=gid,
        prefix_lens=plen, suffix_lens=own, prefix_table_stride=ptab.shape[1],
        suffix_table_stride=stab.shape[1], num_prefix_blocks=npre, num_suffix_blocks=nown,
        prefix_parents=parents if nested else None)
    host_side = {"gid": gid, "plen": plen, "own": own, "parents": parents, "rows": rows,
                 "off": off, "ptab": ptab, "stab": stab}
    return t, prob, host_side


def prepare(c, seed):
    t, prob, at = _inputs(c, seed)
    nested = c["levels"] > 1
    if c["entry"] == "prefill":
        rows = binding.prefill_rows_from_host(at["off"], at["gid"], prob.num_groups,
                                              at["parents"] if nested else None)
        own = binding.Prefiller(prob, rows)
        call = own.bind(t, nested=nested)
    elif c["entry"] == "noalloc":
        own = binding.Decoder(prob)
        call = None
    else:
        own = binding.Decoder(prob)
        call = own.bind(t, shared=c["entry"] != "per_request", nested=c["entry"] == "nested",
                        append=c["entry"] == "append")
    return {"case": c, "t": t, "problem": prob, "buffers": own, "call": call}


def run(state):
    t, own = state["t"], state["buffers"]
    if state["call"] is None:
        binding.parrot_shared_prefix_decode_noalloc(
            state["problem"], t["q"], t["prefix_k"], t["prefix_v"], t["suffix_k"], t["suffix_v"],
            t["prefix_tables"], t["prefix_lens"], t["suffix_tables"], t["suffix_lens"],
            t["group_ids"], own.out, own.lse)
    else:
        state["call"]()
    got = {"out": own.out, "lse": own.lse}
    if state["case"]["entry"] == "append":
        got["suffix_k"], got["suffix_v"] = t["suffix_k"], t["suffix_v"]
    return got


# --------------------------------------------------------------- the results
def tolerance(c):
    """Relative error two correct implementations may show: about four times
    what the outputs are off exact() (3e-7, 2.9e-4 and 2.1e-3)."""
    return {"float32": {"rel": 1.5e-6}, "float16": {"rel": 1.2e-3}, "bfloat16": {"rel": 9e-3}}[c["dtype"]]


def exact(c, seed):
    """The same outputs from plain torch in 64 bits."""
    t, _, at = _inputs(c, seed)
    parents, off, scale = at["parents"], at["off"], c["head_dim"] ** -0.5
    h, d = c["heads"], c["head_dim"]
    dev = torch.device("cuda")
    prefill, append = c["entry"] == "prefill", c["entry"] == "append"
    if append:
        r = torch.arange(len(at["own"]), device=dev)
        last = t["suffix_lens"].long() - 1
        blk = t["suffix_tables"].long()[r, last // BLOCK]
        t["suffix_k"][blk, :, last % BLOCK] = t["k_new"]
        t["suffix_v"][blk, :, last % BLOCK] = t["v_new"]

    def tokens(pool, table, n):          # [H, n, D] in 64 bits
        ids = torch.tensor(table[: -(-n // BLOCK)].astype(np.int64), device=dev)
        return pool[ids].double().transpose(0, 1).reshape(h, -1, d)[:, :n].contiguous()

    def prefix(g):
        a = [(tokens(t["prefix_k"], at["ptab"][x], at["plen"][x]),
              tokens(t["prefix_v"], at["ptab"][x], at["plen"][x])) for x in _chain(g, parents)]
        return [torch.cat([p[i] for p in a], 1) for i in (0, 1)]

    q = t["q_rows"] if prefill else t["q"]
    out = torch.empty(q.shape, dtype=torch.float64, device=dev)
    lse = torch.empty(q.shape[:2], dtype=torch.float64, device=dev)
    held = None
    for r in sorted(range(len(at["gid"])), key=lambda r: at["gid"][r]):
        g, s = at["gid"][r], at["own"][r]
        if held is None or held[0] != g:
            held = None
            held = (g, prefix(g)) if g >= 0 else (g, None)
        k, v = (tokens(t[x], at["stab"][r], s) for x in ("suffix_k", "suffix_v"))
        p = 0
        if held[1] is not None:
            p = held[1][0].shape[1]
            k, v = torch.cat([held[1][0], k], 1), torch.cat([held[1][1], v], 1)
        lo, hi = (int(off[r]), int(off[r + 1])) if prefill else (r, r + 1)
        kt = k.transpose(1, 2).contiguous()
        step = max(1, int(2e8 / (h * (p + s))))
        for a in range(lo, hi, step):
            b = min(hi, a + step)
            x = torch.matmul(q[a:b].double().transpose(0, 1).contiguous(), kt) * scale   # [H, rows, N]
            if prefill:
                seen = p + s - (hi - lo) + 1 + torch.arange(a - lo, b - lo, device=dev)
                hide = torch.arange(p + s, device=dev)[None, :] >= seen[:, None]
                x.masked_fill_(hide[None], -math.inf)
            top = torch.logsumexp(x, -1)
            out[a:b] = torch.matmul(torch.exp_(x.sub_(top[..., None])), v).transpose(0, 1)
            lse[a:b] = top.transpose(0, 1)
    got = {"out": out, "lse": lse}
    if append:
        got["suffix_k"], got["suffix_v"] = t["suffix_k"], t["suffix_v"]
    return got
