"""GPU parity for the prefill of forked contexts: each request's new rows
against its group chain's prefixes and, causally, its own tokens, through
the C ABI, against the float64 oracle.

Every case prints its name before touching the GPU, validates the device
inputs (row offsets included) before the call, and NaN-poisons outputs and
workspace first; unused cache slots hold NaN.
"""
import math
import sys
from dataclasses import replace

import numpy as np
import pytest
import torch

from gpu_util import (assert_close, oracle_prefill_for, prefill_rows_for, problem_for,
                      run_prefill, to_np, workspace_untouched)
from paper_2405_19888_amd import parrot_prefill_single_pass
from workloads import build_plan, make_batch, make_prefill_queries

pytestmark = pytest.mark.gpu

DTYPES = ["float16", "bfloat16", "float32"]


def say(*a):
    print("[case]", *a, flush=True)
    sys.stdout.flush()


def prefill_case(kind, dtype, D, seed=0):
    """(plan, per-request row counts)."""
    rng = np.random.default_rng(seed)
    scale = 1.0 / math.sqrt(D)
    if kind == "mixed":
        # groups of several sizes, ungrouped requests, whole prompts, chunks of
        # prompts, no rows; own lengths across several 256-token chunks
        gor = [0] * 5 + [1] * 3 + [2] + [-1] * 3
        sl = [1, 17, 300, 64, 0, 33, 520, 7, 129, 700, 1, 65]
        qr = [1, 17, 100, 64, 0, 5, 520, 0, 129, 300, 1, 64]
        plan = build_plan(heads=3, head_dim=D, block_size=16, dtype=dtype, group_of_request=gor,
                          prefix_lens=[700, 33, 1], suffix_lens=sl, sm_scale=scale,
                          shuffle=True, rng=rng)
        return plan, [qr[i] for i in plan_order(plan, sl)]
    if kind == "wide_group":
        # 150+ rows read one prefix: three row tiles that cut through requests
        gor = [0] * 9
        sl = [40, 1, 70, 16, 17, 2, 33, 64, 9]
        plan = build_plan(heads=2, head_dim=D, block_size=16, dtype=dtype, group_of_request=gor,
                          prefix_lens=[1100], suffix_lens=sl, sm_scale=scale, shuffle=True, rng=rng)
        return plan, list(plan.suffix_lens)
    if kind == "nested":
        # 0 <- 1 <- 3, 0 <- 2; members at every level, one ungrouped
        gor = [3, 3, 1, 2, 2, 0, -1, 1]
        sl = [90, 5, 130, 1, 64, 20, 300, 0]
        plan = build_plan(heads=4, head_dim=D, block_size=16, dtype=dtype, group_of_request=gor,
                          prefix_lens=[600, 48, 257, 16], prefix_parents=[-1, 0, 0, 1],
                          suffix_lens=sl, sm_scale=scale, shuffle=True, rng=rng)
        return plan, [min(int(s), 70) for s in plan.suffix_lens]
    if kind == "long_rows":
        # one request with many row tiles and own chunks, next to a short one
        plan = build_plan(heads=2, head_dim=D, block_size=16, dtype=dtype,
                          group_of_request=[0, 0], prefix_lens=[300], suffix_lens=[1000, 3],
                          sm_scale=scale, rng=rng)
        return plan, [1000, 3]
    if kind == "many_runs":
        # 160 requests of one group with one row each (at the last own token):
        # the first row tile holds 128 requests' rows, one run per request
        sl = [int(x) for x in rng.integers(1, 50, size=160)]
        plan = build_plan(heads=2, head_dim=D, block_size=16, dtype=dtype,
                          group_of_request=[0] * 160, prefix_lens=[300], suffix_lens=sl,
                          sm_scale=scale, shuffle=True, rng=rng)
        return plan, [1] * 160
    if kind == "single":
        plan = build_plan(heads=1, head_dim=D, block_size=16, dtype=dtype, group_of_request=[-1],
                          prefix_lens=[], suffix_lens=[1], sm_scale=scale, rng=rng)
        return plan, [1]
    raise ValueError(kind)


def plan_order(plan, sl):
    """Map the drawn (shuffled) requests back to the row recipe: request r of
    the plan has suffix length sl[i] for the returned i (first unused match)."""
    used, out = set(), []
    for s in plan.suffix_lens:
        i = next(j for j, x in enumerate(sl) if x == int(s) and j not in used)
        used.add(i)
        out.append(i)
    return out


def device_dict(batch, q, off):
    dev = batch.to("cuda")
    dev["q_rows"] = q.to("cuda")
    dev["query_offsets"] = torch.from_numpy(np.ascontiguousarray(off)).to("cuda")
    return dev


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("dtype", DTYPES)
@pytest.mark.parametrize("kind", ["mixed", "wide_group", "nested", "long_rows", "many_runs",
                                  "single"])
def test_prefill_parity(kind, dtype, D):
    say("prefill", kind, dtype, D)
    plan, qr = prefill_case(kind, dtype, D)
    batch = make_batch(plan, seed=5)
    q, off = make_prefill_queries(plan, qr, seed=5)
    out, lse = run_prefill(plan, device_dict(batch, q, off), off)
    ref = oracle_prefill_for(batch, plan, q, off)
    assert_close(*to_np(out, lse), *ref, dtype, f"prefill {kind} {dtype} D={D}")


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("dtype", ["float16", "bfloat16"])
@pytest.mark.parametrize("kind", ["mixed", "wide_group", "long_rows", "many_runs", "single"])
def test_prefill_single_pass_parity(kind, dtype, D, monkeypatch):
    """The single-pass path (each group tile sees the whole prefix, then its
    rows' own tokens run by run; ungrouped requests' tiles their own tokens)
    on the same cases, forced where the split plan would cut the ranges into
    chunks.  It writes no partial results: the poisoned workspace stays as it
    was, which shows that this path ran."""
    monkeypatch.setenv("PARROT_PREFILL_SINGLE_PASS", "1")
    say("prefill single pass", kind, dtype, D)
    plan, qr = prefill_case(kind, dtype, D)
    batch = make_batch(plan, seed=5)
    q, off = make_prefill_queries(plan, qr, seed=5)
    keep = []
    out, lse = run_prefill(plan, device_dict(batch, q, off), off, keep=keep)
    assert workspace_untouched(keep[0]), "the split path ran"
    assert parrot_prefill_single_pass(problem_for(plan), prefill_rows_for(plan, off))
    ref = oracle_prefill_for(batch, plan, q, off)
    assert_close(*to_np(out, lse), *ref, dtype, f"single pass {kind} {dtype} D={D}")


@pytest.mark.parametrize("kind,dtype", [("nested", "float16"), ("mixed", "float32")])
def test_prefill_single_pass_not_taken(kind, dtype, monkeypatch):
    """Nested groups and fp32 caches keep the split path (partial results and
    the merge) even when the single pass is asked for."""
    monkeypatch.setenv("PARROT_PREFILL_SINGLE_PASS", "1")
    say("prefill single pass not taken", kind, dtype)
    plan, qr = prefill_case(kind, dtype, 64)
    batch = make_batch(plan, seed=6)
    q, off = make_prefill_queries(plan, qr, seed=6)
    keep = []
    out, lse = run_prefill(plan, device_dict(batch, q, off), off, keep=keep)
    assert not workspace_untouched(keep[0])
    ref = oracle_prefill_for(batch, plan, q, off)
    assert_close(*to_np(out, lse), *ref, dtype, f"split {kind} {dtype}")


def test_prefill_rows_as_decode():
    """One row per request at its last own token is a decode step: the prefill
    result equals the decode entry point's on the same queries."""
    from gpu_util import run_gpu
    say("prefill one row per request vs decode")
    plan, _ = prefill_case("mixed", "float16", 128)
    batch = make_batch(plan, seed=2)
    qr = [1 if int(s) > 0 else 0 for s in plan.suffix_lens]
    q, off = make_prefill_queries(plan, qr, seed=2)
    out, lse = run_prefill(plan, device_dict(batch, q, off), off)
    have = [r for r in range(plan.num_requests) if qr[r]]
    qd = batch.q.clone()
    for i, r in enumerate(have):
        qd[r] = q[i]
    dev = batch.to("cuda")
    dev["q"] = qd.to("cuda")
    dout, dlse = run_gpu(plan, dev)
    o, l = to_np(out, lse)
    do, dl = to_np(dout, dlse)
    assert np.max(np.abs(o - do[have])) <= 2e-3
    assert np.max(np.abs(l - dl[have]) / np.maximum(1, np.abs(dl[have]))) <= 1e-4


def test_prefill_validation_catches_bad_rows():
    from paper_2405_19888_amd import ParrotError, parrot_validate_prefill_inputs
    say("prefill validation")
    plan, qr = prefill_case("mixed", "float16", 64)
    batch = make_batch(plan)
    q, off = make_prefill_queries(plan, qr)
    prob = problem_for(plan)
    rows = prefill_rows_for(plan, off)
    scratch = torch.zeros(16, dtype=torch.int32, device="cuda")
    dev = device_dict(batch, q, off)

    def check(offsets, rows_=rows, msg=""):
        d = dict(dev, query_offsets=torch.from_numpy(np.asarray(offsets, np.int32)).to("cuda"))
        with pytest.raises(ParrotError, match=msg):
            parrot_validate_prefill_inputs(prob, rows_, d["query_offsets"], d["prefix_tables"],
                                           d["prefix_lens"], None, d["suffix_tables"],
                                           d["suffix_lens"], d["group_ids"], scratch)
    bad = off.copy()
    bad[0] = 1
    check(bad, msg="query_offsets")
    # a request below the longest own length gets one row more than its own
    # tokens (the row bound on the host still holds)
    r = int(np.argmin(np.where(plan.suffix_lens > 0, plan.suffix_lens, 1 << 30)))
    bad = off.copy()
    bad[r + 1:] += int(plan.suffix_lens[r]) - qr[r] + 1       # one row more than own tokens
    from paper_2405_19888_amd import make_prefill_rows
    check(bad, make_prefill_rows(int(bad[-1]), int(np.diff(bad).max()), rows.max_group_rows + 600),
          msg="suffix length")
    check(off, make_prefill_rows(rows.num_query_rows, rows.max_query_rows,
                                 rows.max_group_rows - 1), msg="max_group_rows")


@pytest.mark.parametrize("name,path", [("prefill", "auto"), ("prefill", "split"),
                                       ("prefill_q16", "auto")])
def test_prefill_workload_sampled(name, path, monkeypatch):
    """The benchmark's prefill workloads at full size, in the launch the
    benchmark times (whole prompts: the single pass; 16 rows per request: the
    split plan, whose chunks fill the device), and whole prompts on the split
    path too: sampled rows (first and last rows of requests, rows at row-tile
    edges, random rows) against the oracle, and every row finite."""
    if path == "split":
        monkeypatch.setenv("PARROT_PREFILL_SINGLE_PASS", "0")
    else:
        monkeypatch.delenv("PARROT_PREFILL_SINGLE_PASS", raising=False)
    from workloads import (get_config, make_device_layer, make_device_prefill_queries,
                           make_plan, prefill_rows)
    cfg = get_config(name)
    plan = make_plan(cfg)
    qr = prefill_rows(plan, cfg.prefill_rows, None)
    say("prefill workload", cfg.name, int(qr.sum()), "rows")
    dev = make_device_layer(plan, 0, "cuda", seed=cfg.seed)
    dev["q_rows"], dev["query_offsets"] = make_device_prefill_queries(plan, qr, "cuda", cfg.seed, 0)
    off = dev["query_offsets"].cpu().numpy()
    keep = []
    out, lse = run_prefill(plan, dev, off, keep=keep)
    single = name == "prefill" and path == "auto"
    assert workspace_untouched(keep[0]) == single, "unexpected prefill path"
    assert parrot_prefill_single_pass(problem_for(plan), prefill_rows_for(plan, off)) == single
    o, l = to_np(out, lse)
    assert np.all(np.isfinite(o)) and np.all(np.isfinite(l))
    rng = np.random.default_rng(1)
    reqs = sorted(set(rng.choice(plan.num_requests, size=6, replace=False).tolist()) | {0, plan.num_requests - 1})
    rows = set()
    for r in reqs:
        a, b = int(off[r]), int(off[r + 1])
        if b > a:
            rows |= {a, b - 1, min(b - 1, a + 127), min(b - 1, a + 128)}
    rows |= set(rng.integers(0, int(off[-1]), size=6).tolist())
    rows = sorted(rows)
    host = type("B", (), {})()
    host.k_pool, host.v_pool = dev["k_pool"].cpu(), dev["v_pool"].cpu()
    ref = oracle_prefill_for(host, plan, dev["q_rows"].cpu(), off, rows=rows)
    assert_close(o[rows], l[rows], *ref, plan.dtype, f"{cfg.name} sampled rows")


@pytest.mark.parametrize("chunked", [False, True])
def test_prefill_contexts_from_store(chunked):
    """Fill through the host context store: prompts that fork from a shared
    system prompt and three task prefixes (and one that shares nothing) are
    registered, and the prefill entry point computes their own tokens' rows
    (all of them, or the last part of each prompt) with the store's group
    forest, against the oracle."""
    from paper_2405_19888_amd.context import ContextStore
    from test_nested_gpu import plan_from_store
    say("prefill from context store, chunked =", chunked)
    rng = np.random.default_rng(8)
    st = ContextStore(block_size=16, num_blocks=800)
    sysp = rng.integers(0, 1000, size=300).tolist()
    tasks = [rng.integers(0, 1000, size=n).tolist() for n in (50, 77, 120)]
    ctxs = []
    for i in range(10):
        t = tasks[i % 3]
        own = rng.integers(0, 1000, size=int(rng.integers(1, 200))).tolist()
        ctxs.append(st.fill(sysp + t + own, [300, 300 + len(t)]))
    ctxs.append(st.fill(rng.integers(0, 1000, size=150).tolist(), []))
    batch = st.build_batch(ctxs, pad_block=st.num_blocks)
    plan = plan_from_store(batch, st, heads=4, head_dim=128, dtype="bfloat16")
    data = make_batch(plan, seed=9)
    S = plan.suffix_lens
    qr = [int(s) - (int(s) // 3 if chunked else 0) for s in S]
    q, off = make_prefill_queries(plan, qr, seed=9)
    out, lse = run_prefill(plan, device_dict(data, q, off), off)
    ref = oracle_prefill_for(data, plan, q, off)
    assert_close(*to_np(out, lse), *ref, "bfloat16", f"store prefill chunked={chunked}")


@pytest.mark.parametrize("dtype,D", [("float16", 128), ("bfloat16", 64)])
def test_prefill_long_prefix_max_chunks(dtype, D):
    """A 9000-token prefix read by enough row tiles that the prefix chunk is
    the largest one (8192 tokens, a 512-block table) and the prefix splits in
    two; own prompts of 256 rows.  Sampled rows against the oracle."""
    say("prefill long prefix", dtype, D)
    rng = np.random.default_rng(3)
    plan = build_plan(heads=32, head_dim=D, block_size=16, dtype=dtype,
                      group_of_request=[0] * 8, prefix_lens=[9000], suffix_lens=[256] * 8,
                      sm_scale=1.0 / math.sqrt(D), shuffle=True, rng=rng)
    batch = make_batch(plan, seed=4)
    q, off = make_prefill_queries(plan, [256] * 8, seed=4)
    out, lse = run_prefill(plan, device_dict(batch, q, off), off)
    o, l = to_np(out, lse)
    assert np.all(np.isfinite(o)) and np.all(np.isfinite(l))
    rows = sorted({0, 1, 127, 128, 255, 256, 1000, 1023, 1024, 2047} |
                  set(rng.integers(0, 2048, size=6).tolist()))
    ref = oracle_prefill_for(batch, plan, q, off, rows=rows)
    assert_close(o[rows], l[rows], *ref, dtype, f"long prefix {dtype} D={D}")


@pytest.mark.parametrize("dtype,D", [("float16", 128), ("bfloat16", 64)])
def test_prefill_single_pass_longest_ranges(dtype, D, monkeypatch):
    """The single pass at its largest ranges: an 8192-token prefix (a
    512-block table) and own prompts of up to 8192 tokens whose last 300 and
    1000 tokens are rows; one group and one ungrouped request.  Sampled rows
    against the oracle."""
    monkeypatch.setenv("PARROT_PREFILL_SINGLE_PASS", "1")
    say("prefill single pass longest ranges", dtype, D)
    rng = np.random.default_rng(11)
    sl = [8192, 5000, 300, 8000]
    plan = build_plan(heads=8, head_dim=D, block_size=16, dtype=dtype,
                      group_of_request=[0, 0, 0, -1], prefix_lens=[8192], suffix_lens=sl,
                      sm_scale=1.0 / math.sqrt(D), rng=rng)
    qr = [1000, 300, 300, 1000]
    batch = make_batch(plan, seed=12)
    q, off = make_prefill_queries(plan, qr, seed=12)
    keep = []
    out, lse = run_prefill(plan, device_dict(batch, q, off), off, keep=keep)
    assert workspace_untouched(keep[0]), "the split path ran"
    o, l = to_np(out, lse)
    assert np.all(np.isfinite(o)) and np.all(np.isfinite(l))
    rows = sorted({0, 127, 128, 999, 1000, 1299, 1300, 1599, 1600, 2599} |
                  set(rng.integers(0, int(off[-1]), size=6).tolist()))
    ref = oracle_prefill_for(batch, plan, q, off, rows=rows)
    assert_close(o[rows], l[rows], *ref, dtype, f"single pass longest {dtype} D={D}")


# ---------------------------------------------------------------- probes
# The graded tolerances cannot see one key too many or too few in a long row
# (its weight is about 1/N).  Two probes pin the visible keys of every row in
# both plans: with q = 0 every visible key has weight exactly 1/N, so the lse
# is ln N to fp32 rounding; a key made to dominate one row's logits (logit
# 40) must become that row's output when the row sees it, and must not when
# it lies after the row's position.

PLANS = {"single": "1", "split": "0", "direct": "2", "rows": "3"}


def _prefix_len(plan, r):
    g = int(plan.group_ids[r])
    return int(plan.prefix_lens[g]) if g >= 0 else 0


@pytest.mark.parametrize("dtype", ["float16", "bfloat16"])
@pytest.mark.parametrize("path", PLANS)
def test_prefill_zero_query_probe(path, dtype, monkeypatch):
    from oracle.attention import prefill_positions
    monkeypatch.setenv("PARROT_PREFILL_SINGLE_PASS", PLANS[path])
    for kind in ("mixed", "wide_group", "long_rows"):
        say("prefill zero-query probe", path, dtype, kind)
        plan, qr = prefill_case(kind, dtype, 128)
        batch = make_batch(plan, seed=5)
        q, off = make_prefill_queries(plan, qr, seed=5)
        q.zero_()
        keep = []
        out, lse = run_prefill(plan, device_dict(batch, q, off), off, keep=keep)
        assert workspace_untouched(keep[0]) == (path != "split"), "unexpected prefill path"
        ref_o, ref_l = oracle_prefill_for(batch, plan, q, off)
        n = np.array([_prefix_len(plan, r) + p + 1 for r, p in prefill_positions(off, plan.suffix_lens)])
        assert np.allclose(ref_l, np.log(n)[:, None], rtol=1e-12, atol=1e-15)
        o, l = to_np(out, lse)
        assert np.max(np.abs(l - ref_l) / np.maximum(1.0, np.abs(ref_l))) < 1e-6, kind
        # the output is the mean of the visible values, exact in fp32 up to a
        # few ulps; its rounding to the cache type (half an ulp) dominates, and
        # rows with one or two keys have means of any size: a relative bound
        half_ulp = 2.0 ** -8 if dtype == "bfloat16" else 2.0 ** -11
        bound = half_ulp * np.maximum(np.abs(ref_o), 2.0 ** -6) + 1e-5
        assert np.all(np.abs(o - ref_o) <= bound), kind


SCALE_CASES = ([(k, d, "split") for k in ("negative_scale", "zero_scale", "ramp")
                for d in ("float16", "bfloat16", "float32")]
               + [(k, d, "single") for k in ("negative_scale", "zero_scale", "ramp")
                  for d in ("float16", "bfloat16")]
               + [("ramp", "float16", "direct"), ("negative_scale", "bfloat16", "direct"),
                  ("ramp", "bfloat16", "rows"), ("ramp", "float32", "rows"),
                  ("negative_scale", "float16", "rows")])


@pytest.mark.parametrize("kind,dtype,path", SCALE_CASES)
def test_prefill_scale_and_logit_range(kind, dtype, path, monkeypatch):
    """sm_scale < 0 and sm_scale = 0, and prefix logits that climb from 0 to
    200 over 1100 tokens (the softmax reference moves several times per
    stage run), on both prefill plans, against the oracle."""
    monkeypatch.setenv("PARROT_PREFILL_SINGLE_PASS", PLANS[path])
    say("prefill scale / logit range", kind, dtype, path)
    D = 128
    scale = {"negative_scale": -1 / math.sqrt(D), "zero_scale": 0.0, "ramp": 1 / math.sqrt(D)}[kind]
    plan, qr = prefill_case("wide_group", dtype, D)
    plan = replace(plan, sm_scale=scale)
    batch = make_batch(plan, seed=5)
    q, off = make_prefill_queries(plan, qr, seed=5)
    if kind == "ramp":
        # every row shares a query direction u (plus noise); prefix key j is
        # ramp_j / (scale |u|^2) u plus noise, so each row's logit of key j is
        # about ramp_j = 200 j / P
        g, P = 0, int(plan.prefix_lens[0])
        td = q.dtype
        qf = q.float()
        k = batch.k_pool.float()
        u = torch.randn((plan.heads, D), generator=torch.Generator().manual_seed(9))
        qf = u[None] + 0.05 * qf
        for j in range(P):
            blk, slot = int(plan.prefix_tables[g][j // plan.block_size]), j % plan.block_size
            for h in range(plan.heads):
                c = 200.0 * j / P / (scale * float(u[h] @ u[h]))
                k[blk, h, slot] = c * u[h] + 0.05 * k[blk, h, slot]
        q = qf.to(td)
        batch = type(batch)(plan=plan, q=batch.q, k_pool=k.to(td), v_pool=batch.v_pool)
    keep = []
    out, lse = run_prefill(plan, device_dict(batch, q, off), off, keep=keep)
    assert workspace_untouched(keep[0]) == (path != "split"), "unexpected prefill path"
    ref = oracle_prefill_for(batch, plan, q, off)
    # fp32 caches: logits near 200 carry about sqrt(D) 2^-24 200 = 1.4e-4 of
    # rounding from their fp32 dot products, and so does each weight relatively;
    # with |v| up to about 4 the output error stays below 6e-4
    loose = kind == "ramp" and dtype == "float32"
    assert_close(*to_np(out, lse), *ref, dtype, f"prefill {kind} {dtype} {path}",
                 out_tol=6e-4 if loose else None, rel_l2=2e-4 if loose else None)


@pytest.mark.parametrize("path", PLANS)
def test_prefill_spike_probe(path, monkeypatch):
    from oracle.attention import prefill_positions
    monkeypatch.setenv("PARROT_PREFILL_SINGLE_PASS", PLANS[path])
    dtype, B = "float16", 16
    plan, qr = prefill_case("wide_group", dtype, 128)
    base = make_batch(plan, seed=4)
    q, off = make_prefill_queries(plan, qr, seed=4)
    pos = prefill_positions(off, plan.suffix_lens)
    T = int(off[-1])
    firsts = [int(off[r]) for r in range(plan.num_requests) if off[r + 1] > off[r]]
    rows = sorted({0, 127, 128, T - 1, firsts[len(firsts) // 2]})
    for t in rows:
        r, p = pos[t]
        g, P, S = int(plan.group_ids[r]), _prefix_len(plan, r), int(plan.suffix_lens[r])
        for j in sorted({0, 15, 16, P - 1, P, P + p - 1, P + p, P + p + 1}):
            if not 0 <= j < P + S:
                continue
            say("prefill spike probe", path, "row", t, "key", j)
            k = base.k_pool.clone()
            if j < P:
                blk, slot = int(plan.prefix_tables[g][j // B]), j % B
            else:
                blk, slot = int(plan.suffix_tables[r][(j - P) // B]), (j - P) % B
            for h in range(plan.heads):
                qv = q[t, h].double()
                k[blk, h, slot] = (40.0 / (plan.sm_scale * float(qv @ qv)) * qv).to(k.dtype)
            batch = type(base)(plan=plan, q=base.q, k_pool=k, v_pool=base.v_pool)
            out, lse = run_prefill(plan, device_dict(batch, q, off), off)
            o, l = to_np(out, lse)
            v = base.v_pool[blk, :, slot].double().numpy()
            if j <= P + p:                               # visible: the key takes over
                s = plan.sm_scale * (q[t].double() * k[blk, :, slot].double()).sum(-1).numpy()
                assert np.max(np.abs(o[t] - v)) <= 1e-3 * max(1.0, np.abs(v).max()), (t, j)
                assert np.max(np.abs(l[t] - s) / np.abs(s)) < 1e-5, (t, j)
            else:                                        # after the row: no effect on it
                ref_o, ref_l = oracle_prefill_for(batch, plan, q, off, rows=[t])
                assert_close(o[[t]], l[[t]], ref_o, ref_l, dtype, f"spike after row {t}")
                assert np.max(np.abs(o[t] - v)) > 0.1, (t, j)


@pytest.mark.parametrize("path", PLANS)
def test_prefill_bitwise_reproducible(path, monkeypatch):
    """The same inputs and plan give bitwise-identical output and lse (no
    atomics or order-dependent sums in either plan)."""
    monkeypatch.setenv("PARROT_PREFILL_SINGLE_PASS", PLANS[path])
    say("prefill reproducibility", path)
    plan, qr = prefill_case("mixed", "bfloat16", 128)
    batch = make_batch(plan, seed=8)
    q, off = make_prefill_queries(plan, qr, seed=8)
    dev = device_dict(batch, q, off)
    a = [t.clone() for t in run_prefill(plan, dev, off)]
    b = run_prefill(plan, dev, off)
    assert torch.equal(a[0], b[0]) and torch.equal(a[1], b[1])


def test_prefill_one_call_torch_api():
    """shared_prefix_prefill on plain torch tensors sizes the problem and the
    row counts itself and matches the oracle."""
    from paper_2405_19888_amd import shared_prefix_prefill
    say("prefill one-call torch API")
    plan, qr = prefill_case("mixed", "bfloat16", 64)
    batch = make_batch(plan, seed=9)
    q, off = make_prefill_queries(plan, qr, seed=9)
    dev = device_dict(batch, q, off)
    out, lse = shared_prefix_prefill(
        dev["q_rows"], dev["query_offsets"], dev["k_pool"], dev["v_pool"], dev["k_pool"],
        dev["v_pool"], dev["prefix_tables"], dev["prefix_lens"], dev["suffix_tables"],
        dev["suffix_lens"], dev["group_ids"], sm_scale=plan.sm_scale)
    torch.cuda.synchronize()
    ref = oracle_prefill_for(batch, plan, q, off)
    assert_close(*to_np(out, lse), *ref, "bfloat16", "prefill one-call")
