"""GPU parity of prefill's per-request single pass (a tile holds rows of one
request and reads its group's prefix itself), of the plan without tiles (a
workgroup per row and head; nested groups and fp32 too) and of the plan the
library picks by itself, against the oracle."""
import ctypes
import math

import numpy as np
import pytest

from gpu_util import (assert_close, oracle_prefill_for, prefill_rows_for, problem_for, run_prefill, to_np,
                      workspace_untouched)
from paper_2405_19888_amd import load_library
from test_prefill_gpu import device_dict, prefill_case, say
from workloads import build_plan, make_batch, make_prefill_queries

pytestmark = pytest.mark.gpu

SPLIT, DIRECT, ROWS4, ROWS8 = 0, 2, 3, 19                     # ROWS8: eight waves per workgroup


def plan_of(plan, off):
    """The plan the library takes, as its own query tells."""
    prob, rows = problem_for(plan), prefill_rows_for(plan, off)
    return load_library().parrot_test_prefill_plan(ctypes.byref(prob), ctypes.byref(rows), int(plan.nested))


@pytest.mark.parametrize("setting", ["2", ""])
@pytest.mark.parametrize("dtype,D", [("float16", 128), ("bfloat16", 64)])
@pytest.mark.parametrize("kind", ["mixed", "wide_group", "long_rows", "many_runs", "single"])
def test_prefill_direct_parity(kind, dtype, D, setting, monkeypatch):
    monkeypatch.setenv("PARROT_PREFILL_SINGLE_PASS", setting)
    say("prefill direct", kind, dtype, D, repr(setting))
    plan, qr = prefill_case(kind, dtype, D)
    batch = make_batch(plan, seed=8)
    q, off = make_prefill_queries(plan, qr, seed=8)
    keep = []
    out, lse = run_prefill(plan, device_dict(batch, q, off), off, keep=keep)
    taken = plan_of(plan, off)
    assert taken == DIRECT or setting == ""
    assert workspace_untouched(keep[0]) == (taken != SPLIT), taken
    ref = oracle_prefill_for(batch, plan, q, off)
    assert_close(*to_np(out, lse), *ref, dtype, f"direct {kind} {dtype} D={D}")


@pytest.mark.parametrize("dtype,D", [("float16", 64), ("bfloat16", 128), ("float32", 64),
                                     ("float32", 128)])
@pytest.mark.parametrize("kind", ["mixed", "wide_group", "nested", "long_rows", "many_runs", "single"])
def test_prefill_rows_parity(kind, dtype, D, monkeypatch):
    monkeypatch.setenv("PARROT_PREFILL_SINGLE_PASS", "3")
    say("prefill rows", kind, dtype, D)
    plan, qr = prefill_case(kind, dtype, D)
    batch = make_batch(plan, seed=9)
    q, off = make_prefill_queries(plan, qr, seed=9)
    keep = []
    out, lse = run_prefill(plan, device_dict(batch, q, off), off, keep=keep)
    assert workspace_untouched(keep[0]), "a tiled plan ran"
    ref = oracle_prefill_for(batch, plan, q, off)
    assert_close(*to_np(out, lse), *ref, dtype, f"rows {kind} {dtype} D={D}")


@pytest.mark.parametrize("heads", [3, 4])                      # 252 workgroups: eight waves; 336: four
@pytest.mark.parametrize("parents", [[-1, -1, -1], [-1, 0, 1]])
@pytest.mark.parametrize("dtype,D", [("float16", 128), ("float32", 64)])
def test_prefill_rows_waves(dtype, D, parents, heads, monkeypatch):
    """Requests with no, one and more rows whose own ranges end at a block, at the
    eighth wave's block (128 tokens) or one token to either side, on one or three
    prefixes of such lengths."""
    monkeypatch.setenv("PARROT_PREFILL_SINGLE_PASS", "3")
    say("prefill rows waves", dtype, D, parents, heads)
    own = [127, 128, 129, 0, 1, 16, 257, 40, 1030, 17, 144, 300]
    new = [1, 2, 3, 0, 1, 16, 5, 0, 20, 17, 16, 3]
    plan = build_plan(heads=heads, head_dim=D, block_size=16, dtype=dtype,
                      group_of_request=[0, 1, 2, 2, 2, -1, 1, 0, 2, 0, -1, 2], prefix_lens=[128, 16, 129],
                      prefix_parents=parents, suffix_lens=own, sm_scale=1.0 / math.sqrt(D),
                      rng=np.random.default_rng(5))
    batch = make_batch(plan, seed=10)
    q, off = make_prefill_queries(plan, new, seed=10)
    assert plan_of(plan, off) == (ROWS8 if heads == 3 else ROWS4)
    keep = []
    out, lse = run_prefill(plan, device_dict(batch, q, off), off, keep=keep)
    assert workspace_untouched(keep[0]), "a tiled plan ran"
    ref = oracle_prefill_for(batch, plan, q, off)
    assert_close(*to_np(out, lse), *ref, dtype, f"rows waves {dtype} D={D} {parents} heads={heads}")


@pytest.mark.parametrize("R", [64, 65, 4096, 4097])
def test_prefill_rows_find_their_request(R, monkeypatch):
    """Few rows spread over many requests: the edges of the search for a row's
    request (64 at a time, then 64 x 64), the first and the last request among
    them, runs of requests without rows between."""
    monkeypatch.setenv("PARROT_PREFILL_SINGLE_PASS", "3")
    say("prefill rows of", R, "requests")
    rng = np.random.default_rng(R)
    own = rng.integers(1, 40, size=R)
    new = np.zeros(R, dtype=int)
    for r in {0, 1, 62, 63, R // 2, R - 2, R - 1} | set(rng.integers(0, R, 12).tolist()):
        new[r] = min(int(own[r]), 1 + r % 3)
    plan = build_plan(heads=2, head_dim=64, block_size=16, dtype="float16",
                      group_of_request=[(r % 3) - 1 for r in range(R)], prefix_lens=[40, 17],
                      suffix_lens=own.tolist(), sm_scale=0.125, rng=rng)
    batch = make_batch(plan, seed=R)
    q, off = make_prefill_queries(plan, new.tolist(), seed=R)
    out, lse = run_prefill(plan, device_dict(batch, q, off), off)
    ref = oracle_prefill_for(batch, plan, q, off)
    assert_close(*to_np(out, lse), *ref, "float16", f"rows of {R} requests")
