"""GPU parity of prefill's causal tiles where a wave's rows end: prompts whose
rows fill a wave (32 rows) or a tile (128 rows) exactly, by one less or one more,
whole or continued, beside a grouped request, over head counts that do and do
not divide evenly over the eight XCDs; on both plans, against the oracle."""
import math

import numpy as np
import pytest

from gpu_util import assert_close, oracle_prefill_for, run_prefill, to_np, workspace_untouched
from test_prefill_gpu import device_dict, say
from workloads import build_plan, make_batch, make_prefill_queries

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("path", ["single", "split"])
@pytest.mark.parametrize("heads", [1, 9])
@pytest.mark.parametrize("dtype,D", [("float16", 128), ("bfloat16", 64)])
def test_prefill_causal_tile_edges(dtype, D, heads, path, monkeypatch):
    monkeypatch.setenv("PARROT_PREFILL_SINGLE_PASS", "1" if path == "single" else "0")
    say("prefill causal edges", dtype, D, heads, path)
    own = [1, 31, 32, 33, 127, 128, 129, 160, 257, 300, 40, 385]
    rows = [1, 31, 32, 33, 127, 128, 129, 1, 257, 33, 40, 96]
    plan = build_plan(heads=heads, head_dim=D, block_size=16, dtype=dtype,
                      group_of_request=[-1] * 10 + [0, 0], prefix_lens=[45], suffix_lens=own,
                      sm_scale=1.0 / math.sqrt(D), rng=np.random.default_rng(3))
    batch = make_batch(plan, seed=3)
    q, off = make_prefill_queries(plan, rows, seed=3)
    keep = []
    out, lse = run_prefill(plan, device_dict(batch, q, off), off, keep=keep)
    assert workspace_untouched(keep[0]) == (path == "single"), "unexpected prefill path"
    ref = oracle_prefill_for(batch, plan, q, off)
    assert_close(*to_np(out, lse), *ref, dtype, f"causal edges {dtype} D={D} heads={heads} {path}")
